// Streaming optimisers for f: Three Sieves (the paper cites it in Sec. 2 and
// runs it beside greedy in the Sec. 6 case study) and Sieve Streaming (named
// with greedy in Sec. 2 and Sec. 4.1 as an optimiser that scores many sets
// per step).
//
// Both walk a stream of points of V. Three Sieves keeps one summary S and a
// threshold v that walks down the grid of guesses (1+eps)^i in [m, k m]
// (m = max_e f({e})) after T consecutive rejections; Sieve Streaming keeps
// one summary per guess. A point e joins summary S (guess v) while |S| < k
// and
//     Delta(e|S) >= (v/2 - f(S)) / (k - |S|),
//     Delta(e|S) = |V|^-1 sum_v max(0, m_v - d(v, e))      (Sec. 3, Sec. 4.1)
// with m_v the running minima of S u {e0}.
//
// What a decision needs of the arriving point e is the distance vector
// d(., e) over the ground set, and that vector does not depend on any
// summary. So the stream is processed in stretches of points: one launch
// computes the float64 distances of a stretch's points to every ground point
// (direct differences, the same definition as the float64 re-score and the
// oracle), and one launch with a workgroup per summary walks the stretch in
// stream order, each workgroup clamping and summing its own minima against
// each distance row, deciding, and on acceptance lowering its minima and
// recomputing f(S) -- all in float64 on the device, so every decision is a
// float64 one in every distance dtype, and no host round trip happens
// between the first launch and the result. Distance rows are prefetched into
// registers several points ahead (they do not depend on the decisions), so
// the sequential walk waits only on its own reductions.
#include <math.h>

#include <algorithm>
#include <vector>

#include "ebc_internal.h"

using namespace ebc;

namespace {

constexpr int kST = 256;             // threads of the stream kernels
constexpr int kDI = 32;              // stream points and ground points per distance tile
constexpr int kDK = 8;               // dimensions per LDS stage of the distance tile
constexpr int kDW = 4;               // waves of a distance tile, each a quarter of the dimension
constexpr int kRegMax = 16;          // ground points per thread kept in registers (n_pad <= 4096)
constexpr size_t kStretchBytes = size_t(256) << 20;  // distance rows of one default stretch, at most

// One summary's state, in the caller's scratch.
struct Summary {
    int32_t cnt;      // members so far
    int32_t t;        // consecutive rejections (Three Sieves)
    int32_t gi;       // index of the current guess (Three Sieves)
    int32_t pad;
    int64_t full_at;  // stream position of the k-th acceptance, -1 before
    double fS;        // f of the summary
};

struct Result {
    int32_t count;     // members of the returned summary
    int32_t best;      // its index (0 for Three Sieves)
    int64_t examined;  // points taken from the stream
};

__device__ __forceinline__ int64_t stream_row(const int32_t* __restrict__ order, int64_t p) {
    return order ? int64_t(order[p]) : p;
}

// Lane exchanges of a butterfly without LDS: halves and quarters of the wave
// by the permlane swaps, within a row of 16 lanes by rotations. A rotation by
// 4 stands for lane ^ 4 once lanes 8 apart hold the same value, and so on.
template <int OFF>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    if constexpr (OFF == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    } else if constexpr (OFF == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (threadIdx.x & 16) ? r[0] : r[1];
    } else {
        return __builtin_amdgcn_update_dpp(0, v, 0x120 + OFF, 0xf, 0xf, false);  // row_ror:OFF
    }
}
template <int OFF>
__device__ __forceinline__ double add_xor(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint64_t lo = lane_xor<OFF>(uint32_t(u)), hi = lane_xor<OFF>(uint32_t(u >> 32));
    return v + __longlong_as_double((hi << 32) | lo);
}
template <int CTRL>
__device__ __forceinline__ double add_quad(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint64_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, uint32_t(u), CTRL, 0xf, 0xf, false));
    const uint64_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, uint32_t(u >> 32), CTRL, 0xf, 0xf, false));
    return v + __longlong_as_double((hi << 32) | lo);
}
// Lane ^ 4: the banks of 4 lanes of a row take their neighbour bank, even
// banks by row_shl:4, odd ones by row_shr:4.
__device__ __forceinline__ uint32_t four_apart(uint32_t v) {
    const uint32_t t = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0x5, false);
    return __builtin_amdgcn_update_dpp(t, v, 0x114, 0xf, 0xa, false);
}
__device__ __forceinline__ double add_four_apart(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint64_t lo = four_apart(uint32_t(u)), hi = four_apart(uint32_t(u >> 32));
    return v + __longlong_as_double((hi << 32) | lo);
}
// float64 sum over the 64 lanes, in every lane: pairs 32 lanes apart, then 16,
// ... 1 (one fixed association). Through the LDS permute each of the six
// steps would wait about 130 cycles; the walk makes one such sum per point.
__device__ __forceinline__ double wave_sum(double v) {
    v = add_xor<32>(v);
    v = add_xor<16>(v);
    v = add_xor<8>(v);
    v = add_xor<4>(v);
    v = add_xor<2>(v);
    return add_xor<1>(v);
}

// The sums of P values (P = 2, 4 or 8) over the wave together: every exchange
// halves the values a lane still carries, so all of them take about as long as
// one (10 exchanges for 8 values instead of 48). The same pairs are added as
// by wave_sum. Lane l ends with the sum of value sums_index<P>(l).
template <int P>
__device__ __forceinline__ int sums_index(int lane) {
    return P == 8 ? (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1)
                  : (P == 4 ? (lane >> 5) * 2 + ((lane >> 4) & 1) : lane >> 5);
}
__device__ __forceinline__ double swap_add32(double x, double y) {  // lanes below 32: x, the others: y
    const uint64_t a = __double_as_longlong(x), b = __double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane32_swap(uint32_t(a), uint32_t(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(uint32_t(a >> 32), uint32_t(b >> 32), false, false);
    return __longlong_as_double((uint64_t(hi[0]) << 32) | lo[0]) + __longlong_as_double((uint64_t(hi[1]) << 32) | lo[1]);
}
__device__ __forceinline__ double swap_add16(double x, double y) {  // even rows of 16 lanes: x, odd rows: y
    const uint64_t a = __double_as_longlong(x), b = __double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane16_swap(uint32_t(a), uint32_t(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(uint32_t(a >> 32), uint32_t(b >> 32), false, false);
    return __longlong_as_double((uint64_t(hi[0]) << 32) | lo[0]) + __longlong_as_double((uint64_t(hi[1]) << 32) | lo[1]);
}
template <int P>
__device__ __forceinline__ double wave_sums(const double (&p)[P]) {
    static_assert(P == 2 || P == 4 || P == 8, "pairs halve down to one value");
    double v;
    if constexpr (P == 8) {
        double a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = swap_add32(p[i], p[i + 4]);
        const double b0 = swap_add16(a[0], a[2]), b1 = swap_add16(a[1], a[3]);
        const bool up = (threadIdx.x & 8) != 0;
        const double send = up ? b0 : b1;
        const uint64_t u = __double_as_longlong(send);
        const uint64_t lo = lane_xor<8>(uint32_t(u)), hi = lane_xor<8>(uint32_t(u >> 32));
        v = (up ? b1 : b0) + __longlong_as_double((hi << 32) | lo);
    } else if constexpr (P == 4) {
        v = add_xor<8>(swap_add16(swap_add32(p[0], p[2]), swap_add32(p[1], p[3])));
    } else {
        v = add_xor<8>(add_xor<16>(swap_add32(p[0], p[1])));
    }
    // within 8 lanes
    v = add_four_apart(v);
    v = add_quad<0x4e>(v);     // quad_perm 2 3 0 1: lane ^ 2
    return add_quad<0xb1>(v);  // quad_perm 1 0 3 2: lane ^ 1
}

// Distances of stream points pos + [0, cnt) to every ground point, float64
// direct differences, into D [cnt][n_pad] (columns >= n are not written). A
// workgroup computes a 32 x 32 tile; wave w sums quarter w of the dimension in
// dimension order, and the four sums are added in order. Lane (ti, tv)
// owns stream points 4 ti .. 4 ti + 3 and ground points 4 tv .. 4 tv + 3, both
// sides staged through the wave's own LDS as float64, 8 dimensions at a time
// (the next stage's values loaded into registers while the current one is
// used; no barrier, the wave alone reads what it wrote). Bound: float64 vector
// instructions, a subtraction and an fma per pair and dimension (97 us at 1000
// x 3524), at two waves per SIMD; one wave summing the whole dimension left
// each SIMD with one wave, which waits 10 cycles per instruction. In index
// order the distances are symmetric, bit for bit, and a tile whose mirror
// lies in the stretch is computed once and written twice. 1000 x 3524: 585 ->
// 290 us (8 waves and eighths 277 us, but idle waves in short rows; 16
// dimensions a stage 302 us). Nothing runs once every summary is full.
constexpr int kDS = kDI + 2;  // LDS row stride
// Orders a wave's LDS writes before its lanes' reads (and the other way round).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int METRIC>
__global__ void __launch_bounds__(64 * kDW) k_stream_dist(const float* __restrict__ x, int64_t n, int32_t d,
                                                     const int32_t* __restrict__ order, int64_t pos, int32_t cnt,
                                                     int64_t n_pad, double* __restrict__ D,
                                                     const Summary* __restrict__ sm, int32_t ns, int32_t k) {
    __shared__ __align__(16) double stage[kDW][2][2][kDK][kDS];  // [wave][buffer][side][dimension][row]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double (*A)[kDK][kDS] = &stage[wave][0][0];  // side 0 of buffer b: A[2 b], side 1: A[2 b + 1]
    bool open = false;
    for (int j = lane; j < ns; j += 64) open |= sm[j].cnt < k;
    if (__builtin_amdgcn_ballot_w64(open) == 0) return;

    const int64_t v0 = int64_t(blockIdx.x) * kDI;
    const int i0 = int(blockIdx.y) * kDI;
    // mirrored tiles: stream point i is ground point pos + i, tiles aligned on both sides
    const bool mirror = !order && pos % kDI == 0;
    const bool inside = mirror && v0 >= pos && v0 < pos + cnt;  // the tile's columns are stream points of the stretch
    if (inside && v0 < pos + i0) return;                        // written by its mirror
    const bool twice = inside && v0 > pos + i0;

    const int tv = lane & 7, ti = lane >> 3;
    // loader: row lr of each side, dimensions lk .. lk + 3 of a stage; rows
    // past the end repeat the last one (their distances are not stored)
    const int lr = lane >> 1, lk = 4 * (lane & 1);
    const float* rows[2];
    rows[0] = x + stream_row(order, pos + (i0 + lr < cnt ? i0 + lr : cnt - 1)) * d;
    rows[1] = x + (v0 + lr < n ? v0 + lr : n - 1) * d;
    const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    float reg[2][4];
    // no branch around a load: all of a stage's are in flight together.
    // Dimensions past d read an earlier one and are stored as 0.
    auto load = [&](int k0) {
        const int kk = k0 + lk;
        if (vec) {
            const int at = kk < d ? kk : 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 t = *reinterpret_cast<const float4*>(rows[h] + at);
                reg[h][0] = t.x;
                reg[h][1] = t.y;
                reg[h][2] = t.z;
                reg[h][3] = t.w;
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) reg[h][q] = rows[h][kk + q < d ? kk + q : 0];
        }
    };
    auto store = [&](int buf, int k0) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) A[2 * buf + h][lk + q][lr] = double(k0 + lk + q < d ? reg[h][q] : 0.0f);
    };

    double acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = 0.0;
    // stages of this wave's part of the dimension
    const int nk_all = (d + kDK - 1) / kDK;
    const int per = (nk_all + kDW - 1) / kDW;
    const int c0 = wave * per;
    const int c1 = c0 + per < nk_all ? c0 + per : nk_all;
    if (c0 < c1) {
        load(c0 * kDK);
        store(c0 & 1, c0 * kDK);
    }
    for (int c = c0; c < c1; ++c) {
        const int buf = c & 1;
        wave_lds_fence();  // this stage is written; the other one has been read
        if (c + 1 < c1) load((c + 1) * kDK);
#pragma unroll 4
        for (int kk = 0; kk < kDK; ++kk) {
            const double2 a01 = *reinterpret_cast<const double2*>(&A[2 * buf][kk][4 * ti]);
            const double2 a23 = *reinterpret_cast<const double2*>(&A[2 * buf][kk][4 * ti + 2]);
            const double2 b01 = *reinterpret_cast<const double2*>(&A[2 * buf + 1][kk][4 * tv]);
            const double2 b23 = *reinterpret_cast<const double2*>(&A[2 * buf + 1][kk][4 * tv + 2]);
            const double a[4] = {a01.x, a01.y, a23.x, a23.y}, b[4] = {b01.x, b01.y, b23.x, b23.y};
            // all subtractions before the sums that need them: a lone wave
            // waits for every instruction that uses the one before it
            double df[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) df[q] = a[q / 4] - b[q % 4];
            asm volatile(""
                         : "+v"(df[0]), "+v"(df[1]), "+v"(df[2]), "+v"(df[3]), "+v"(df[4]), "+v"(df[5]), "+v"(df[6]),
                           "+v"(df[7]), "+v"(df[8]), "+v"(df[9]), "+v"(df[10]), "+v"(df[11]), "+v"(df[12]),
                           "+v"(df[13]), "+v"(df[14]), "+v"(df[15]));
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                if (METRIC == 1)
                    acc[q / 4][q % 4] += fabs(df[q]);
                else
                    acc[q / 4][q % 4] = fma(df[q], df[q], acc[q / 4][q % 4]);
            }
        }
        if (c + 1 < c1) store(buf ^ 1, (c + 1) * kDK);
    }
    // the parts of each pair, added in order; wave w takes 4 of a lane's 16 pairs
    static_assert(kDW * 16 * 64 * sizeof(double) <= sizeof(stage), "the sums fit the stages");
    double* red = &stage[0][0][0][0][0];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) red[(wave * 16 + q) * 64 + lane] = acc[q / 4][q % 4];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 16 / kDW; ++h) {
        const int q = wave * (16 / kDW) + h;
        double sum = red[q * 64 + lane];
#pragma unroll
        for (int t = 1; t < kDW; ++t) sum += red[(t * 16 + q) * 64 + lane];
        const int i = i0 + 4 * ti + q / 4;
        const int64_t v = v0 + 4 * tv + q % 4;
        if (i >= cnt || v >= n) continue;
        D[int64_t(i) * n_pad + v] = sum;
        if (twice && v < pos + cnt) D[(v - pos) * n_pad + pos + i] = sum;
    }
}

// Arguments of the decision walk over one stretch.
struct WalkArgs {
    const double* D;       // [cnt][n_pad] distances of the stretch
    int64_t n, n_pad;
    int32_t cnt;           // points in the stretch
    int32_t k;
    int64_t pos;           // stream position of the stretch's first point
    const int32_t* order;  // stream indices (null: 0, 1, ...)
    const double* grid;    // guesses, largest first
    int32_t J;             // guesses
    int32_t pad;
    int64_t T;             // Three Sieves: rejections before the next guess; 0: Sieve Streaming
    const DevState* dst;   // L({e0}) of the dataset
    Summary* sm;           // [summaries]
    double* M;             // [summaries][n_pad] running minima
    int32_t* sel;          // [summaries][k] members
    double* fv;            // [summaries][k] f after each acceptance
};

// The rule's bound on a gain, for the summary's present state.
__device__ __forceinline__ double bound_of(const WalkArgs& w, int j, const Summary& s) {
    const double v = w.T > 0 ? w.grid[s.gi] : w.grid[j];
    return (0.5 * v - s.fS) / double(w.k - s.cnt);
}

// The rule for one point, given its float64 gain sum over V (uniform across
// the workgroup): gsum / n >= bound. Returns true when the point joins. The
// division is made only where the product leaves the comparison open (within
// 8 roundings); it would otherwise be on the path of every point.
__device__ __forceinline__ bool decide(const WalkArgs& w, double bound, double gsum) {
    const double n = double(w.n);
    const double edge = bound * n, slack = fabs(edge) * 0x1p-50;
    if (gsum > edge + slack) return true;
    if (gsum < edge - slack) return false;
    return gsum / n >= bound;
}

// Bookkeeping after a decision; returns true once the summary is full.
__device__ __forceinline__ bool record(const WalkArgs& w, int j, Summary& s, bool take, int i, double msum) {
    if (take) {
        const double fS = w.dst->l0 - msum / double(w.n);
        if (threadIdx.x == 0) {
            w.sel[int64_t(j) * w.k + s.cnt] = int32_t(stream_row(w.order, w.pos + i));
            w.fv[int64_t(j) * w.k + s.cnt] = fS;
        }
        s.fS = fS;
        s.cnt += 1;
        s.t = 0;
        if (s.cnt == w.k) {
            s.full_at = w.pos + i;
            return true;
        }
    } else if (w.T > 0) {
        if (++s.t >= w.T && s.gi + 1 < w.J) {
            s.gi += 1;
            s.t = 0;
        }
    }
    return false;
}

// Workgroup-uniform float64 sum of one value per thread: lane 0 of each wave
// writes its wave's sum, then every thread adds the four in wave order.
__device__ __forceinline__ double block_sum(double v, double* slot) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((slot[0] + slot[1]) + slot[2]) + slot[3];
}

// Decision walk, one workgroup per summary, thread t owning ground points
// t + 256 r (r < R) with their minima in registers. The gains of P points are
// summed together against the present minima (their reductions overlap; one
// barrier) and decided in stream order; an accepted point lowers the minima,
// and the points after it are summed again. Accepted points are few (at most
// k), so a point costs about an eighth of a reduction's latency instead of
// all of it. The rows of the next 2 P points are in flight. 1000 points, 41
// summaries: 640 -> 217 us.
template <int R, int P>
__global__ void __launch_bounds__(kST) k_stream_walk(WalkArgs w) {
    const int j = blockIdx.x;
    Summary s = w.sm[j];
    if (s.cnt >= w.k) return;
    __shared__ __align__(16) double red[2][P][4];
    __shared__ double fred[4];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    double* __restrict__ m = w.M + int64_t(j) * w.n_pad;
    double mr[R];
    bool ok[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t v = tid + int64_t(kST) * r;
        ok[r] = v < w.n;
        mr[r] = ok[r] ? m[v] : 0.0;
    }
    auto load_rows = [&](int i0, double (&dst)[P][R]) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int i = i0 + q < w.cnt ? i0 + q : w.cnt - 1;  // rows past the stretch are not decided
            const double* __restrict__ src = w.D + int64_t(i) * w.n_pad + tid;
#pragma unroll
            for (int r = 0; r < R; ++r) dst[q][r] = ok[r] ? src[kST * r] : 0.0;
        }
    };
    bool changed = false, stop = false;
    int par = 0;
    double bound = bound_of(w, j, s);
    auto walk = [&](int i0, const double (&row)[P][R]) {
        int from = 0;  // first point not yet decided
        while (!stop && from < P && i0 + from < w.cnt) {
            double p[P];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                p[q] = 0.0;
#pragma unroll
                for (int r = 0; r < R; ++r) p[q] += fmax(0.0, mr[r] - row[q][r]);
            }
            const double mine = wave_sums<P>(p);
            if ((lane & (P == 8 ? 7 : (P == 4 ? 15 : 31))) == 0) red[par][sums_index<P>(lane)][wave] = mine;
            __syncthreads();
            // lane q decides point q; up to the next guess (Three Sieves) the
            // bound does not change with the rejections
            const int q = lane < P ? lane : P - 1;
            const double g = ((red[par][q][0] + red[par][q][1]) + red[par][q][2]) + red[par][q][3];
            int taken = P;
            while (from < P && i0 + from < w.cnt) {
                int to = w.cnt - i0 < P ? w.cnt - i0 : P;
                const bool steps = w.T > 0 && s.gi + 1 < w.J;
                if (steps && w.T - s.t < to - from) to = from + int(w.T - s.t);
                const uint64_t hit =
                    __builtin_amdgcn_ballot_w64(lane >= from && lane < to && decide(w, bound, g));
                const int last = hit ? __builtin_ctzll(hit) : to;
                if (w.T > 0) s.t += last - from;  // rejections
                from = last;
                if (hit) {
                    taken = last;
                    break;
                }
                if (steps && s.t >= w.T) {
                    s.gi += 1;
                    s.t = 0;
                    bound = bound_of(w, j, s);
                }
            }
            par ^= 1;
            if (taken == P) return;
            double qs = 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                double at = row[0][r];
#pragma unroll
                for (int q = 1; q < P; ++q) at = taken == q ? row[q][r] : at;
                mr[r] = fmin(mr[r], at);
                qs += mr[r];
            }
            const double msum = block_sum(qs, fred);
            changed = true;
            stop = record(w, j, s, true, i0 + taken, msum);
            if (!stop) bound = bound_of(w, j, s);
            from = taken + 1;
        }
    };
    double rowA[P][R], rowB[P][R];
    load_rows(0, rowA);
    load_rows(P, rowB);
    for (int i0 = 0; i0 < w.cnt && !stop; i0 += 2 * P) {
        walk(i0, rowA);
        load_rows(i0 + 2 * P, rowA);
        walk(i0 + P, rowB);
        load_rows(i0 + 3 * P, rowB);
    }
    if (changed) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (ok[r]) m[tid + int64_t(kST) * r] = mr[r];
    }
    if (tid == 0) w.sm[j] = s;
}

// The same walk for ground sets above 256 * kRegMax points: minima in the
// scratch, rows read as they are used (same per-thread summation order).
__global__ void __launch_bounds__(kST) k_stream_walk_big(WalkArgs w) {
    const int j = blockIdx.x;
    Summary s = w.sm[j];
    if (s.cnt >= w.k) return;
    __shared__ double red[2][4];
    __shared__ double fred[4];
    const int tid = threadIdx.x;
    double* __restrict__ m = w.M + int64_t(j) * w.n_pad;
    for (int i = 0; i < w.cnt; ++i) {
        const double* __restrict__ row = w.D + int64_t(i) * w.n_pad;
        double p = 0.0;
        for (int64_t v = tid; v < w.n; v += kST) p += fmax(0.0, m[v] - row[v]);
        const double g = block_sum(p, red[i & 1]);
        const bool take = decide(w, bound_of(w, j, s), g);
        double msum = 0.0;
        if (take) {
            double qs = 0.0;
            for (int64_t v = tid; v < w.n; v += kST) {
                const double mv = fmin(m[v], row[v]);
                m[v] = mv;
                qs += mv;
            }
            msum = block_sum(qs, fred);
        }
        if (record(w, j, s, take, i, msum)) break;
    }
    if (tid == 0) w.sm[j] = s;
}

// Every summary starts at S = {}: minima m0 = d(., e0), empty state.
__global__ void __launch_bounds__(kST) k_stream_init(const double* __restrict__ m0, int64_t n_pad, int32_t ns,
                                                     double* __restrict__ M, Summary* __restrict__ sm) {
    const int64_t r = int64_t(blockIdx.x) * kST + threadIdx.x;
    if (r < int64_t(ns) * n_pad) M[r] = m0[r % n_pad];
    if (r < ns) {
        Summary s;
        s.cnt = 0;
        s.t = 0;
        s.gi = 0;
        s.pad = 0;
        s.full_at = -1;
        s.fS = 0.0;
        sm[r] = s;
    }
}

// The returned summary (Sieve Streaming: the first in grid order with the
// largest f), the points examined (the stream stops once every summary is
// full), and its members and f values copied to the caller's outputs.
__global__ void __launch_bounds__(kST) k_stream_finish(const Summary* __restrict__ sm, int32_t ns, int32_t k,
                                                       int64_t n_order, const int32_t* __restrict__ sel,
                                                       const double* __restrict__ fv, int32_t* __restrict__ sel_out,
                                                       double* __restrict__ f_out, Result* __restrict__ res) {
    __shared__ int best_s, count_s;
    if (threadIdx.x == 0) {
        int best = 0;
        bool all_full = true;
        int64_t last = -1;
        for (int j = 0; j < ns; ++j) {
            if (sm[j].fS > sm[best].fS) best = j;
            if (sm[j].cnt < k)
                all_full = false;
            else if (sm[j].full_at > last)
                last = sm[j].full_at;
        }
        res->count = sm[best].cnt;
        res->best = best;
        res->examined = all_full ? last + 1 : n_order;
        best_s = best;
        count_s = sm[best].cnt;
    }
    __syncthreads();
    if (sel == sel_out) return;  // a single summary writes the outputs directly
    for (int t = threadIdx.x; t < count_s; t += kST) {
        sel_out[t] = sel[int64_t(best_s) * k + t];
        f_out[t] = fv[int64_t(best_s) * k + t];
    }
}

// The returned summary's minima into `out` (then loaded as the dataset state).
__global__ void __launch_bounds__(kST) k_stream_take_m(const double* __restrict__ M, int64_t n_pad,
                                                       const Result* __restrict__ res, double* __restrict__ out) {
    const int64_t r = int64_t(blockIdx.x) * kST + threadIdx.x;
    if (r < n_pad) out[r] = M[int64_t(res->best) * n_pad + r];
}

// The returned summary's members marked selected in the dataset state.
__global__ void __launch_bounds__(kST) k_stream_mark(const int32_t* __restrict__ sel, const Result* __restrict__ res,
                                                     uint8_t* __restrict__ selected) {
    for (int t = threadIdx.x; t < res->count; t += kST) selected[sel[t]] = 1;
}

// ---- host side ----

// Guesses (1+eps)^i, m <= (1+eps)^i <= k m, largest first.
std::vector<double> sieve_grid(double m, int32_t k, double eps) {
    std::vector<double> g;
    if (!(m > 0.0)) return g;
    const double base = log1p(eps);
    const int64_t lo = int64_t(ceil(log(m) / base));
    const int64_t hi = int64_t(floor(log(double(k) * m) / base));
    for (int64_t i = hi; i >= lo; --i) g.push_back(pow(1.0 + eps, double(i)));
    return g;
}

// Most guesses (1+eps)^i in [m, k m] for any m > 0: floor(log k / log(1+eps)) + 1,
// plus one for rounding in the logarithms that place the grid ends.
int64_t max_guesses(int32_t k, double eps) { return int64_t(floor(log(double(k)) / log1p(eps))) + 2; }

bool valid_n(int64_t n) { return n >= 1 && n < (int64_t(1) << 31) - kRowAlign; }

size_t al256(size_t v) { return (v + 255) & ~size_t(255); }

// Stream points per stretch: `batch`, or by default as many as keep the
// stretch's distance rows within kStretchBytes (32 .. 1024); never more than
// the stream.
int32_t stretch_len(int64_t n_pad, int64_t n_order, int32_t batch) {
    int64_t b = batch;
    if (b == 0) b = std::min<int64_t>(1024, std::max<int64_t>(32, int64_t(kStretchBytes / (8 * size_t(n_pad)))));
    return int32_t(std::max<int64_t>(1, std::min<int64_t>(b, n_order)));
}

// Scratch of one call with `ns` summaries (1 for Three Sieves) and J guesses.
struct StreamLayout {
    size_t d, m, sel, fv, sm, grid, res, total;
};

StreamLayout stream_layout(int64_t n_pad, int32_t k, int64_t ns, int64_t J, int32_t stretch) {
    StreamLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += al256(bytes);
        return at;
    };
    // the distance rows; also the returned minima at the end (n_pad <= stretch rows)
    L.d = take(size_t(std::max<int64_t>(stretch, 1)) * size_t(n_pad) * sizeof(double));
    L.m = take(size_t(ns) * size_t(n_pad) * sizeof(double));
    L.sel = take(ns > 1 ? size_t(ns) * size_t(k) * sizeof(int32_t) : 0);
    L.fv = take(ns > 1 ? size_t(ns) * size_t(k) * sizeof(double) : 0);
    L.sm = take(size_t(ns) * sizeof(Summary));
    L.grid = take(size_t(J) * sizeof(double));
    L.res = take(sizeof(Result));
    L.total = o;
    return L;
}

hipError_t read_state(const ebc_dataset* ds, DevState* st, hipStream_t s) {
    hipError_t e = hipMemcpyAsync(st, ds->b.state, sizeof(DevState), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e;
}

// The caller's stream indices, checked on the host before any work.
ebc_status check_order(const ebc_dataset* ds, const int32_t* order, int64_t n_order, hipStream_t s) {
    if (!order || n_order == 0) return EBC_OK;
    std::vector<int32_t> h(static_cast<size_t>(n_order));
    if (hipMemcpyAsync(h.data(), order, size_t(n_order) * sizeof(int32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return EBC_E_DEVICE;
    for (int32_t v : h)
        if (v < 0 || int64_t(v) >= ds->n) return EBC_E_INDEX;
    return EBC_OK;
}

// S = {} in the dataset state; m = max_e f({e}) unless given (> 0): one
// greedy step (the float64 re-scored best singleton), then S = {} again.
ebc_status start_stream(ebc_dataset* ds, double* m_max, int32_t* sel_tmp, double* f_tmp, hipStream_t s,
                        DevState* st) {
    if (launch_reset_state(ds, s) != hipSuccess) return EBC_E_DEVICE;
    if (!(*m_max > 0.0)) {
        if (launch_greedy_step(ds, 0, 1, sel_tmp, f_tmp, nullptr, s, nullptr) != hipSuccess ||
            read_state(ds, st, s) != hipSuccess)
            return EBC_E_DEVICE;
        *m_max = st->gstar / double(ds->n);
        return launch_reset_state(ds, s) == hipSuccess ? EBC_OK : EBC_E_DEVICE;
    }
    return read_state(ds, st, s) == hipSuccess ? EBC_OK : EBC_E_DEVICE;
}

template <int R, int P>
void launch_walk(int32_t ns, const WalkArgs& w, hipStream_t s) {
    hipLaunchKernelGGL((k_stream_walk<R, P>), dim3(unsigned(ns)), dim3(kST), 0, s, w);
}

// Both optimisers: T > 0 runs Three Sieves (one summary, the guess walking
// down after T rejections), T = 0 Sieve Streaming (one summary per guess).
ebc_status run_stream(ebc_dataset* ds, int32_t k, double eps, int64_t T, double m_max, const int32_t* order,
                      int64_t n_order, int32_t batch, int32_t* sel_out, double* f_out, int32_t* count_out,
                      double* v_out, int64_t* examined_out, void* scratch, size_t scratch_bytes, hipStream_t s) {
    if (!scratch || reinterpret_cast<uintptr_t>(scratch) % 256 != 0) return EBC_E_INVALID_ARG;
    const int32_t stretch = stretch_len(ds->n_pad, n_order, batch);
    const int64_t ns_max = T > 0 ? 1 : max_guesses(k, eps);
    if (scratch_bytes < stream_layout(ds->n_pad, k, ns_max, max_guesses(k, eps), stretch).total)
        return EBC_E_INVALID_ARG;
    ebc_status st_ = check_order(ds, order, n_order, s);
    if (st_ != EBC_OK) return st_;
    DevState st;
    if ((st_ = start_stream(ds, &m_max, sel_out, f_out, s, &st)) != EBC_OK) return st_;
    if (st.error != 0) return EBC_OK;  // reported by ebc_sync_status
    const std::vector<double> grid = sieve_grid(m_max, k, eps);
    const int64_t J = int64_t(grid.size());
    if (J == 0) return EBC_OK;
    if (J > max_guesses(k, eps)) return EBC_E_INVALID_ARG;  // not reached: the grid spans a factor k
    const int32_t ns = T > 0 ? 1 : int32_t(J);

    const StreamLayout L = stream_layout(ds->n_pad, k, ns, J, stretch);
    char* base = static_cast<char*>(scratch);
    double* D = reinterpret_cast<double*>(base + L.d);
    double* M = reinterpret_cast<double*>(base + L.m);
    int32_t* sel = ns > 1 ? reinterpret_cast<int32_t*>(base + L.sel) : sel_out;
    double* fv = ns > 1 ? reinterpret_cast<double*>(base + L.fv) : f_out;
    Summary* sm = reinterpret_cast<Summary*>(base + L.sm);
    double* d_grid = reinterpret_cast<double*>(base + L.grid);
    Result* d_res = reinterpret_cast<Result*>(base + L.res);

    if (hipMemcpyAsync(d_grid, grid.data(), size_t(J) * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
        return EBC_E_DEVICE;
    const int64_t init_n = std::max<int64_t>(int64_t(ns) * ds->n_pad, ns);
    hipLaunchKernelGGL(k_stream_init, dim3(unsigned((init_n + kST - 1) / kST)), dim3(kST), 0, s, ds->b.m0, ds->n_pad,
                       ns, M, sm);

    WalkArgs w;
    w.D = D;
    w.n = ds->n;
    w.n_pad = ds->n_pad;
    w.k = k;
    w.order = order;
    w.grid = d_grid;
    w.J = int32_t(J);
    w.pad = 0;
    w.T = T;
    w.dst = ds->b.state;
    w.sm = sm;
    w.M = M;
    w.sel = sel;
    w.fv = fv;
    const int64_t rpt = ds->n_pad / kST;  // ground points per thread of the walk
    for (int64_t pos = 0; pos < n_order; pos += stretch) {
        const int32_t cnt = int32_t(std::min<int64_t>(stretch, n_order - pos));
        const dim3 g(unsigned(ds->n_pad / kDI), unsigned((cnt + kDI - 1) / kDI));
        if (ds->metric == 1)
            hipLaunchKernelGGL(k_stream_dist<1>, g, dim3(64 * kDW), 0, s, ds->x, ds->n, ds->d, order, pos, cnt, ds->n_pad,
                               D, sm, ns, k);
        else
            hipLaunchKernelGGL(k_stream_dist<0>, g, dim3(64 * kDW), 0, s, ds->x, ds->n, ds->d, order, pos, cnt, ds->n_pad,
                               D, sm, ns, k);
        w.cnt = cnt;
        w.pos = pos;
        if (rpt <= 1)
            launch_walk<1, 8>(ns, w, s);
        else if (rpt <= 2)
            launch_walk<2, 8>(ns, w, s);
        else if (rpt <= 4)
            launch_walk<4, 8>(ns, w, s);
        else if (rpt <= 8)
            launch_walk<8, 4>(ns, w, s);
        else if (rpt <= kRegMax)
            launch_walk<kRegMax, 2>(ns, w, s);
        else
            hipLaunchKernelGGL(k_stream_walk_big, dim3(unsigned(ns)), dim3(kST), 0, s, w);
        if (hipGetLastError() != hipSuccess) return EBC_E_DEVICE;
    }
    hipLaunchKernelGGL(k_stream_finish, dim3(1), dim3(kST), 0, s, sm, ns, k, n_order, sel, fv, sel_out, f_out, d_res);
    // the dataset state afterwards: the returned summary's minima and members
    hipLaunchKernelGGL(k_stream_take_m, dim3(unsigned(ds->n_pad / kST)), dim3(kST), 0, s, M, ds->n_pad, d_res, D);
    if (launch_load_m(ds, D, s) != hipSuccess) return EBC_E_DEVICE;
    hipLaunchKernelGGL(k_stream_mark, dim3(1), dim3(kST), 0, s, sel_out, d_res, ds->b.selected);
    Result res;
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&res, d_res, sizeof(Result), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return EBC_E_DEVICE;
    *count_out = res.count;
    if (v_out) *v_out = T > 0 ? 0.0 : grid[size_t(res.best)];
    if (examined_out) *examined_out = res.examined;
    ds->stats.steps = res.count;
    ds->stats.list_steps = 0;
    return EBC_OK;
}

}  // namespace

extern "C" {

size_t ebc_three_sieves_bytes(int64_t n, int32_t k, double eps, int64_t n_order, int32_t batch) {
    if (!valid_n(n) || k < 1 || int64_t(k) > n || !(eps > 0.0) || n_order < 0 || batch < 0) return 0;
    const int64_t np = pad_rows(n);
    return stream_layout(np, k, 1, max_guesses(k, eps), stretch_len(np, n_order, batch)).total;
}

ebc_status ebc_three_sieves(ebc_dataset* ds, int32_t k, double eps, int64_t T, double m_max, const int32_t* order,
                            int64_t n_order, int32_t batch, int32_t* sel_out, double* f_out, int32_t* count_out,
                            int64_t* examined_out, void* scratch, size_t scratch_bytes, void* stream) {
    if (!ds || !count_out || k < 1 || int64_t(k) > ds->n || !(eps > 0.0) || T < 1 || batch < 0) return EBC_E_INVALID_ARG;
    if (!sel_out || !f_out || n_order < 0 || (!order && n_order > ds->n)) return EBC_E_INVALID_ARG;
    *count_out = 0;
    if (examined_out) *examined_out = 0;
    return run_stream(ds, k, eps, T, m_max, order, n_order, batch, sel_out, f_out, count_out, nullptr, examined_out,
                      scratch, scratch_bytes, reinterpret_cast<hipStream_t>(stream));
}

size_t ebc_sieve_streaming_bytes(int64_t n, int32_t k, double eps, int64_t n_order, int32_t batch) {
    if (!valid_n(n) || k < 1 || int64_t(k) > n || !(eps > 0.0) || n_order < 0 || batch < 0) return 0;
    const int64_t np = pad_rows(n);
    const int64_t J = max_guesses(k, eps);
    return stream_layout(np, k, J, J, stretch_len(np, n_order, batch)).total;
}

ebc_status ebc_sieve_streaming(ebc_dataset* ds, int32_t k, double eps, double m_max, const int32_t* order,
                               int64_t n_order, int32_t batch, int32_t* sel_out, double* f_out, int32_t* count_out,
                               double* v_out, int64_t* examined_out, void* scratch, size_t scratch_bytes,
                               void* stream) {
    if (!ds || !count_out || k < 1 || int64_t(k) > ds->n || !(eps > 0.0) || batch < 0) return EBC_E_INVALID_ARG;
    if (!sel_out || !f_out || n_order < 0 || (!order && n_order > ds->n)) return EBC_E_INVALID_ARG;
    *count_out = 0;
    if (v_out) *v_out = 0.0;
    if (examined_out) *examined_out = 0;
    return run_stream(ds, k, eps, 0, m_max, order, n_order, batch, sel_out, f_out, count_out, v_out, examined_out,
                      scratch, scratch_bytes, reinterpret_cast<hipStream_t>(stream));
}

}  // extern "C"
