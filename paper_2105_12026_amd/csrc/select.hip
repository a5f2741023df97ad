// One greedy step after the gains kernel (Sec. 3 and Sec. 4.1: greedy picks
// the not-yet-selected point of largest marginal gain). Each stage is a
// device function of (instance descriptor, step, block); the solo kernels
// run it on one instance, the batched kernels map their blocks onto many.
//   k_gsum     sum the per-chunk gain sums, mask selected points, block maxima
//   k_wcount   every candidate within tau*|best| of the best enters the window
//   k_wselect  choose at most kWindowMax window candidates, deterministically
//   k_rescore  float64 direct-difference gains of the window candidates
//   k_pick     best float64 gain, ties to the lowest index; record the pick
//   k_update   m_v <- min(m_v, d(v, c*)) in float64, per-block sums of m_v
//   k_fsum     f(S_t) = L({e0}) - |V|^-1 sum_v m_v  (Alg. 1: sum, then / |V|)
// Steps that score a list instead of every candidate (lazy.h) replace the
// first three stages by
//   k_list_sum    per-chunk sums of the heads or the list -> gsum
//   k_list_build  candidates whose old gain reaches the window of the best head
//   k_list_window the window out of the list, or which of it to score again
// where k_rescore makes the window out of the candidates scored again;
// and k_update / k_fsum also choose the heads of the next step's list.
// No step reads anything back to the host; all sums run in a fixed order.
#include <math.h>

#include "ebc_internal.h"
#include "lazy.h"
#include "quant.h"

namespace ebc {

__device__ inline bool better(double ga, int ia, double gb, int ib) {
    return ga > gb || (ga == gb && ia < ib);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}
// Best (gain, index) of the wave, with an extra value that goes along.
__device__ __forceinline__ void wave_best(double& g, int& i, int& extra) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double og = __shfl_xor(g, off, 64);
        const int oi = __shfl_xor(i, off, 64), oe = __shfl_xor(extra, off, 64);
        if (better(og, oi, g, i)) {
            g = og;
            i = oi;
            extra = oe;
        }
    }
}

// Sum of 256 values of a block of 256 threads through red: pairs 128 apart,
// then 64, 32, ... 1 (one fixed tree). The first wave returns it in lane 0.
__device__ __forceinline__ double tree_sum256(const double* __restrict__ red, int lane) {
    double s = (red[lane] + red[lane + 128]) + (red[lane + 64] + red[lane + 192]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    return s;
}

// Threshold of the re-score window from the global best float32 gain.
__device__ double window_threshold(double gmax, const DevState* st) {
    return gmax - (st->tau * fabs(gmax) + st->tau_abs * st->nmax);
}

// Block-wide maximum of bmax[0..nb) (every block computes the same value).
__device__ double block_gmax(const double* bmax, int nb, double* red) {
    double m = -INFINITY;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) m = fmax(m, bmax[i]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// ---- gsum: per-chunk sums -> gsum, selected masked, block maxima ----
__device__ void gsum_body(const InstDesc& c, int64_t blk, int32_t splits) {
    __shared__ double sg[kBlock / 64];
    __shared__ int si[kBlock / 64];
    const Buffers& b = c.b;
    const int64_t i = blk * kBlock + threadIdx.x;
    double g = 0.0;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) g += b.part[int64_t(s) * c.n_pad + i];
    if (b.selected[i]) g = -INFINITY;
    b.gsum[i] = g;
    int row = int(i), none = 0;
    wave_best(g, row, none);
    if ((threadIdx.x & 63) == 0) {
        sg[threadIdx.x >> 6] = g;
        si[threadIdx.x >> 6] = row;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w)
            if (better(sg[w], si[w], g, row)) {
                g = sg[w];
                row = si[w];
            }
        b.bmax[blk] = g;
        b.barg[blk] = row;
    }
}

// ---- wcount: candidates within the window, compacted per block in index order ----
__device__ void wcount_body(const InstDesc& c, int64_t blk) {
    __shared__ double red[kBlock];
    __shared__ int scan[kBlock];
    const Buffers& b = c.b;
    const double gmax = block_gmax(b.bmax, c.nb, red);
    const double thr = window_threshold(gmax, b.state);
    const int64_t i = blk * kBlock + threadIdx.x;
    const double g = b.gsum[i];
    const int q = (g >= thr && g > -INFINITY) ? 1 : 0;
    // inclusive scan of q across the block (Hillis-Steele), index order kept
    scan[threadIdx.x] = q;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        const int add = threadIdx.x >= off ? scan[threadIdx.x - off] : 0;
        __syncthreads();
        scan[threadIdx.x] += add;
        __syncthreads();
    }
    if (q) {
        WindowEntry e;
        e.g = g;
        e.idx = int(i);
        e.pad = 0;
        b.wstage[blk * kBlock + scan[threadIdx.x] - 1] = e;
    }
    if (threadIdx.x == kBlock - 1) b.bcnt[blk] = scan[kBlock - 1];
}

// ---- wselect (one block of 1024 threads per instance) ----
// Gather the window entries in index order, then keep at most kWindowMax:
//   total <= kWindowMax          all of them;
//   total <= kWindowCap          the kWindowMax best by (gain desc, index asc);
//   otherwise (counted overflow) the best one plus the lowest-index others.
constexpr int kSelThreads = 1024;
__device__ void wselect_body(const InstDesc& c) {
    __shared__ WindowEntry list[kWindowCap];
    __shared__ int scan[kSelThreads];
    __shared__ double red[kSelThreads];
    const Buffers& b = c.b;
    const int nb = c.nb;
    const int tid = threadIdx.x;
    int total = 0;
    for (int base = 0; base < nb; base += kSelThreads) {
        const int blk = base + tid;
        const int cnt = blk < nb ? b.bcnt[blk] : 0;
        scan[tid] = cnt;
        __syncthreads();
        for (int off = 1; off < kSelThreads; off <<= 1) {
            const int add = tid >= off ? scan[tid - off] : 0;
            __syncthreads();
            scan[tid] += add;
            __syncthreads();
        }
        const int excl = total + scan[tid] - cnt;
        for (int i = 0; i < cnt; ++i) {
            const int pos = excl + i;
            if (pos < kWindowCap) list[pos] = b.wstage[int64_t(blk) * kBlock + i];
        }
        total += scan[kSelThreads - 1];
        __syncthreads();
    }
    const int nl = total < kWindowCap ? total : kWindowCap;
    if (total <= kWindowMax) {
        if (tid < total) b.wfinal[tid] = list[tid];
    } else if (total <= kWindowCap) {
        for (int i = tid; i < nl; i += kSelThreads) {
            int rank = 0;
            for (int j = 0; j < nl; ++j)
                rank += better(list[j].g, list[j].idx, list[i].g, list[i].idx) ? 1 : 0;
            if (rank < kWindowMax) b.wfinal[rank] = list[i];
        }
    } else {
        // overflow: the global best float32 candidate first ...
        const double gmax = block_gmax(b.bmax, nb, red);
        if (tid == 0) {
            int first = -1;
            for (int i = 0; i < nb && first < 0; ++i)
                if (b.bmax[i] == gmax) first = b.barg[i];
            WindowEntry e;
            e.g = gmax;
            e.idx = first;
            e.pad = 0;
            b.wfinal[0] = e;
            int w = 1;
            for (int i = 0; i < nl && w < kWindowMax; ++i)
                if (list[i].idx != first) b.wfinal[w++] = list[i];
        }
    }
    if (tid == 0) {
        const int W = total < kWindowMax ? total : kWindowMax;
        b.state->window_count = W;
        if (total > b.state->window_max) b.state->window_max = total;
        if (total > kWindowCap) b.state->window_overflow += 1;
    }
}

// ---- rescore: float64 direct-difference gains of the window candidates ----
// One thread per ground point, from the caller's float32 points; candidates
// in groups of 8 staged in LDS as float64, up to 128 dimensions at a time
// (longer rows take several passes, summed in dimension order); each thread
// reads its own row in 16-byte pieces when rows are 16-byte aligned, four
// pieces in flight (the other lanes' pieces of the same cache lines follow
// in the next iterations); per-block sums in a fixed order.
constexpr int kRescoreGroup = 8;
constexpr int kRescoreChunk = 128;

// One dimension's term for the NJ staged candidates (stride kRescoreChunk):
// squared difference (METRIC 0) or absolute difference (METRIC 1).
template <int METRIC, int NJ>
__device__ __forceinline__ void dim_terms(double xk, const double* __restrict__ cxk, double (&acc)[NJ]) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const double t = xk - cxk[j * kRescoreChunk];
        if (METRIC == 1)
            acc[j] += fabs(t);
        else
            acc[j] = fma(t, t, acc[j]);
    }
}

// acc[j] += sum over k < kn, in k order, of the terms between row piece xv
// (float32, global) and the staged candidates cx[j][0..kn).
template <int METRIC, int NJ>
__device__ __forceinline__ void row_terms(const float* __restrict__ xv, bool vec, int kn,
                                          const double* __restrict__ cx, double (&acc)[NJ]) {
    int k = 0;
    if (vec) {
        const float4* __restrict__ x4 = reinterpret_cast<const float4*>(xv);
        for (; k + 16 <= kn; k += 16) {
            float4 q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = x4[k / 4 + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                dim_terms<METRIC, NJ>(double(q[u].x), cx + k + 4 * u, acc);
                dim_terms<METRIC, NJ>(double(q[u].y), cx + k + 4 * u + 1, acc);
                dim_terms<METRIC, NJ>(double(q[u].z), cx + k + 4 * u + 2, acc);
                dim_terms<METRIC, NJ>(double(q[u].w), cx + k + 4 * u + 3, acc);
            }
        }
        for (; k + 4 <= kn; k += 4) {
            const float4 q = x4[k / 4];
            dim_terms<METRIC, NJ>(double(q.x), cx + k, acc);
            dim_terms<METRIC, NJ>(double(q.y), cx + k + 1, acc);
            dim_terms<METRIC, NJ>(double(q.z), cx + k + 2, acc);
            dim_terms<METRIC, NJ>(double(q.w), cx + k + 3, acc);
        }
    }
    for (; k < kn; ++k) dim_terms<METRIC, NJ>(double(xv[k]), cx + k, acc);
}

// Windows of at most stored_window(c) candidates keep their distances for the
// update of the same step, in the partial sums (not needed between the window
// and the next gains, but while row blocks may still read a recount's there):
// 8 bytes a point read there instead of a whole row.
__device__ __forceinline__ bool distances_stored(const InstDesc& c) {
    const int most = c.v_splits < kRescoreGroup ? c.v_splits : kRescoreGroup;
    return c.b.state->window_count <= most && !(c.lazy && c.b.state->list_exact > 0);
}
__device__ __forceinline__ bool window_has_distances(const InstDesc& c, int rank) {
    return rank >= 0 && distances_stored(c);
}

// METRIC 0: squared Euclidean (the paper's d); 1: L1, sum of |x_vk - x_ck|.
// One group of at most NJ window candidates from position g0.
template <int METRIC, int NJ>
__device__ __forceinline__ void rescore_group(const InstDesc& c, int64_t blk, int g0, int W, double* __restrict__ cx,
                                              double (*red)[kBlock]) {
    const Buffers& b = c.b;
    const float* __restrict__ x = c.x;
    const int d = c.d;
    const int64_t v = blk * kBlock + threadIdx.x;
    const bool live = v < c.n;
    const double mv = live ? b.m64[v] : 0.0;
    const float* __restrict__ xv = x + (live ? v : 0) * d;
    const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    const int gn = (W - g0) < NJ ? (W - g0) : NJ;
    double acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = 0.0;
    for (int k0 = 0; k0 < d; k0 += kRescoreChunk) {
        const int kn = (d - k0) < kRescoreChunk ? (d - k0) : kRescoreChunk;
        __syncthreads();
        for (int e = threadIdx.x; e < NJ * kn; e += kBlock) {
            const int j = e / kn, k = e % kn;
            // rows past the group's end repeat its first candidate (their sums are not used)
            cx[j * kRescoreChunk + k] = double(x[int64_t(b.wfinal[g0 + (j < gn ? j : 0)].idx) * d + k0 + k]);
        }
        __syncthreads();
        if (live) row_terms<METRIC, NJ>(xv + k0, vec, kn, cx, acc);
    }
    if (distances_stored(c) && live) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (j < gn) b.part[int64_t(g0 + j) * c.n_pad + v] = acc[j];
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < NJ; ++j) red[j][threadIdx.x] = live ? fmax(0.0, mv - acc[j]) : 0.0;
    __syncthreads();
    for (int j = wave; j < gn; j += kBlock / 64) {
        const double sum = tree_sum256(red[j], lane);
        if (lane == 0) b.rpart[blk * kWindowMax + g0 + j] = sum;
    }
}

// Groups of 8; a window of 1 or 2 takes the kernel of its size (the LDS reads
// of the staged candidates, one per candidate and dimension, are what bounds
// it: 100000 x 100, W = 1: 17.4 -> 9 us).
template <int METRIC>
__device__ void rescore_impl(const InstDesc& c, int64_t blk, double* __restrict__ cx, double (*red)[kBlock]) {
    const int W = c.b.state->window_count;
    if (W == 1)
        rescore_group<METRIC, 1>(c, blk, 0, W, cx, red);
    else if (W == 2)
        rescore_group<METRIC, 2>(c, blk, 0, W, cx, red);
    else if (W <= 4)
        rescore_group<METRIC, 4>(c, blk, 0, W, cx, red);
    else
        for (int g0 = 0; g0 < W; g0 += kRescoreGroup) rescore_group<METRIC, kRescoreGroup>(c, blk, g0, W, cx, red);
}

__device__ void list_exact_body(const InstDesc& c, bool count);

__device__ void rescore_body(const InstDesc& c, int64_t blk) {
    if (c.lazy && c.b.state->list_exact > 0) list_exact_body(c, blk == 0);  // lazy.h
    __shared__ double cx[kRescoreGroup * kRescoreChunk];
    __shared__ double red[kRescoreGroup][kBlock];
    if (c.metric == 1)
        rescore_impl<1>(c, blk, cx, red);
    else
        rescore_impl<0>(c, blk, cx, red);
}

__device__ __forceinline__ int rescore_rows(const InstDesc& c, int W);

// ---- pick (one block per instance) ----
// float64 gain of each window candidate = sum of the per-block sums: up to
// kPickColumnRows of them, thread j adds candidate j's in block order;
// otherwise wave w takes candidates w, w + NT/64, ...: 256 running sums (i
// takes blocks i, i+256, ...), then a fixed tree. Best gain wins, ties to the
// lowest index. A step with no valid candidate (only possible with non-finite
// input) picks -1. Every thread of the block gets the pick, its gain and its
// position in the window (-1: chosen outside of it).
constexpr int kPickColumnRows = 64;
constexpr int kPickThreads = 1024;
// Solo runs of at most this many row blocks make the pick in every block of the
// update, for itself, instead of in a launch before it (a launch is 4 to 5 us;
// with more blocks the sums of a large window are read too often).
constexpr int kPickBlocks = 128;

template <int NT>
__device__ int pick_choose(const InstDesc& c, double* gain, int* rank) {
    __shared__ double sg[kWindowMax];
    __shared__ int out_cs, out_rank;
    __shared__ double out_gain;
    const Buffers& b = c.b;
    const int tid = threadIdx.x;
    const int W = b.state->window_count;
    const int nbv = rescore_rows(c, W);
    if (nbv <= kPickColumnRows) {
        for (int j = tid; j < W; j += NT) {
            double s = 0.0;
#pragma unroll 8  // loads in flight together: 40 row blocks 11 -> 5 us
            for (int blk = 0; blk < nbv; ++blk) s += b.rpart[int64_t(blk) * kWindowMax + j];
            sg[j] = s;
        }
    } else {
        const int lane = tid & 63;
        for (int j = tid >> 6; j < W; j += NT / 64) {
            double q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                q[i] = 0.0;
                for (int blk = lane + 64 * i; blk < nbv; blk += 256) q[i] += b.rpart[int64_t(blk) * kWindowMax + j];
            }
            double s = (q[0] + q[2]) + (q[1] + q[3]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
            if (lane == 0) sg[j] = s;
        }
    }
    __syncthreads();
    if (tid < 64) {
        double g = -INFINITY;
        int idx = 0x7fffffff, at = -1;
        for (int j = tid; j < W; j += 64) {
            const int i = b.wfinal[j].idx;
            if (better(sg[j], i, g, idx)) {
                g = sg[j];
                idx = i;
                at = j;
            }
        }
        wave_best(g, idx, at);
        if (W > 0 && g == 0.0) {
            // The best float64 gain of the window is 0: every point is covered, so
            // every unselected point has gain 0 and the pick is the lowest
            // unselected index (also when more zero-gain candidates than the
            // window holds were ranked by their reduced-precision gains).
            int lo = 0x7fffffff;
            for (int64_t i = tid; i < c.n; i += 64)
                if (!b.selected[i]) {
                    lo = int(i);
                    break;
                }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const int o = __shfl_xor(lo, off, 64);
                lo = o < lo ? o : lo;
            }
            if (lo != 0x7fffffff && lo != idx) {
                idx = lo;
                at = -1;
            }
        }
        if (tid == 0) {
            out_cs = W > 0 && idx >= 0 && int64_t(idx) < c.n ? idx : -1;
            out_rank = at;
            out_gain = g;
        }
    }
    __syncthreads();
    *gain = out_gain;
    *rank = out_rank;
    return out_cs;
}

// Record the pick (one thread). mark: set `selected` here; where other blocks
// may still look for an unselected point, a later kernel does it.
__device__ void pick_record(const InstDesc& c, int32_t t, int cs, double gain, int rank, bool mark) {
    const Buffers& b = c.b;
    b.state->cstar = cs;
    b.state->crank = rank;
    c.sel[t] = cs;
    if (cs >= 0) {
        b.state->gstar = gain;
        if (mark) b.selected[cs] = 1;
        if (c.gain) c.gain[t] = gain / double(c.n);
    } else {
        atomicCAS(&b.state->error, 0, kDevErrNonFinite);
        if (c.gain) c.gain[t] = NAN;
    }
}

__device__ void pick_body(const InstDesc& c, int32_t t) {
    double gain;
    int rank;
    const int cs = pick_choose<kPickThreads>(c, &gain, &rank);
    if (threadIdx.x == 0) pick_record(c, t, cs, gain, rank, true);
}

// Estimate of candidate v's present gain, and the block's best one: the gain
// it had when it was last scored, times what is left of its own minimum since
// (old: m_v before this step, which is what a full step scores every candidate
// with). The best of each block goes to bmax / barg.
__device__ void block_best_estimate(const InstDesc& c, int64_t blk, int32_t t, int cs, double old, double mv,
                                    double* red, int* ri) {
    const Buffers& b = c.b;
    const int64_t v = blk * kBlock + threadIdx.x;
    float* __restrict__ lm = list_m(c);
    float m_scored = float(old);
    if (!list_step(c, t))
        lm[v] = m_scored;
    else
        m_scored = lm[v];
    double est = -INFINITY;
    if (!b.selected[v] && v != cs) est = b.gsum[v] * (m_scored > 0.0f ? mv / double(m_scored) : 1.0);
    int row = int(v), none = 0;
    wave_best(est, row, none);
    __syncthreads();  // red has been read
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = est;
        ri[threadIdx.x >> 6] = row;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w)
            if (better(red[w], ri[w], est, row)) {
                est = red[w];
                row = ri[w];
            }
        b.bmax[blk] = est;
        b.barg[blk] = row;
    }
}

// ---- update: m_v <- min(m_v, d(v, c*)) in float64, per-block sums of m_v ----
__device__ void update_body(const InstDesc& c, int64_t blk, int32_t t, int cs, int rank) {
    static_assert(kNarrowMaxK <= kRescoreChunk, "short rows fit one staged piece");
    __shared__ double cx[kRescoreChunk];
    __shared__ double red[kBlock];
    __shared__ int ri[kBlock];
    const Buffers& b = c.b;
    const float* __restrict__ x = c.x;
    const int d = c.d;
    const bool stored = window_has_distances(c, rank);
    if (cs >= 0 && !stored)
        for (int k = threadIdx.x; k < d; k += kBlock) cx[k] = double(x[int64_t(cs) * d + k]);
    __syncthreads();
    const int64_t v = blk * kBlock + threadIdx.x;
    double mv = 0.0, old = 0.0;
    if (v < c.n && cs < 0) {
        mv = old = b.m64[v];
    } else if (v < c.n) {
        const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
        double acc[1] = {0.0};
        if (stored)
            acc[0] = b.part[int64_t(rank) * c.n_pad + v];
        else
            row_terms<0, 1>(x + v * d, vec, d, cx, acc);
        mv = old = b.m64[v];
        if (acc[0] < mv) {
            mv = acc[0];
            b.m64[v] = mv;
            set_point_terms(b, v, mv);
        }
    }
    red[threadIdx.x] = mv;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double sum = tree_sum256(red, threadIdx.x);
        if (threadIdx.x == 0) b.fpart[blk] = sum;
    }
    if (c.lazy) block_best_estimate(c, blk, t, cs, old, mv, red, ri);
}

// ---- L1 update (any row length): m_v <- min(m_v, sum_k |x_vk - x_c*k|) in
// float64, the new member's values staged in LDS 128 at a time; per-block
// sums of m_v as in update_body ----
__device__ void update_l1_body(const InstDesc& c, int64_t blk, int32_t t, int cs, int rank) {
    __shared__ float cx[kRescoreChunk];
    __shared__ double red[kBlock];
    __shared__ int ri[kBlock];
    const Buffers& b = c.b;
    const float* __restrict__ x = c.x;
    const int d = c.d;
    const int64_t v = blk * kBlock + threadIdx.x;
    const bool live = v < c.n;
    const float* xv = x + (live ? v : 0) * d;
    double acc = 0.0;
    const bool stored = window_has_distances(c, rank);
    if (stored && live) acc = b.part[int64_t(rank) * c.n_pad + v];
    for (int k0 = 0; k0 < d && cs >= 0 && !stored; k0 += kRescoreChunk) {
        const int kn = (d - k0) < kRescoreChunk ? (d - k0) : kRescoreChunk;
        __syncthreads();
        for (int k = threadIdx.x; k < kn; k += kBlock) cx[k] = x[int64_t(cs) * d + k0 + k];
        __syncthreads();
        if (live)
            for (int k = 0; k < kn; ++k) acc += fabs(double(xv[k0 + k]) - double(cx[k]));
    }
    double mv = 0.0, old = 0.0;
    if (live) {
        mv = old = b.m64[v];
        if (cs >= 0 && acc < mv) {
            mv = acc;
            b.m64[v] = mv;
            set_point_terms(b, v, mv);
        }
    }
    red[threadIdx.x] = mv;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double sum = tree_sum256(red, threadIdx.x);
        if (threadIdx.x == 0) b.fpart[blk] = sum;
    }
    if (c.lazy) block_best_estimate(c, blk, t, cs, old, mv, red, ri);
}

// ---- long rows (padded length above 128): re-score and update ----
// One thread per ground point, as for short rows, reading its own row in
// 16-byte pieces when the rows are 16-byte aligned (the other lanes' pieces of the
// same cache lines follow in the next iterations); the candidates' values
// are staged in LDS 512 dimensions at a time. Every per-thread float64 sum
// runs in dimension order, as for short rows.
constexpr int kLongChunk = 512;

template <int NJ>
__device__ __forceinline__ void long_sums(const InstDesc& c, int64_t v, bool live, const int64_t (&cand)[kRescoreGroup],
                                          int nc, float (&cx)[kRescoreGroup][kLongChunk], double (&acc)[NJ]) {
    const float* __restrict__ x = c.x;
    const int d = c.d;
    const float* __restrict__ xv = x + (live ? v : 0) * d;
    const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
#pragma unroll
    for (int q = 0; q < NJ; ++q) acc[q] = 0.0;
    for (int k0 = 0; k0 < d; k0 += kLongChunk) {
        const int kn = (d - k0) < kLongChunk ? (d - k0) : kLongChunk;
        __syncthreads();  // the previous piece of cx is no longer read
        for (int e = threadIdx.x; e < nc * kLongChunk; e += kBlock) {
            const int q = e / kLongChunk, k = e % kLongChunk;
            cx[q][k] = k < kn ? x[cand[q] * d + k0 + k] : 0.0f;
        }
        __syncthreads();
        if (!live) continue;
        if (vec) {
            const float4* __restrict__ x4 = reinterpret_cast<const float4*>(xv + k0);
#pragma unroll 4
            for (int k4 = 0; k4 < kn / 4; ++k4) {
                const float4 a = x4[k4];
                const float av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double xk = double(av[i]);
#pragma unroll
                    for (int q = 0; q < NJ; ++q) {
                        const double t = xk - double(cx[q][4 * k4 + i]);
                        acc[q] = fma(t, t, acc[q]);
                    }
                }
            }
        } else {
            for (int k = 0; k < kn; ++k) {
                const double xk = double(xv[k0 + k]);
#pragma unroll
                for (int q = 0; q < NJ; ++q) {
                    const double t = xk - double(cx[q][k]);
                    acc[q] = fma(t, t, acc[q]);
                }
            }
        }
    }
}

__host__ __device__ inline int split_window(const InstDesc& c);
__device__ __forceinline__ int long_quarter(int d);
__device__ void rescore_split_sum(const InstDesc& c, int64_t blk, double (*red)[kBlock]);

// One-pass re-score of long rows (windows above the two-pass size). A
// workgroup takes 64 ground points (sub-block s of row block blk) and group
// g of the window, blockIdx.y = 4 g + s; the window is cut into at most 32
// groups of 1, 2, 4 or 8 candidates (the smallest size that fits), so
// small windows still spread over the chip. Wave w sums
// dimension quarter w; the candidates' values are staged in LDS as
// float64, 128 dimensions of every quarter at a time. The four partial sums
// are added in quarter order and the clamped terms of the 64 points summed in
// a fixed tree into rpart row 4 blk + s.
constexpr int kLongQChunk = 128;

template <int NJ>
__device__ __forceinline__ void quarter_chunk(const float* __restrict__ xv, bool vec, int k0, int kn,
                                              const double (&cq)[kRescoreGroup][kLongQChunk],
                                              double (&acc)[kRescoreGroup]) {
    constexpr int kUnroll = NJ <= 2 ? 8 : 2;  // 16-byte loads in flight per lane
    if (vec) {
        const float4* __restrict__ x4 = reinterpret_cast<const float4*>(xv + k0);
#pragma unroll kUnroll
        for (int k4 = 0; k4 < kn / 4; ++k4) {
            const float4 a = x4[k4];
            const float av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double xk = double(av[i]);
#pragma unroll
                for (int q = 0; q < NJ; ++q) {
                    const double t = xk - cq[q][4 * k4 + i];
                    acc[q] = fma(t, t, acc[q]);
                }
            }
        }
    } else {
        for (int k = 0; k < kn; ++k) {
            const double xk = double(xv[k0 + k]);
#pragma unroll
            for (int q = 0; q < NJ; ++q) {
                const double t = xk - cq[q][k];
                acc[q] = fma(t, t, acc[q]);
            }
        }
    }
}

__device__ void rescore_long_body(const InstDesc& c, int64_t blk, int y) {
    __shared__ double cq[4][kRescoreGroup][kLongQChunk];
    __shared__ double red[4][kRescoreGroup][64];
    __shared__ int64_t scand[kRescoreGroup];
    const Buffers& b = c.b;
    const int W = b.state->window_count;
    if (W <= split_window(c)) {
        // small windows: pass 2 of the two-pass re-score, on the blocks of y = 0
        // (same for the whole block), in the LDS of cq
        if (y == 0) rescore_split_sum(c, blk, reinterpret_cast<double (*)[kBlock]>(&cq[0][0][0]));
        return;
    }
    const int gsz = W <= 32 ? 1 : (W <= 64 ? 2 : (W <= 128 ? 4 : kRescoreGroup));
    const int g0 = (y / 4) * gsz, sub = y % 4;
    if (g0 >= W) return;  // the same for the whole block
    const int gn = (W - g0) < gsz ? (W - g0) : gsz;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t v = blk * kBlock + sub * 64 + lane;
    const bool live = v < c.n;
    const float* __restrict__ x = c.x;
    const int d = c.d;
    const int Q = long_quarter(d);
    const int qb = w * Q;
    const int qe = (qb + Q) < d ? (qb + Q) : d;
    const float* __restrict__ xv = x + (live ? v : 0) * d;
    const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    if (threadIdx.x < kRescoreGroup) scand[threadIdx.x] = threadIdx.x < gn ? int64_t(b.wfinal[g0 + threadIdx.x].idx) : 0;
    double acc[kRescoreGroup];
#pragma unroll
    for (int q = 0; q < kRescoreGroup; ++q) acc[q] = 0.0;
    for (int t0 = 0; t0 < Q; t0 += kLongQChunk) {
        __syncthreads();  // scand is written; the previous piece of cq is no longer read
        for (int e = threadIdx.x; e < 4 * gn * kLongQChunk; e += kBlock) {
            const int qq = e / (gn * kLongQChunk);
            const int q = (e / kLongQChunk) % gn, k = e % kLongQChunk;
            const int kk = qq * Q + t0 + k;
            const int ke = (qq * Q + Q) < d ? (qq * Q + Q) : d;
            cq[qq][q][k] = kk < ke ? double(x[scand[q] * d + kk]) : 0.0;
        }
        __syncthreads();
        const int rest = qe - (qb + t0);
        const int kn = rest < kLongQChunk ? rest : kLongQChunk;
        if (!live || kn <= 0) continue;
        if (gn == 1)
            quarter_chunk<1>(xv, vec, qb + t0, kn, cq[w], acc);
        else if (gn == 2)
            quarter_chunk<2>(xv, vec, qb + t0, kn, cq[w], acc);
        else if (gn <= 4)
            quarter_chunk<4>(xv, vec, qb + t0, kn, cq[w], acc);
        else
            quarter_chunk<kRescoreGroup>(xv, vec, qb + t0, kn, cq[w], acc);
    }
#pragma unroll
    for (int q = 0; q < kRescoreGroup; ++q) red[w][q][lane] = acc[q];
    __syncthreads();
    const double mv = live ? b.m64[v] : 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int q = w + 4 * h;
        double val = 0.0;
        if (live && q < gn) {
            const double dist = ((red[0][q][lane] + red[1][q][lane]) + red[2][q][lane]) + red[3][q][lane];
            val = fmax(0.0, mv - dist);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) val += __shfl_xor(val, off, 64);
        if (lane == 0 && q < gn) b.rpart[(4 * blk + sub) * kWindowMax + g0 + q] = val;
    }
}

__device__ void update_long_body(const InstDesc& c, int64_t blk) {
    __shared__ float cx[kRescoreGroup][kLongChunk];
    __shared__ double red[kBlock];
    const Buffers& b = c.b;
    const int cs = b.state->cstar;
    const int64_t v = blk * kBlock + threadIdx.x;
    double dist[1] = {0.0};
    if (cs >= 0) {
        int64_t cand[kRescoreGroup];
#pragma unroll
        for (int q = 0; q < kRescoreGroup; ++q) cand[q] = cs;
        long_sums<1>(c, v, v < c.n, cand, 1, cx, dist);
    }
    double mv = 0.0;
    if (v < c.n) {
        mv = b.m64[v];
        if (cs >= 0 && dist[0] < mv) {
            mv = dist[0];
            b.m64[v] = mv;
            set_point_terms(b, v, mv);
        }
    }
    red[threadIdx.x] = mv;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double sum = tree_sum256(red, threadIdx.x);
        if (threadIdx.x == 0) b.fpart[blk] = sum;
    }
}

// Long rows with at least 4 ground-set chunks (small ground sets): the
// float64 squared distance of every point to one row in two passes, so the
// update and small re-score windows use more workgroups. Pass 1
// (blockIdx.y = slice q of the dimension, 16-byte reads as above) writes
// each point's partial sum to the per-chunk gains buffer, free at that point
// of a step, at part[q * n_pad + v]. Pass 2 adds the slices in order. The
// update takes one slice per chunk (up to 16); small re-score windows share
// the chunks among their candidates.
// Long rows take the long-row re-score and update kernels under the squared
// distance; L1 datasets take the generic ones (any row length) at every d.
__host__ __device__ inline bool long_path(const InstDesc& c) { return wide_rows(c.k_pad) && c.metric == 0; }
__host__ __device__ inline bool long_split(const InstDesc& c) { return long_path(c) && c.v_splits >= 4; }
__host__ __device__ inline int update_slices(const InstDesc& c) { return c.v_splits < 16 ? c.v_splits : 16; }
__device__ __forceinline__ int long_slice(int d, int S) { return ((d + S - 1) / S + 3) / 4 * 4; }
__device__ __forceinline__ int long_quarter(int d) { return long_slice(d, 4); }

__device__ void dist_slice_body(const InstDesc& c, int64_t blk, int q, int S, int64_t row) {
    if (row < 0 || q >= S) return;
    const float* __restrict__ x = c.x;
    const int d = c.d;
    const int Q = long_slice(d, S);
    const int k0 = q * Q;
    const int k1 = (k0 + Q) < d ? (k0 + Q) : d;
    const int64_t v = blk * kBlock + threadIdx.x;
    if (v >= c.n) return;
    const float* __restrict__ xv = x + v * d;
    const float* __restrict__ xc = x + row * d;
    double acc = 0.0;
    if ((d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0) {
        const float4* __restrict__ a4 = reinterpret_cast<const float4*>(xv);
        const float4* __restrict__ c4 = reinterpret_cast<const float4*>(xc);
#pragma unroll 8
        for (int k4 = k0 / 4; k4 < k1 / 4; ++k4) {
            const float4 a = a4[k4], b = c4[k4];
            const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double t = double(av[i]) - double(bv[i]);
                acc = fma(t, t, acc);
            }
        }
    } else {
        for (int k = k0; k < k1; ++k) {
            const double t = double(xv[k]) - double(xc[k]);
            acc = fma(t, t, acc);
        }
    }
    c.b.part[int64_t(q) * c.n_pad + v] = acc;
}

__device__ __forceinline__ double slices_sum(const InstDesc& c, int64_t v, int S) {
    const double* __restrict__ p = c.b.part;
    double s = p[v];
    for (int q = 1; q < S; ++q) s += p[int64_t(q) * c.n_pad + v];
    return s;
}

// Small re-score windows of long rows (at most v_splits/4, and 4,
// candidates): the same two passes per candidate, each candidate's distances
// over S = min(16, v_splits / W) slices; pass 1 over (candidate, slice) on
// blockIdx.y writing part[(S j + q) * n_pad + v].
__host__ __device__ inline int split_window(const InstDesc& c) {
    return long_split(c) ? (c.v_splits / 4 < 4 ? c.v_splits / 4 : 4) : 0;
}
__device__ __forceinline__ int window_slices(const InstDesc& c, int W) {
    const int s = c.v_splits / W;
    return s < 16 ? s : 16;
}

// Does the window's pass 1 hold the pick's distances (window position rank)?
// Their slices, and so the rounding of m_v, follow the window's size, which is
// the same in every run: the gains of long rows are, bit for bit (gains_wide.hip).
__device__ __forceinline__ bool window_has_slices(const InstDesc& c, int rank) {
    return rank >= 0 && c.b.state->window_count <= split_window(c);
}

// m_v update from the slice sums of the pick (pass 2), per-block sums of m_v.
// A small window's pass 1 has them already; otherwise dist_slices does.
__device__ void update_split_body(const InstDesc& c, int64_t blk, int cs, int rank) {
    __shared__ double red[kBlock];
    const Buffers& b = c.b;
    InstDesc w = c;
    int S = update_slices(c);
    if (window_has_slices(c, rank)) {
        S = window_slices(c, b.state->window_count);
        w.b.part = b.part + int64_t(S) * rank * c.n_pad;
    }
    const int64_t v = blk * kBlock + threadIdx.x;
    double mv = 0.0;
    if (v < c.n) {
        mv = b.m64[v];
        if (cs >= 0) {
            const double dist = slices_sum(w, v, S);
            if (dist < mv) {
                mv = dist;
                b.m64[v] = mv;
                set_point_terms(b, v, mv);
            }
        }
    }
    red[threadIdx.x] = mv;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double sum = tree_sum256(red, threadIdx.x);
        if (threadIdx.x == 0) b.fpart[blk] = sum;
    }
}

// Pass 1 of the update: the pick's slices, unless the window's pass 1 has them.
__device__ void update_slices_body(const InstDesc& c, int64_t blk, int q, int cs, int rank) {
    if (!window_has_slices(c, rank)) dist_slice_body(c, blk, q, update_slices(c), int64_t(cs));
}

// rpart rows a re-score of W candidates fills: one per 64-point sub-block
// for the one-pass long-row re-score, one per row block otherwise
__device__ __forceinline__ int rescore_rows(const InstDesc& c, int W) {
    return (long_path(c) && W > split_window(c)) ? 4 * c.nb : c.nb;
}

__device__ void dist_window_body(const InstDesc& c, int64_t blk, int y) {
    const int W = c.b.state->window_count;
    if (W > split_window(c)) return;  // the one-pass re-score takes it
    if (W == 0) return;
    const int S = window_slices(c, W);
    const int j = y / S, q = y % S;
    if (j >= W) return;
    // slice q of candidate j into the slot block S j + q
    InstDesc cj = c;
    cj.b.part = c.b.part + int64_t(S * j) * c.n_pad;
    dist_slice_body(cj, blk, q, S, int64_t(c.b.wfinal[j].idx));
}

__device__ void rescore_split_sum(const InstDesc& c, int64_t blk, double (*red)[kBlock]) {
    const int W = c.b.state->window_count;
    if (W > split_window(c) || W == 0) return;  // the same for the whole block
    const int64_t v = blk * kBlock + threadIdx.x;
    const double mv = v < c.n ? c.b.m64[v] : 0.0;
    const int S = window_slices(c, W);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        double val = 0.0;
        if (j < W && v < c.n) {
            InstDesc cj = c;
            cj.b.part = c.b.part + int64_t(S * j) * c.n_pad;
            val = fmax(0.0, mv - slices_sum(cj, v, S));
        }
        red[j][threadIdx.x] = val;
    }
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
#pragma unroll
            for (int j = 0; j < 4; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x < W) c.b.rpart[blk * kWindowMax + threadIdx.x] = red[threadIdx.x][0];
}

// ---- fsum (one block per instance): f(S_t) = L({e0}) - |V|^-1 sum m_v ----
__device__ void fsum_body(const InstDesc& c, int32_t t) {
    __shared__ double red[kBlock];
    double s = 0.0;
    for (int i = threadIdx.x; i < c.nb; i += kBlock) s += c.b.fpart[i];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < 64) s = tree_sum256(red, threadIdx.x);
    if (threadIdx.x == 0) {
        c.f[t] = c.b.state->l0 - s / double(c.n);
        if (c.b.state->cstar >= 0) c.b.selected[c.b.state->cstar] = 1;  // where the pick has not
    }
    if (!c.lazy) return;
    // heads of the next step's list: the best estimate of each stretch
    const int bps = list_stretch(c);
    const int heads = (c.nb + bps - 1) / bps;
    for (int h = threadIdx.x; h < heads; h += kBlock) {
        double e = -INFINITY;
        int row = c.b.barg[h * bps];
        for (int i = h * bps; i < (h + 1) * bps && i < c.nb; ++i)
            if (c.b.bmax[i] > e) {
                e = c.b.bmax[i];
                row = c.b.barg[i];
            }
        list_part(c, 0)[h] = c.b.inv ? c.b.inv[row] : row;
    }
    if (threadIdx.x == 0) {
        c.b.state->list_heads = heads;
        c.b.state->list_len = 0;
        c.b.state->list_exact = 0;
    }
}

// ---- lists (lazy.h) ----
// Per-chunk sums of the heads or the list -> gsum of their rows, and the m each
// was scored with. A workgroup of 1024 threads takes 32 list positions at a
// time; thread (p, q) adds chunks q, q + 32, ... of position p and the 32
// sums are added in q order.
constexpr int kListSumThreads = 1024;
constexpr int kListSumPos = 32;
__device__ void list_sum_body(const InstDesc& c, int32_t part, int64_t first, int64_t step) {
    __shared__ double red[kListSumThreads / kListSumPos][kListSumPos];
    const Buffers& b = c.b;
    const int64_t cnt = list_count(c, part);
    const ListGeom g = list_part_geom(c, part, cnt, list_tile(c.dt, c.metric));
    int32_t* __restrict__ rows = list_part(c, part);
    const int p = threadIdx.x % kListSumPos, q = threadIdx.x / kListSumPos;
    constexpr int Q = kListSumThreads / kListSumPos;
    for (int64_t p0 = first * kListSumPos; p0 < cnt; p0 += step * kListSumPos) {
        double s = 0.0;
        if (p0 + p < cnt)
            for (int i = q; i < g.splits; i += Q) s += b.part[int64_t(i) * g.stride + p0 + p];
        red[q][p] = s;
        __syncthreads();
        if (q == 0 && p0 + p < cnt) {
            for (int i = 1; i < Q; ++i) s += red[i][p];
            int32_t row = rows[p0 + p];
            if (b.perm) rows[p0 + p] = row = b.perm[row];
            b.gsum[row] = b.selected[row] ? -INFINITY : s;
            list_m(c)[row] = float(b.m64[row]);
        }
        __syncthreads();
    }
}

// Append every unselected candidate whose last gain reaches the window of the
// best head, less the rounding of the sums (lazy.h).
// Rows are taken in the grouped order where there is one, so that neighbours
// in the list are neighbours in space (their tiles clamp together).
__device__ void list_build_body(const InstDesc& c, int64_t blk) {
    __shared__ int wave_n[kBlock / 64];
    __shared__ int base;
    const Buffers& b = c.b;
    const int heads = b.state->list_heads;
    const int32_t* __restrict__ head = list_part(c, 0);
    double best = -INFINITY;  // each wave for itself
    for (int i = threadIdx.x & 63; i < heads; i += 64) best = fmax(best, b.gsum[head[i]]);
    best = wave_max(best);
    const double thr = window_threshold(best, b.state) - list_slack(c, best);
    const int64_t i = blk * kBlock + threadIdx.x;
    const int64_t row = b.perm ? int64_t(b.perm[i]) : i;
    const bool take = !b.selected[row] && b.gsum[row] >= thr;
    const uint64_t hit = __builtin_amdgcn_ballot_w64(take);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) wave_n[wave] = __popcll(hit);
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int w = 0; w < kBlock / 64; ++w) n += wave_n[w];
        base = n ? atomicAdd(&b.state->list_len, n) : 0;
    }
    __syncthreads();
    if (!take) return;
    int at = base + __popcll(hit & ((uint64_t(1) << lane) - 1));
    for (int w = 0; w < wave; ++w) at += wave_n[w];
    list_rows(c)[at] = int32_t(i);
}

// The window out of `len` candidates (one block): rows[0 .. len), or rows 0 ..
// len - 1 where rows is null. The same candidates, and the same rules above
// kWindowMax and kWindowCap of them, as wcount and wselect. Entries land in
// index or rank order, so nothing depends on the order of `rows`. perm
// non-null: `rows` holds slots of the grouped order. count: this block counts
// the window in the statistics (several blocks may make the same window).
// rounded (sums of other chunks than those of a step that scores all): where
// more than kWindowMax candidates reach the window or come as near as its
// rounding, no window is made, and the gain that they reach is returned;
// otherwise infinity.
template <int NT>
__device__ double window_body(const InstDesc& c, const int32_t* __restrict__ rows, const int32_t* __restrict__ perm,
                              int len, bool rounded, bool count) {
    __shared__ WindowEntry list[kWindowCap];
    __shared__ int hist[256];
    __shared__ int close;
    __shared__ double wg[NT / 64];
    __shared__ int wi[NT / 64];
    __shared__ int found;
    const Buffers& b = c.b;
    const int tid = threadIdx.x, lane = tid & 63;
    auto row_at = [&](int i) { return !rows ? i : (perm ? perm[rows[i]] : rows[i]); };
    double gb = -INFINITY, g0 = -INFINITY;
    int ib = 0x7fffffff, r0 = 0, none = 0;
    for (int i = tid; i < len; i += NT) {
        const int r = row_at(i);
        const double g = b.gsum[r];
        if (i == tid) {  // kept for the second pass
            g0 = g;
            r0 = r;
        }
        if (better(g, r, gb, ib)) {
            gb = g;
            ib = r;
        }
    }
    wave_best(gb, ib, none);
    if (lane == 0) {
        wg[tid >> 6] = gb;
        wi[tid >> 6] = ib;
    }
    if (tid == 0) found = close = 0;
    __syncthreads();
    gb = lane < NT / 64 ? wg[lane] : -INFINITY;
    ib = lane < NT / 64 ? wi[lane] : 0x7fffffff;
    wave_best(gb, ib, none);
    const double gmax = gb;
    const int first = ib;
    const double thr = window_threshold(gmax, b.state);
    auto inside = [&](double g) { return g >= thr && g > -INFINITY; };
    const double low = rounded ? thr - list_slack(c, gmax) : thr;
    int reach = 0;  // lane 0, which makes the most passes, has those of its wave
    for (int i = tid; i < len; i += NT) {
        const int r = i == tid ? r0 : row_at(i);
        const double g = i == tid ? g0 : b.gsum[r];
        if (rounded) reach += __popcll(__builtin_amdgcn_ballot_w64(g >= low && g > -INFINITY));
        if (!inside(g)) continue;
        const int at = atomicAdd(&found, 1);
        if (at >= kWindowCap) continue;
        list[at].g = g;
        list[at].idx = r;
        list[at].pad = 0;
    }
    if (rounded && lane == 0) atomicAdd(&close, reach);
    __syncthreads();
    const int total = found, near = close;
    __syncthreads();  // every wave has read it: found is reused below
    if (rounded && near > kWindowMax) return low;
    if (total <= kWindowCap) {
        for (int i = tid; i < total; i += NT) {
            int rank = 0;
            if (total <= kWindowMax)
                for (int j = 0; j < total; ++j) rank += list[j].idx < list[i].idx ? 1 : 0;
            else
                for (int j = 0; j < total; ++j) rank += better(list[j].g, list[j].idx, list[i].g, list[i].idx) ? 1 : 0;
            if (rank < kWindowMax) b.wfinal[rank] = list[i];
        }
    } else {
        // overflow: the best one, then the lowest indices among the others. The
        // largest index taken, byte by byte from the top: of the indices that
        // share the bytes so far, how many have each next byte?
        int hi = 0, need = kWindowMax - 1, shift = 0;
        while (int64_t(c.n) >> (shift + 8)) shift += 8;
        for (; shift >= 0; shift -= 8) {
            for (int i = tid; i < 256; i += NT) hist[i] = 0;
            __syncthreads();
            for (int i = tid; i < len; i += NT) {
                const int r = row_at(i);
                if (inside(b.gsum[r]) && r != first && int64_t(r) >> (shift + 8) == int64_t(hi) >> (shift + 8))
                    atomicAdd(&hist[(r >> shift) & 255], 1);
            }
            __syncthreads();
            // each wave for itself: the byte with which `need` indices are reached
            int n4[4], upto = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) upto += n4[i] = hist[4 * lane + i];
            const int own = upto;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int add = __shfl_up(upto, off, 64);
                if (lane >= off) upto += add;
            }
            const int at = __popcll(__builtin_amdgcn_ballot_w64(upto < need));  // its four bytes
            int before = upto - own, byte = 4 * lane;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (byte == 4 * lane + i && before + n4[i] < need) {
                    before += n4[i];
                    ++byte;
                }
            need -= __shfl(before, at, 64);
            hi |= __shfl(byte, at, 64) << shift;
            __syncthreads();  // hist is cleared again
        }
        if (tid == 0) found = 0;
        __syncthreads();
        for (int i = tid; i < len; i += NT) {
            const int r = row_at(i);
            const double g = b.gsum[r];
            if (!(inside(g) && r <= hi && r != first)) continue;
            const int at = atomicAdd(&found, 1);
            if (at >= kWindowMax - 1) continue;
            list[at].g = g;
            list[at].idx = r;
            list[at].pad = 0;
        }
        __syncthreads();
        for (int i = tid; i < kWindowMax - 1; i += NT) {
            int rank = 0;
            for (int j = 0; j < kWindowMax - 1; ++j) rank += list[j].idx < list[i].idx ? 1 : 0;
            b.wfinal[1 + rank] = list[i];
        }
        if (tid == 0) {
            WindowEntry e;
            e.g = gmax;
            e.idx = first;
            e.pad = 0;
            b.wfinal[0] = e;
        }
    }
    if (tid == 0) {
        b.state->window_count = total < kWindowMax ? total : kWindowMax;
        if (count && total > b.state->window_max) b.state->window_max = total;
        if (count && total > kWindowCap) b.state->window_overflow += 1;
    }
    return INFINITY;
}

// The window out of the list, or the candidates of the recount (lazy.h).
__device__ void list_window_body(const InstDesc& c) {
    __shared__ int kept;
    const Buffers& b = c.b;
    const int len = b.state->list_len, tid = threadIdx.x;
    int32_t* rows = list_rows(c);
    if (tid == 0) kept = 0;
    const double lower = window_body<kSelThreads>(c, rows, nullptr, len, !list_full_cut(c, len), true);
    if (lower < INFINITY)
        for (int i0 = 0; i0 < len; i0 += kSelThreads) {
            const int row = i0 + tid < len ? rows[i0 + tid] : -1;
            const double g = row >= 0 ? b.gsum[row] : -INFINITY;
            __syncthreads();  // entries up to here have been read: those kept take their places
            if (g >= lower && g > -INFINITY) rows[atomicAdd(&kept, 1)] = b.inv ? b.inv[row] : row;
            __syncthreads();
        }
    if (tid == 0) b.state->list_exact = kept;
}

// The recount's sums, added as gsum_body does, and the window out of them. Rare,
// and then one of the row blocks' own stages: every block makes the same sums
// and the same window and writes the same values, so none waits for another and
// the steps without a recount pay no launch for it.
__device__ void list_exact_body(const InstDesc& c, bool count) {
    const Buffers& b = c.b;
    const int len = b.state->list_exact;
    const ListGeom g = list_part_geom(c, 2, len, list_tile(c.dt, c.metric));
    const int32_t* rows = list_rows(c);
    for (int i = threadIdx.x; i < len; i += kBlock) {
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < g.splits; ++q) s += b.part[int64_t(q) * g.stride + i];
        const int32_t row = b.perm ? b.perm[rows[i]] : rows[i];
        b.gsum[row] = b.selected[row] ? -INFINITY : s;
    }
    __syncthreads();
    window_body<kBlock>(c, rows, b.perm, len, false, count);
    __syncthreads();
}

// ---- small ground sets (at most kSmallBlocks row blocks), solo, all
// candidates scored: the stages that need one block run as one kernel, and
// the pick is made by every block of the update for itself. 4 launches a step
// (gains, select, re-score, update) instead of 8: at this size each costs 2
// to 5 us and little else counts (1000 x 16, 5 steps with the data set: 208 -> 105 us) ----
constexpr int kSmallBlocks = 16;

// f of the previous step, the gain sums, the window.
__device__ void select_small_body(const InstDesc& c, int32_t t, int32_t splits) {
    const Buffers& b = c.b;
    const int tid = threadIdx.x;
    const int prev = t > 0 ? b.state->cstar : -1;  // not marked by its step's blocks
    if (t > 0 && tid < 64) {
        // the tree of fsum over at most kSmallBlocks sums
        double s = tid < c.nb ? b.fpart[tid] : 0.0;
#pragma unroll
        for (int off = kSmallBlocks / 2; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if (tid == 0) {
            c.f[t - 1] = b.state->l0 - s / double(c.n);
            if (prev >= 0) b.selected[prev] = 1;
        }
    }
    for (int64_t i = tid; i < c.n_pad; i += kSelThreads) {
        double g = 0.0;
#pragma unroll 8
        for (int s = 0; s < splits; ++s) g += b.part[int64_t(s) * c.n_pad + i];
        b.gsum[i] = b.selected[i] || i == prev ? -INFINITY : g;
    }
    window_body<kSelThreads>(c, nullptr, nullptr, int(c.n_pad), false, true);  // each thread reads the sums it wrote
}

__device__ int pick_small(const InstDesc& c, int32_t t, int64_t blk, int* rank) {
    double gain;
    const int cs = pick_choose<kBlock>(c, &gain, rank);
    if (blk == 0 && threadIdx.x == 0) pick_record(c, t, cs, gain, *rank, false);
    return cs;
}

// ---- solo kernels ----
__global__ void __launch_bounds__(kBlock) k_gsum(InstDesc c, int32_t splits) {
    gsum_body(c, blockIdx.x, splits);
}
__global__ void __launch_bounds__(kBlock) k_wcount(InstDesc c) { wcount_body(c, blockIdx.x); }
__global__ void __launch_bounds__(kSelThreads) k_wselect(InstDesc c) { wselect_body(c); }
__global__ void __launch_bounds__(kBlock) k_rescore(InstDesc c) { rescore_body(c, blockIdx.x); }
__global__ void __launch_bounds__(kPickThreads) k_pick(InstDesc c, int32_t t) { pick_body(c, t); }
__global__ void __launch_bounds__(kBlock) k_update(InstDesc c, int32_t t) {
    update_body(c, blockIdx.x, t, c.b.state->cstar, c.b.state->crank);
}
__global__ void __launch_bounds__(kBlock) k_update_l1(InstDesc c, int32_t t) {
    update_l1_body(c, blockIdx.x, t, c.b.state->cstar, c.b.state->crank);
}
__global__ void __launch_bounds__(kBlock) k_rescore_long(InstDesc c) { rescore_long_body(c, blockIdx.x, blockIdx.y); }
__global__ void __launch_bounds__(kBlock) k_update_long(InstDesc c) { update_long_body(c, blockIdx.x); }
__global__ void __launch_bounds__(kBlock) k_dist_slices(InstDesc c) {
    update_slices_body(c, blockIdx.x, blockIdx.y, c.b.state->cstar, c.b.state->crank);
}
__global__ void __launch_bounds__(kBlock) k_update_split(InstDesc c) {
    update_split_body(c, blockIdx.x, c.b.state->cstar, c.b.state->crank);
}
__global__ void __launch_bounds__(kSelThreads) k_select_small(InstDesc c, int32_t t, int32_t splits) {
    select_small_body(c, t, splits);
}
__global__ void __launch_bounds__(kBlock) k_update_small(InstDesc c, int32_t t) {
    int rank;
    const int cs = pick_small(c, t, blockIdx.x, &rank);
    if (c.metric == 1)
        update_l1_body(c, blockIdx.x, t, cs, rank);
    else
        update_body(c, blockIdx.x, t, cs, rank);
}
__global__ void __launch_bounds__(kBlock) k_slices_small(InstDesc c, int32_t t) {
    double gain;
    int rank;
    const int cs = pick_choose<kBlock>(c, &gain, &rank);
    update_slices_body(c, blockIdx.x, blockIdx.y, cs, rank);
}
__global__ void __launch_bounds__(kBlock) k_update_split_small(InstDesc c, int32_t t) {
    int rank;
    const int cs = pick_small(c, t, blockIdx.x, &rank);
    update_split_body(c, blockIdx.x, cs, rank);
}
__global__ void __launch_bounds__(kBlock) k_dist_window(InstDesc c) { dist_window_body(c, blockIdx.x, blockIdx.y); }
__global__ void __launch_bounds__(kBlock) k_fsum(InstDesc c, int32_t t) { fsum_body(c, t); }
__global__ void __launch_bounds__(kListSumThreads) k_list_sum(InstDesc c, int32_t part) {
    list_sum_body(c, part, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(kBlock) k_list_build(InstDesc c) { list_build_body(c, blockIdx.x); }
__global__ void __launch_bounds__(kSelThreads) k_list_window(InstDesc c) { list_window_body(c); }

// ---- batched kernels: blocks of row_pre[i] .. row_pre[i+1] belong to instance i;
// tick t runs step t0 + t of each instance; instances whose k is reached skip ----
#define EBC_ROW_KERNEL(NAME, COND, BODY)                                                               \
    __global__ void __launch_bounds__(kBlock)                                                          \
        NAME(const InstDesc* __restrict__ descs, const int64_t* __restrict__ row_pre, int32_t count,   \
             int32_t t) {                                                                              \
        const int i = find_slot(row_pre, count, blockIdx.x);                                           \
        const InstDesc c = descs[i];                                                                   \
        const int32_t step = c.t0 + t;                                                                 \
        const int64_t blk = int64_t(blockIdx.x) - row_pre[i];                                          \
        if (step < c.k && (COND)) BODY;                                                                \
    }
EBC_ROW_KERNEL(kb_gsum, !list_step(c, step), gsum_body(c, blk, gain_splits(c, step)))
EBC_ROW_KERNEL(kb_wcount, !list_step(c, step), wcount_body(c, blk))
EBC_ROW_KERNEL(kb_list_build, list_step(c, step), list_build_body(c, blk))
// mixed batches: each re-score / update body runs only for its own row length
__device__ __forceinline__ void update_long(const InstDesc& c, int64_t blk) {
    if (long_split(c))
        update_split_body(c, blk, c.b.state->cstar, c.b.state->crank);
    else
        update_long_body(c, blk);
}
EBC_ROW_KERNEL(kb_rescore, !wide_rows(c.k_pad), rescore_body(c, blk))
EBC_ROW_KERNEL(kb_update, !wide_rows(c.k_pad), update_body(c, blk, step, c.b.state->cstar, c.b.state->crank))
EBC_ROW_KERNEL(kb_rescore_long, wide_rows(c.k_pad), rescore_long_body(c, blk, blockIdx.y))
EBC_ROW_KERNEL(kb_update_long, wide_rows(c.k_pad), update_long(c, blk))
EBC_ROW_KERNEL(kb_dist_slices, long_split(c),
               update_slices_body(c, blk, blockIdx.y, c.b.state->cstar, c.b.state->crank))
EBC_ROW_KERNEL(kb_dist_window, long_split(c), dist_window_body(c, blk, blockIdx.y))
#undef EBC_ROW_KERNEL

__global__ void __launch_bounds__(kSelThreads) kb_wselect(const InstDesc* __restrict__ descs, int32_t t) {
    const InstDesc c = descs[blockIdx.x];
    if (c.t0 + t < c.k && !list_step(c, c.t0 + t)) wselect_body(c);
}
// lists: instance on blockIdx.y / blockIdx.x
__global__ void __launch_bounds__(kListSumThreads) kb_list_sum(const InstDesc* __restrict__ descs, int32_t t,
                                                               int32_t part) {
    const InstDesc c = descs[blockIdx.y];
    if (c.t0 + t < c.k && list_step(c, c.t0 + t)) list_sum_body(c, part, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(kSelThreads) kb_list_window(const InstDesc* __restrict__ descs, int32_t t) {
    const InstDesc c = descs[blockIdx.x];
    if (c.t0 + t < c.k && list_step(c, c.t0 + t)) list_window_body(c);
}
__global__ void __launch_bounds__(kPickThreads) kb_pick(const InstDesc* __restrict__ descs, int32_t t) {
    const InstDesc c = descs[blockIdx.x];
    if (c.t0 + t < c.k) pick_body(c, c.t0 + t);
}
__global__ void __launch_bounds__(kBlock) kb_fsum(const InstDesc* __restrict__ descs, int32_t t) {
    const InstDesc c = descs[blockIdx.x];
    if (c.t0 + t < c.k) fsum_body(c, c.t0 + t);
}

hipError_t launch_greedy_step(const ebc_dataset* ds, int32_t t, int32_t k, int32_t* sel_out, double* f_out,
                              double* gain_out, hipStream_t s, hipEvent_t ev_gains_done) {
    InstDesc c;
    fill_desc(ds, k, sel_out, f_out, gain_out, &c);
    if (ds->prof) {  // a timed step is a whole launch
        c.lazy = 0;
        c.b.pairs = nullptr;
    }
    const int nb = c.nb;
    hipError_t e = hipSuccess;
    if (list_step(c, t)) {
        if ((e = launch_list_step(c, s)) != hipSuccess) return e;
    } else {
        if (matrix_step(c, t))
            e = launch_gains_matrix(c, s);
        else if (c.metric == 0 && pair_matrix(c.n_pad, c.k_pad))
            e = launch_gains_wide_pairs(c, s);
        else
            e = launch_gains(ds, s);
        if (e != hipSuccess) return e;
        if (ev_gains_done && (e = hipEventRecord(ev_gains_done, s)) != hipSuccess) return e;
        if (nb <= kSmallBlocks && c.lazy == 0 && (c.metric == 1 || !wide_rows(c.k_pad) || long_split(c))) {
            hipLaunchKernelGGL(k_select_small, dim3(1), dim3(kSelThreads), 0, s, c, t, gain_splits(c, t));
            if (c.metric == 0 && wide_rows(c.k_pad)) {
                hipLaunchKernelGGL(k_dist_window, dim3(nb, 16), dim3(kBlock), 0, s, c);
                hipLaunchKernelGGL(k_rescore_long, dim3(nb, 4 * kWindowMax / kRescoreGroup), dim3(kBlock), 0, s, c);
                hipLaunchKernelGGL(k_slices_small, dim3(nb, update_slices(c)), dim3(kBlock), 0, s, c, t);
                hipLaunchKernelGGL(k_update_split_small, dim3(nb), dim3(kBlock), 0, s, c, t);
            } else {
                hipLaunchKernelGGL(k_rescore, dim3(nb), dim3(kBlock), 0, s, c);
                hipLaunchKernelGGL(k_update_small, dim3(nb), dim3(kBlock), 0, s, c, t);
            }
            // f(S_t) and the mark of the pick: the next step's select, or here
            if (t + 1 == k) hipLaunchKernelGGL(k_fsum, dim3(1), dim3(kBlock), 0, s, c, t);
            return hipGetLastError();
        }
        hipLaunchKernelGGL(k_gsum, dim3(nb), dim3(kBlock), 0, s, c, gain_splits(c, t));
        hipLaunchKernelGGL(k_wcount, dim3(nb), dim3(kBlock), 0, s, c);
        hipLaunchKernelGGL(k_wselect, dim3(1), dim3(kSelThreads), 0, s, c);
    }
    if (nb <= kPickBlocks && (c.metric == 1 || !wide_rows(c.k_pad))) {
        hipLaunchKernelGGL(k_rescore, dim3(nb), dim3(kBlock), 0, s, c);
        hipLaunchKernelGGL(k_update_small, dim3(nb), dim3(kBlock), 0, s, c, t);
    } else if (c.metric == 1) {
        hipLaunchKernelGGL(k_rescore, dim3(nb), dim3(kBlock), 0, s, c);
        hipLaunchKernelGGL(k_pick, dim3(1), dim3(kPickThreads), 0, s, c, t);
        hipLaunchKernelGGL(k_update_l1, dim3(nb), dim3(kBlock), 0, s, c, t);
    } else if (wide_rows(c.k_pad)) {
        // small windows: pass 1 over slices of the dimension here, pass 2 inside k_rescore_long
        if (long_split(c)) hipLaunchKernelGGL(k_dist_window, dim3(nb, 16), dim3(kBlock), 0, s, c);
        hipLaunchKernelGGL(k_rescore_long, dim3(nb, 4 * kWindowMax / kRescoreGroup), dim3(kBlock), 0, s, c);
        hipLaunchKernelGGL(k_pick, dim3(1), dim3(kPickThreads), 0, s, c, t);
        if (long_split(c)) {
            hipLaunchKernelGGL(k_dist_slices, dim3(nb, update_slices(c)), dim3(kBlock), 0, s, c);
            hipLaunchKernelGGL(k_update_split, dim3(nb), dim3(kBlock), 0, s, c);
        } else {
            hipLaunchKernelGGL(k_update_long, dim3(nb), dim3(kBlock), 0, s, c);
        }
    } else {
        hipLaunchKernelGGL(k_rescore, dim3(nb), dim3(kBlock), 0, s, c);
        hipLaunchKernelGGL(k_pick, dim3(1), dim3(kPickThreads), 0, s, c, t);
        hipLaunchKernelGGL(k_update, dim3(nb), dim3(kBlock), 0, s, c, t);
    }
    hipLaunchKernelGGL(k_fsum, dim3(1), dim3(kBlock), 0, s, c, t);
    return hipGetLastError();
}

// Gains, sums, list and window of a step that scores a list.
hipError_t launch_list_step(const InstDesc& c, hipStream_t s) {
    const unsigned sums = 256;  // workgroups; each walks its share of the list
    for (int32_t part = 0; part < 3; ++part) {
        const hipError_t e = launch_gains_list(c, part, s);
        if (e != hipSuccess) return e;
        if (part < 2)
            hipLaunchKernelGGL(k_list_sum, dim3(part ? sums : kListHeads / kListSumPos), dim3(kListSumThreads), 0, s, c,
                               part);
        if (part == 0) hipLaunchKernelGGL(k_list_build, dim3(c.nb), dim3(kBlock), 0, s, c);
        if (part == 1) hipLaunchKernelGGL(k_list_window, dim3(1), dim3(kSelThreads), 0, s, c);
    }
    return hipGetLastError();
}

hipError_t launch_tick(const std::vector<GainsBucket>& buckets, const InstDesc* descs, const int64_t* row_pre,
                       const int32_t* slot_inst, const int64_t* wg_pre, int32_t count, int64_t total_rows, int32_t t,
                       bool full, bool lists, bool long_rows, hipStream_t s) {
    const dim3 rows = dim3(unsigned(total_rows)), one = dim3(unsigned(count));
    hipError_t e = hipSuccess;
    if (full) {
        for (const GainsBucket& b : buckets)
            if ((e = launch_gains_batched(b.key, descs, slot_inst + b.slot_begin, wg_pre + b.pre_off, b.slots,
                                          b.total_wgs, t, s)) != hipSuccess)
                return e;
        if (long_rows && (e = launch_gains_matrix_batched(descs, row_pre, count, total_rows, t, s)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(kb_gsum, rows, dim3(kBlock), 0, s, descs, row_pre, count, t);
        hipLaunchKernelGGL(kb_wcount, rows, dim3(kBlock), 0, s, descs, row_pre, count, t);
        hipLaunchKernelGGL(kb_wselect, one, dim3(kSelThreads), 0, s, descs, t);
    }
    if (lists) {
        for (int32_t part = 0; part < 3; ++part) {
            for (const GainsBucket& b : buckets)
                if (b.lists && (e = launch_gains_list_batched(b.key, descs, slot_inst + b.slot_begin, b.slots, t, part,
                                                              s)) != hipSuccess)
                    return e;
            if (part < 2)
                hipLaunchKernelGGL(kb_list_sum, dim3(part ? 32 : kListHeads / kListSumPos, unsigned(count)),
                                   dim3(kListSumThreads), 0, s, descs, t, part);
            if (part == 0) hipLaunchKernelGGL(kb_list_build, rows, dim3(kBlock), 0, s, descs, row_pre, count, t);
            if (part == 1) hipLaunchKernelGGL(kb_list_window, one, dim3(kSelThreads), 0, s, descs, t);
        }
    }
    hipLaunchKernelGGL(kb_rescore, rows, dim3(kBlock), 0, s, descs, row_pre, count, t);
    if (long_rows) {
        hipLaunchKernelGGL(kb_dist_window, dim3(unsigned(total_rows), 16), dim3(kBlock), 0, s, descs, row_pre, count,
                           t);
        hipLaunchKernelGGL(kb_rescore_long, dim3(unsigned(total_rows), 4 * kWindowMax / kRescoreGroup), dim3(kBlock), 0, s,
                           descs, row_pre, count, t);
    }
    hipLaunchKernelGGL(kb_pick, one, dim3(kPickThreads), 0, s, descs, t);
    hipLaunchKernelGGL(kb_update, rows, dim3(kBlock), 0, s, descs, row_pre, count, t);
    if (long_rows) {
        hipLaunchKernelGGL(kb_dist_slices, dim3(unsigned(total_rows), 16), dim3(kBlock), 0, s, descs, row_pre, count,
                           t);
        hipLaunchKernelGGL(kb_update_long, rows, dim3(kBlock), 0, s, descs, row_pre, count, t);
    }
    hipLaunchKernelGGL(kb_fsum, one, dim3(kBlock), 0, s, descs, t);
    return hipGetLastError();
}

static hipError_t launch_gains_args(const ebc_dataset* ds, const GainsArgs& ga, hipStream_t s) {
    if (ds->metric == 1) return launch_gains_l1(ds, ga, s);
    if (wide_rows(ds->k_pad)) return launch_gains_wide(ds, ga, s);
    return ds->dt == EBC_DT_F32 ? launch_gains_f32(ds, ga, s) : launch_gains_lp(ds, ga, s);
}

hipError_t launch_gains(const ebc_dataset* ds, hipStream_t s) {
    InstDesc c;
    fill_desc(ds, 0, nullptr, nullptr, nullptr, &c);
    return launch_gains_args(ds, gains_args(c, nullptr, ds->n_pad), s);
}

hipError_t launch_gains_call(const ebc_dataset* ds, const int32_t* cand, int64_t n_cand, hipStream_t s) {
    InstDesc c;
    fill_desc(ds, 0, nullptr, nullptr, nullptr, &c);
    c.v_splits = call_splits_for(ds->n_pad, ds->k_pad, ds->dt);
    c.chunk = gains_chunk(ds, c.v_splits);
    return launch_gains_args(ds, gains_args(c, cand, n_cand), s);
}

hipError_t launch_gains_list(const InstDesc& c, int32_t part, hipStream_t s) {
    if (c.metric == 1) return launch_gains_l1_list(c, part, s);
    return c.dt == EBC_DT_F32 ? launch_gains_f32_list(c, part, s) : launch_gains_lp_list(c, part, s);
}

// Marginal-gains output: sum the per-chunk sums, divide by |V|.
__global__ void __launch_bounds__(kBlock)
k_gains_out(int64_t n, int64_t n_cand, int64_t stride, int32_t v_splits, const double* part, double* out) {
    const int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= n_cand) return;
    double g = 0.0;
#pragma unroll 8
    for (int s = 0; s < v_splits; ++s) g += part[int64_t(s) * stride + p];
    out[p] = g / double(n);
}

hipError_t launch_gains_out(const ebc_dataset* ds, int64_t n_cand, double* out, hipStream_t s) {
    const unsigned nb = unsigned((n_cand + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_gains_out, dim3(nb), dim3(kBlock), 0, s, ds->n, n_cand, ds->n_pad,
                       call_splits_for(ds->n_pad, ds->k_pad, ds->dt), ds->b.part, out);
    return hipGetLastError();
}

}  // namespace ebc
