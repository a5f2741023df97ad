// Marginal gains of many candidates at once, float32 on the MFMA units.
//
// For the current running minima m_v (the per-point terms of L(S u {e0}),
// Sec. 4.1, Eq. loss_decomposed) the gain of candidate c is
//     G[c] = sum_v max(0, m_v - d(v, c))               (|V| * Delta(c|S), Sec. 3)
// With d(v,c) = ||v||^2 + ||c||^2 - 2 v.c and all terms halved (exact in
// binary floating point):
//     G[c] / 2 = sum_v med3( v.c + ha_v - hn_c, 0, hm_v )
// where hn = ||.||^2/2, hm_v = m_v/2, ha_v = hm_v - hn_v, and med3 clamps the
// per-point term to [0, m_v/2] (the clamp at m_v is the clamp d >= 0).
//
// The paper's kernel (Alg. 2) gives every (set, point) cell of the work
// matrix W its own thread and writes W to global memory before a W*1 sum.
// Here the dot products v.c are a dense contraction on the matrix cores
// (v_mfma_f32_32x32x2_f32), the clamp and the sum over v are fused into the
// accumulator epilogue, and no distance or work matrix is ever written.
//
// Work decomposition: a workgroup (4 waves) owns 128 candidates (32 per
// wave, their rows held in registers for the whole kernel) and one chunk of
// the ground set; it streams that chunk through LDS in tiles of 64 points.
// MFMA tile: rows = 32 candidates, columns = 32 ground points, K = the
// dimension, split in two halves so that every lane reads contiguous K.
// Rows are padded to KP (a multiple of 8); when the last 4 values of a row
// are padding (TRIM: d <= KP - 4), the last two K steps pair values KH - 4,
// KH - 3 (lane half 0) with KH - 2, KH - 1 (lane half 1) instead of running
// two more steps whose half-1 values are all zeros: KH - 2 matrix
// instructions per column block instead of KH (50 instead of 52 at d = 100).
#include "ebc_internal.h"
#include "lazy.h"

namespace ebc {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// The prefetched tile lives in one wide vector value (not an array) so that
// it stays in registers across the loop.
template <int PER>
using PreVec = float __attribute__((ext_vector_type(4 * PER)));

template <int PER, int NV4>
__device__ __forceinline__ PreVec<PER> load_rows(const float4* __restrict__ src, int tid) {
    PreVec<PER> pre;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = tid + i * 256;
        const float4 t = src[e < NV4 ? e : NV4 - 1];  // clamped: stays inside the tile
        pre[4 * i + 0] = t.x;
        pre[4 * i + 1] = t.y;
        pre[4 * i + 2] = t.z;
        pre[4 * i + 3] = t.w;
    }
    return pre;
}

template <int KP, bool TRIM>
__device__ __forceinline__ void gains_f32_body(const GainsArgs& ga, int64_t bid) {
    const float* __restrict__ xq = static_cast<const float*>(ga.xq);
    const float* __restrict__ hn = ga.hn;
    const float* __restrict__ ha = ga.ha;
    const float* __restrict__ hm = ga.hm;
    const int32_t* __restrict__ cand = ga.cand;
    const int64_t n_cand = ga.n_cand, n_pad = ga.n_pad, chunk = ga.chunk, part_stride = ga.part_stride;
    const int32_t v_splits = ga.v_splits;
    double* __restrict__ part = ga.part;
    int* __restrict__ err = ga.err;
    constexpr int KH = KP / 2;        // K values per lane half
    constexpr int S = KP + 4;         // LDS row stride in floats (S/4 odd: conflict-free b128)
    constexpr int VT = kGainsVTile;   // ground points per LDS stage
    constexpr int NV4 = VT * KP / 4;  // float4 per stage
    constexpr int PER = (NV4 + 255) / 256;
    static_assert(KP % 8 == 0, "row length must be a multiple of 8");

    __shared__ float4 lds_x4[VT * S / 4];
    __shared__ float lds_ha[VT];
    __shared__ float lds_hm[VT];
    float* lds_x = reinterpret_cast<float*>(lds_x4);

    const int tid = fresh_tid();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int col = lane & 31;  // MFMA column within a 32-block
    const int half = lane >> 5;

    // (candidate tile, ground chunk) of this workgroup. Consecutive ids go to
    // the 8 XCDs in turn; with 8 G chunks, XCD x takes chunks x, x + 8, ...
    // one after the other (every candidate tile of chunk x first), so its L2
    // holds one chunk's rows at a time. 8 chunks: chunk = id % 8.
    int split;
    int64_t ctile;
    if (v_splits % 8 == 0) {
        const uint32_t ntiles = uint32_t((n_cand + kGainsCandTile - 1) / kGainsCandTile);
        const uint32_t r = uint32_t(bid) / 8;
        split = int(uint32_t(bid) % 8) + 8 * int(r / ntiles);
        ctile = r % ntiles;
    } else {
        split = int(uint32_t(bid) % uint32_t(v_splits));
        ctile = uint32_t(bid) / uint32_t(v_splits);
    }

    // ---- candidate rows of this wave, in registers (MFMA A operand) ----
    const int64_t cpos = ctile * kGainsCandTile + wave * 32 + col;  // position in the candidate list
    // Candidate rows outside [0, n_pad) (a bad caller list) compute as zero
    // rows and raise EBC_E_INDEX.
    int64_t crow = -1;
    if (cpos < n_cand) crow = cand ? int64_t(cand[cpos]) : cpos;
    if (crow >= n_pad || crow < -1 || (cpos < n_cand && crow < 0)) {
        atomicCAS(err, 0, kDevErrIndex);
        crow = -1;
    }
    constexpr int QF = TRIM ? KH / 4 - 1 : KH / 4;  // groups of 4 K steps on contiguous halves
    float a[KH];
    if (crow >= 0) {
        const float4* src = reinterpret_cast<const float4*>(xq + crow * KP + half * KH);
#pragma unroll
        for (int q = 0; q < QF; ++q) {
            const float4 t = src[q];
            a[4 * q + 0] = t.x;
            a[4 * q + 1] = t.y;
            a[4 * q + 2] = t.z;
            a[4 * q + 3] = t.w;
        }
        if constexpr (TRIM) {  // half 0: values KH-4, KH-3; half 1: KH-2, KH-1
            const float2 t = *reinterpret_cast<const float2*>(xq + crow * KP + (half ? KH - 2 : KH - 4));
            a[KH - 4] = t.x;
            a[KH - 3] = t.y;
            a[KH - 2] = 0.0f;
            a[KH - 1] = 0.0f;
        }
    } else {
#pragma unroll
        for (int j = 0; j < KH; ++j) a[j] = 0.0f;
    }
    // -hn of the 16 candidate rows this lane holds in the MFMA result, from
    // the lanes that loaded these rows
    const float hc = crow >= 0 ? hn[crow] : 0.0f;
    float nhn[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) nhn[r] = -__shfl(hc, acc_row(r, half), 64);
    float acc_sum[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_sum[r] = 0.0f;
    // the previous column block, its clamp-and-sum still to do (none yet:
    // -inf clamps to +0, which leaves the sums as they are)
    floatx16 accP;
    float hmP = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) accP[r] = -INFINITY;

    // ---- stream the ground-set chunk ----
    const int64_t v_begin = int64_t(split) * chunk;
    int64_t v_end = v_begin + chunk;
    if (v_end > n_pad) v_end = n_pad;

    // Next tile's rows are fetched into registers while the current tile's
    // MFMAs run, then written to LDS between two barriers.
    PreVec<PER> pre;
    float pre_ha = 0.0f, pre_hm = 0.0f;
    if (v_begin < v_end) {
        pre = load_rows<PER, NV4>(reinterpret_cast<const float4*>(xq + v_begin * KP), tid);
        if (tid < VT) {
            pre_ha = ha[v_begin + tid];
            pre_hm = hm[v_begin + tid];
        }
    }
    for (int64_t v0 = v_begin; v0 < v_end; v0 += VT) {
        __syncthreads();  // previous tile fully consumed
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = tid + i * 256;
            if (e < NV4) {
                const int row = e / (KP / 4);
                const int q = e % (KP / 4);
                lds_x4[(row * S) / 4 + q] = make_float4(pre[4 * i], pre[4 * i + 1], pre[4 * i + 2], pre[4 * i + 3]);
            }
        }
        if (tid < VT) {
            lds_ha[tid] = pre_ha;
            lds_hm[tid] = pre_hm;
        }
        __syncthreads();
        if (v0 + VT < v_end) {  // in flight during the MFMAs
            pre = load_rows<PER, NV4>(reinterpret_cast<const float4*>(xq + (v0 + VT) * KP), tid);
            if (tid < VT) {
                pre_ha = ha[v0 + VT + tid];
                pre_hm = hm[v0 + VT + tid];
            }
        }

#pragma unroll
        for (int cb = 0; cb < VT / 32; ++cb) {
            const int vrow = cb * 32 + col;
            const float hav = lds_ha[vrow];
            const float hmv = lds_hm[vrow];
            floatx16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = nhn[r] + hav;
            const float4* b4 = reinterpret_cast<const float4*>(lds_x + vrow * S + half * KH);
            // The previous block's clamp-and-sum is issued in slices between
            // groups of this block's MFMAs (it does not depend on them, and
            // the sums keep their block order); the next group's operand read
            // is issued before each group.
            constexpr int SL = QF > 0 ? (16 + QF - 1) / QF : 16;  // terms per group
            float4 bv = b4[0];
#pragma unroll
            for (int q = 0; q < QF; ++q) {
                const float4 bn = q + 1 < QF ? b4[q + 1] : bv;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 0], bv.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 1], bv.y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 2], bv.z, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 3], bv.w, acc, 0, 0, 0);
#pragma unroll
                for (int r = q * SL; r < (q + 1) * SL && r < 16; ++r)
                    acc_sum[r] += __builtin_amdgcn_fmed3f(accP[r], 0.0f, hmP);
                __builtin_amdgcn_sched_barrier(0);
                bv = bn;
            }
            if constexpr (TRIM) {
                const float2 bt = *reinterpret_cast<const float2*>(lds_x + vrow * S + (half ? KH - 2 : KH - 4));
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[KH - 4], bt.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[KH - 3], bt.y, acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = QF * SL; r < 16; ++r) acc_sum[r] += __builtin_amdgcn_fmed3f(accP[r], 0.0f, hmP);  // QF = 0
            accP = acc;
            hmP = hmv;
        }
    }
    // the last block's clamp-and-sum
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_sum[r] += __builtin_amdgcn_fmed3f(accP[r], 0.0f, hmP);

    // ---- sum over the 32 columns (ground points) of each half, in float64 ----
    const double mine = column_sums16(acc_sum, col);
    if ((col & 1) == 0) {
        const int64_t p = ctile * kGainsCandTile + wave * 32 + acc_row(col >> 1, half);
        if (p < n_cand) part[int64_t(split) * part_stride + p] = 2.0 * mine;
    }
}

// Short candidate lists: 32 candidates per workgroup instead of 128, each wave
// taking one of the four 32-point blocks of a 128-point tile. The clamped
// terms of the four blocks meet in LDS and are added in block order (wave w
// adds the result rows of registers 4w .. 4w + 3), so every sum is, bit for
// bit, the one the 128-candidate kernel makes of the same chunk, while a
// chunk takes a quarter of the time and a list four times the workgroups.
// Bound: matrix instructions, as there; the terms cost 16 LDS writes and reads
// per lane and block of 50 of them (d = 100). 50000 x 100: a call for one
// candidate 172 -> 67 us, for 300 178 -> 71 us.
template <int KP, bool TRIM>
__global__ void __launch_bounds__(256) k_gains_f32_narrow(GainsArgs ga) {
    const float* __restrict__ xq = static_cast<const float*>(ga.xq);
    const int64_t n_pad = ga.n_pad;
    constexpr int KH = KP / 2;
    constexpr int S = KP + 4;
    constexpr int VT = 128;
    constexpr int NV4 = VT * KP / 4;
    constexpr int PER = (NV4 + 255) / 256;
    constexpr int QF = TRIM ? KH / 4 - 1 : KH / 4;

    __shared__ float4 lds_x4[VT * S / 4];
    __shared__ float lds_ha[VT];
    __shared__ float lds_hm[VT];
    __shared__ float terms[4][16][64];
    float* lds_x = reinterpret_cast<float*>(lds_x4);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int col = lane & 31;
    const int half = lane >> 5;
    const int split = int(uint32_t(blockIdx.x) % uint32_t(ga.v_splits));
    const int64_t cbase = int64_t(uint32_t(blockIdx.x) / uint32_t(ga.v_splits)) * 32;

    const int64_t cpos = cbase + col;
    int64_t crow = -1;
    if (cpos < ga.n_cand) {
        crow = ga.cand ? int64_t(ga.cand[cpos]) : cpos;
        if (crow >= n_pad || crow < 0) {
            atomicCAS(ga.err, 0, kDevErrIndex);
            crow = -1;
        }
    }
    float a[KH];
    if (crow >= 0) {
        const float4* src = reinterpret_cast<const float4*>(xq + crow * KP + half * KH);
#pragma unroll
        for (int q = 0; q < QF; ++q) {
            const float4 t = src[q];
            a[4 * q + 0] = t.x;
            a[4 * q + 1] = t.y;
            a[4 * q + 2] = t.z;
            a[4 * q + 3] = t.w;
        }
        if constexpr (TRIM) {
            const float2 t = *reinterpret_cast<const float2*>(xq + crow * KP + (half ? KH - 2 : KH - 4));
            a[KH - 4] = t.x;
            a[KH - 3] = t.y;
            a[KH - 2] = 0.0f;
            a[KH - 1] = 0.0f;
        }
    } else {
#pragma unroll
        for (int j = 0; j < KH; ++j) a[j] = 0.0f;
    }
    const float hc = crow >= 0 ? ga.hn[crow] : 0.0f;
    float nhn[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) nhn[r] = -__shfl(hc, acc_row(r, half), 64);
    float acc_sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // result rows of registers 4 wave + i

    const int64_t v_begin = int64_t(split) * ga.chunk;
    int64_t v_end = v_begin + ga.chunk;
    if (v_end > n_pad) v_end = n_pad;

    // rows past v_end (a chunk is a multiple of 64 points) are read from the
    // tile's first rows instead and their block is not added
    auto load = [&](int64_t v0) {
        const int64_t rows = v_end - v0 < VT ? v_end - v0 : VT;
        const int nv4 = int(rows) * (KP / 4);
        const float4* __restrict__ src = reinterpret_cast<const float4*>(xq + v0 * KP);
        PreVec<PER> pre;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = tid + i * 256;
            const float4 t = src[e < nv4 ? e : 0];
            pre[4 * i + 0] = t.x;
            pre[4 * i + 1] = t.y;
            pre[4 * i + 2] = t.z;
            pre[4 * i + 3] = t.w;
        }
        return pre;
    };
    PreVec<PER> pre;
    float pre_ha = 0.0f, pre_hm = 0.0f;
    auto load_points = [&](int64_t v0) {
        if (tid < VT && v0 + tid < v_end) {
            pre_ha = ga.ha[v0 + tid];
            pre_hm = ga.hm[v0 + tid];
        }
    };
    if (v_begin < v_end) {
        pre = load(v_begin);
        load_points(v_begin);
    }
    int blocks = 0;  // blocks whose terms are in LDS, not yet added
    auto add_terms = [&]() {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (b >= blocks) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) acc_sum[i] += terms[b][4 * wave + i][lane];
        }
    };
    for (int64_t v0 = v_begin; v0 < v_end; v0 += VT) {
        __syncthreads();  // previous tile multiplied, its terms written
        add_terms();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = tid + i * 256;
            if (e < NV4) {
                const int row = e / (KP / 4);
                const int q = e % (KP / 4);
                lds_x4[(row * S) / 4 + q] = make_float4(pre[4 * i], pre[4 * i + 1], pre[4 * i + 2], pre[4 * i + 3]);
            }
        }
        if (tid < VT) {
            lds_ha[tid] = pre_ha;
            lds_hm[tid] = pre_hm;
        }
        __syncthreads();
        if (v0 + VT < v_end) {
            pre = load(v0 + VT);
            load_points(v0 + VT);
        }
        blocks = v_end - v0 < VT ? int(v_end - v0) / 32 : 4;
        const int vrow = wave * 32 + col;
        const float hav = lds_ha[vrow];
        const float hmv = lds_hm[vrow];
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = nhn[r] + hav;
        const float4* b4 = reinterpret_cast<const float4*>(lds_x + vrow * S + half * KH);
        float4 bv = b4[0];
#pragma unroll
        for (int q = 0; q < QF; ++q) {
            const float4 bn = q + 1 < QF ? b4[q + 1] : bv;  // read ahead of the group that needs it
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 0], bv.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 1], bv.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 2], bv.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[4 * q + 3], bv.w, acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            bv = bn;
        }
        if constexpr (TRIM) {
            const float2 bt = *reinterpret_cast<const float2*>(lds_x + vrow * S + (half ? KH - 2 : KH - 4));
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[KH - 4], bt.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[KH - 3], bt.y, acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) terms[wave][r][lane] = __builtin_amdgcn_fmed3f(acc[r], 0.0f, hmv);
    }
    __syncthreads();
    add_terms();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        double v = double(acc_sum[i]);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        const int64_t p = cbase + acc_row(4 * wave + i, half);
        if (col == 0 && p < ga.n_cand) ga.part[int64_t(split) * ga.part_stride + p] = 2.0 * v;
    }
}

template <int KP, bool TRIM>
__global__ void __launch_bounds__(256) k_gains_f32(GainsArgs ga) {
    gains_f32_body<KP, TRIM>(ga, blockIdx.x);
}

// Batched: workgroups wg_pre[j] .. wg_pre[j+1] serve descriptor slot_inst[j]
// (all candidates, in the same geometry as a solo launch).
template <int KP, bool TRIM>
__global__ void __launch_bounds__(256)
kb_gains_f32(const InstDesc* __restrict__ descs, const int32_t* __restrict__ slot_inst,
             const int64_t* __restrict__ wg_pre, int32_t slots, int64_t first, int32_t t) {
    const int64_t bid = first + blockIdx.x;
    const int j = find_slot(wg_pre, slots, bid);
    const InstDesc c = descs[slot_inst[j]];
    if (c.t0 + t >= c.k || list_step(c, c.t0 + t)) return;
    gains_f32_body<KP, TRIM>(gains_args(c, nullptr, c.n_pad), bid - wg_pre[j]);
}

// Heads or list (lazy.h): the workgroups walk its (tile, chunk) pairs.
template <int KP, bool TRIM>
__global__ void __launch_bounds__(256) k_gains_f32_list(InstDesc c, int32_t part) {
    int64_t items;
    const GainsArgs ga = list_args(c, part, kGainsCandTile, &items);
    for (int64_t i = blockIdx.x; i < items; i += gridDim.x) gains_f32_body<KP, TRIM>(ga, i);
}

template <int KP, bool TRIM>
__global__ void __launch_bounds__(256, 2)
kb_gains_f32_list(const InstDesc* __restrict__ descs, const int32_t* __restrict__ slot_inst, int32_t slots, int32_t t,
                  int32_t part) {
    list_walk(descs, slot_inst, slots, t, part, kGainsCandTile,
              [](const GainsArgs& ga, int64_t pair) { gains_f32_body<KP, TRIM>(ga, pair); });
}

// How many of the 128-candidate tiles take the wide kernel; the rest of the
// candidates take the narrow one. Chosen to end first: rounds of 256 workgroups
// (a wide and a narrow workgroup of a chunk measured 2.7 and 1.2 us per 64
// points at d = 100) plus a launch each. Full rounds go to the wide kernel, a
// partial last one to the narrow: 50000 x 100, 2303 candidates: 288 wide
// workgroups 321 us a call, 256 wide and 128 narrow ones 243 us; 5000: 485 and
// 445 us. A step over all of 1000 x 100 in 4 chunks: 33 -> 24 us.
static int64_t wide_tiles(const GainsArgs& ga) {
    const int64_t tiles = (ga.n_cand + kGainsCandTile - 1) / kGainsCandTile;
    const double len = double(ga.chunk) / kGainsVTile;
    auto cost = [&](int64_t w) {
        const int64_t rest = ga.n_cand - w * kGainsCandTile;
        const int64_t nar = rest > 0 ? (rest + 31) / 32 : 0;
        return double((w * ga.v_splits + 255) / 256) * len + double((nar * ga.v_splits + 255) / 256) * 0.46 * len +
               (w > 0 && nar > 0 ? 2.0 : 0.0);
    };
    int64_t best = tiles;
    // candidates for the split: none, and whole rounds of wide workgroups
    const int64_t step = ga.v_splits < 256 ? 256 / ga.v_splits : 1;
    // (all rows: one of the kernels takes them all)
    for (int64_t w = 0; w < (ga.cand ? tiles : 1); w += step)
        if (cost(w) < cost(best)) best = w;
    return best;
}

template <int KP, bool TRIM>
static void launch_kpt(const GainsArgs& ga, hipStream_t s) {
    const int64_t w = wide_tiles(ga);
    const int64_t first = w * kGainsCandTile < ga.n_cand ? w * kGainsCandTile : ga.n_cand;
    GainsArgs part = ga;
    if (w > 0) {
        part.n_cand = first;
        hipLaunchKernelGGL((k_gains_f32<KP, TRIM>), dim3(unsigned(w * ga.v_splits)), dim3(256), 0, s, part);
    }
    if (first < ga.n_cand) {
        part.cand = ga.cand ? ga.cand + first : nullptr;
        part.n_cand = ga.n_cand - first;
        part.part = ga.part + first;
        const unsigned wgs = unsigned((part.n_cand + 31) / 32 * ga.v_splits);
        hipLaunchKernelGGL((k_gains_f32_narrow<KP, TRIM>), dim3(wgs), dim3(256), 0, s, part);
    }
}

template <int KP>
static void launch_kp(const ebc_dataset* ds, const GainsArgs& ga, hipStream_t s) {
    if (ds->d <= KP - 4)  // the rows' last 4 padded slots are empty
        launch_kpt<KP, true>(ga, s);
    else
        launch_kpt<KP, false>(ga, s);
}

#define EBC_F32_KPS(X) \
    X(8) X(16) X(24) X(32) X(40) X(48) X(56) X(64) X(72) X(80) X(88) X(96) X(104) X(112) X(120) X(128)

hipError_t launch_gains_f32(const ebc_dataset* ds, const GainsArgs& ga, hipStream_t s) {
    switch (ds->k_pad) {
#define EBC_KP(K) \
    case K: launch_kp<K>(ds, ga, s); break;
        EBC_F32_KPS(EBC_KP)
#undef EBC_KP
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gains_f32_list(const InstDesc& c, int32_t part, hipStream_t s) {
    const unsigned grid = list_grid(c, part, kGainsCandTile);
    switch (c.k_pad) {
#define EBC_KP(K)                                                                                              \
    case K:                                                                                                    \
        if (c.d <= K - 4)                                                                                      \
            hipLaunchKernelGGL((k_gains_f32_list<K, true>), dim3(grid), dim3(256), 0, s, c, part);        \
        else                                                                                                   \
            hipLaunchKernelGGL((k_gains_f32_list<K, false>), dim3(grid), dim3(256), 0, s, c, part);       \
        break;
        EBC_F32_KPS(EBC_KP)
#undef EBC_KP
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// trim: every instance of the bucket has d <= k_pad - 4 (the bucket key says so)
hipError_t launch_gains_f32_batched(int32_t k_pad, bool trim, const InstDesc* descs, const int32_t* slot_inst,
                                    const int64_t* wg_pre, int32_t slots, int64_t first, int64_t wgs, int32_t t,
                                    hipStream_t s) {
    switch (k_pad) {
#define EBC_KP(K)                                                                                             \
    case K:                                                                                                   \
        if (trim)                                                                                             \
            hipLaunchKernelGGL((kb_gains_f32<K, true>), dim3(unsigned(wgs)), dim3(256), 0, s, descs,    \
                               slot_inst, wg_pre, slots, first, t);                                                  \
        else                                                                                                  \
            hipLaunchKernelGGL((kb_gains_f32<K, false>), dim3(unsigned(wgs)), dim3(256), 0, s, descs,   \
                               slot_inst, wg_pre, slots, first, t);                                                  \
        break;
        EBC_F32_KPS(EBC_KP)
#undef EBC_KP
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gains_f32_list_batched(int32_t k_pad, bool trim, const InstDesc* descs, const int32_t* slot_inst,
                                         int32_t slots, int32_t t, int32_t part, hipStream_t s) {
    switch (k_pad) {
#define EBC_KP(K)                                                                                               \
    case K:                                                                                                     \
        if (trim)                                                                                               \
            hipLaunchKernelGGL((kb_gains_f32_list<K, true>), dim3(list_grid_batched(part)), dim3(256), 0, s, descs, slot_inst, \
                               slots, t, part);                                                                 \
        else                                                                                                    \
            hipLaunchKernelGGL((kb_gains_f32_list<K, false>), dim3(list_grid_batched(part)), dim3(256), 0, s, descs,          \
                               slot_inst, slots, t, part);                                                      \
        break;
        EBC_F32_KPS(EBC_KP)
#undef EBC_KP
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ebc
