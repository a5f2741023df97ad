// Marginal gains for long rows: padded row length above 128 values (the
// paper's case study summarises N = 1000 series of d = 3524 samples, Sec. 6).
//
// Same quantity and halving as the short-row kernels (Sec. 3 discrete
// derivative, Sec. 4.1 per-point decomposition):
//     G[c]/2 = sum_v med3( x_v . x_c + ha_v - hn_c, 0, hm_v )
// with the dataset's distance-dtype rows, their norms and (FP8) per-row E8M0
// scales. A whole row no longer fits in registers, so each wave walks the
// dimension: row pieces are loaded straight from global memory (the next
// batch while the current one is multiplied) and fed to the dtype's 32x32
// matrix instruction. MFMA tile: rows = 32 candidates, columns = 32 ground
// points; lane half h takes half h of every piece, for both operands.
//
// Work decomposition: a workgroup owns 128/KS candidates and one chunk of
// the ground set, walked in tiles of 64 points. KS = 1: each wave owns 32
// candidates of its own. KS = 4 (small ground sets, where candidate blocks
// alone leave most of the chip idle): the four waves share one block of 32
// candidates, each multiplies a quarter of the dimension, and the four
// partial dot products of a tile are added through LDS in wave order before
// the clamp. The clamp sums and the float64 column sums run in a fixed
// order, so results do not depend on the schedule.
#include "ebc_internal.h"
#include "wide_row.h"

namespace ebc {

namespace {

// PAIRS (KS = 4; greedy steps of data sets that may keep a pair matrix): the
// term is taken from the pair's own value e = x_v . x_c - hn_c - hn_v as
// med3(e + hm_v, 0, hm_v), and e is written to the matrix where there is one.
// Steps that read the matrix, and runs without one, so make the same terms.
template <int DT, int KS, bool PAIRS = false>
__device__ __forceinline__ void gains_wide_body(const GainsArgs& ga, int32_t k_pad, int64_t bid,
                                                float* __restrict__ pairs = nullptr) {
    using R = WideRow<DT>;
    using Piece = typename R::Piece;
    constexpr int B = R::kBatch;
    constexpr int CT = 32 * 4 / KS;             // candidates per workgroup
    constexpr int NR = KS > 1 ? 8 : 16;         // candidate rows whose clamps this lane sums
    constexpr bool kFp8 = DT == EBC_DT_FP8_E4M3;
    static_assert(KS == 1 || KS == 4, "K split of 1 or 4 waves");
    // KS = 4: partial dot products [wave][cb][r][lane], then column sums [wave][half][8]
    __shared__ float red[KS > 1 ? 4 * 2 * 16 * 64 : 1];
    __shared__ double tot[KS > 1 ? 4 * 2 * 8 : 1];

    const void* xq = ga.xq;
    const float* __restrict__ hn = ga.hn;
    const float* __restrict__ ha = ga.ha;
    const float* __restrict__ hm = ga.hm;
    const int* __restrict__ scale = ga.scale;
    const int32_t* __restrict__ cand = ga.cand;
    const int64_t n_cand = ga.n_cand, n_pad = ga.n_pad;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int col = lane & 31;
    const int half = lane >> 5;
    const int split = int(bid % ga.v_splits);
    const int64_t ctile = bid / ga.v_splits;
    const int64_t cbase = ctile * CT + (KS > 1 ? 0 : wave * 32);  // this wave's candidate block
    const int r0 = KS > 1 ? 8 * (wave & 1) : 0;                    // first of its NR rows

    // candidate row of this lane (A operand row `col`); rows outside
    // [0, n_pad) in a caller's list compute as zero rows and raise EBC_E_INDEX
    const int64_t cpos = cbase + col;
    int64_t crow = -1;
    if (cpos < n_cand) crow = cand ? int64_t(cand[cpos]) : cpos;
    if (crow >= n_pad || crow < -1 || (cpos < n_cand && crow < 0)) {
        atomicCAS(ga.err, 0, kDevErrIndex);
        crow = -1;
    }
    const bool alive = crow >= 0;
    const int64_t arow = alive ? crow : 0;
    const int sa = kFp8 ? (alive ? scale[crow] : 127) : 127;
    // -hn of the candidate rows this lane sums (result rows 8*(r/4) + 4*half + r%4)
    float nhn[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int r = r0 + i;
        const int64_t p = cbase + 8 * (r / 4) + 4 * half + (r % 4);
        float v = 0.0f;
        if (p < n_cand) {
            const int64_t row = cand ? int64_t(cand[p]) : p;
            if (row >= 0 && row < n_pad) v = hn[row];
        }
        nhn[i] = -v;
    }
    float acc_sum[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) acc_sum[i] = 0.0f;

    const int np = R::pieces(k_pad);
    const int kq = KS > 1 ? wave : 0;
    const int p0 = KS > 1 ? np * kq / 4 : 0;
    const int p1 = KS > 1 ? np * (kq + 1) / 4 : np;

    const int64_t v_begin = int64_t(split) * ga.chunk;
    int64_t v_end = v_begin + ga.chunk;
    if (v_end > n_pad) v_end = n_pad;

    for (int64_t v0 = v_begin; v0 < v_end; v0 += 64) {
        int64_t prow[2];
        int sb[2];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            prow[cb] = v0 + cb * 32 + col;
            sb[cb] = kFp8 ? scale[prow[cb]] : 127;
        }
        floatx16 acc[2];
        float hmv[2] = {0.0f, 0.0f};
        if constexpr (KS == 1) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const float hav = ha[prow[cb]];
                hmv[cb] = hm[prow[cb]];
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] = nhn[r % NR] + hav;
            }
        } else {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
        }
        // this wave's pieces [p0, p1), batches of B, the next batch in flight
        Piece a[B], b[2][B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const bool in = p0 + i < p1;
            a[i] = (in && alive) ? R::load(xq, arow, k_pad, p0 + i, half) : Piece{};
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) b[cb][i] = in ? R::load(xq, prow[cb], k_pad, p0 + i, half) : Piece{};
        }
        for (int p = p0; p < p1; p += B) {
            const bool more = p + B < p1;
            Piece an[B], bn[2][B];
            if (more) {
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const bool in = p + B + i < p1;
                    an[i] = (in && alive) ? R::load(xq, arow, k_pad, p + B + i, half) : Piece{};
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
                        bn[cb][i] = in ? R::load(xq, prow[cb], k_pad, p + B + i, half) : Piece{};
                }
            }
#pragma unroll
            for (int i = 0; i < B; ++i)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) acc[cb] = R::mma(a[i], b[cb][i], acc[cb], sa, sb[cb]);
            if (more) {
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    a[i] = an[i];
                    b[0][i] = bn[0][i];
                    b[1][i] = bn[1][i];
                }
            }
        }
        if constexpr (KS == 1) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_sum[r % NR] += __builtin_amdgcn_fmed3f(acc[cb][r], 0.0f, hmv[cb]);
        } else {
            // the four quarters of this tile's dot products, added in wave order
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[((wave * 2 + cb) * 16 + r) * 64 + lane] = acc[cb][r];
            __syncthreads();
            const int cbe = wave >> 1;  // the 32-point block whose clamps this wave takes
            const int64_t v = v0 + cbe * 32 + col;
            const float vt = PAIRS ? -hn[v] : ha[v], hmw = hm[v];
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int r = r0 + i;
                float t = nhn[i] + vt;
#pragma unroll
                for (int w = 0; w < 4; ++w) t += red[((w * 2 + cbe) * 16 + r) * 64 + lane];
                if constexpr (PAIRS) {
                    if (pairs) pairs[(cbase + acc_row(r, half)) * n_pad + v] = t;
                    t += hmw;
                }
                acc_sum[i] += __builtin_amdgcn_fmed3f(t, 0.0f, hmw);
            }
            __syncthreads();  // red is rewritten by the next tile
        }
    }

    // ---- float64 sums over the 32 columns (ground points) of each half ----
    double mine = 0.0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        double v = double(acc_sum[i]);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (col == i) mine = v;
    }
    double* __restrict__ part = ga.part + int64_t(split) * ga.part_stride;
    if constexpr (KS == 1) {
        if (col < 16) {
            const int r = col;
            const int64_t p = cbase + 8 * (r / 4) + 4 * half + (r % 4);
            if (p < n_cand) part[p] = 2.0 * mine;
        }
    } else {
        // waves w and w+2 hold the same rows for the two 32-point blocks
        if (col < 8) tot[(wave * 2 + half) * 8 + col] = mine;
        __syncthreads();
        if (wave < 2 && col < 8) {
            const double g = tot[(wave * 2 + half) * 8 + col] + tot[((wave + 2) * 2 + half) * 8 + col];
            const int r = r0 + col;
            const int64_t p = cbase + 8 * (r / 4) + 4 * half + (r % 4);
            if (p < n_cand) part[p] = 2.0 * g;
        }
    }
}

// Gains of one candidate from the pair matrix, by one wave: the terms, the
// float32 sums of a chunk and the float64 sums after it, all in the order of
// the kernel that multiplies the rows (lane l stands for the points l of a
// chunk's 64-point tiles), so that both give the same bits. 4 bytes a pair are
// what bounds it, with the sums' lane exchanges: 1000 points (4 MB, in the L2s)
// 92 -> 4 us a step against multiplying rows of 3524 values again (one float32
// sum a lane over all chunks: 3.2 us, but other sums than a run without a matrix).
__device__ __forceinline__ void gains_matrix_row(const InstDesc& c, int64_t row) {
    const int lane = threadIdx.x & 63;
    const float* __restrict__ e = c.b.pairs + row * c.n_pad;  // row: the same for the wave
    const float* __restrict__ hm = c.b.hm;
    float acc[16];  // chunks; a data set with a matrix has at most 16
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    for (int64_t o = 0; o < c.chunk; o += 64) {
        // no branch around a load: all of a row of tiles are in flight together
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t v = i * c.chunk + o;
            const bool in = v < c.n_pad;
            const int64_t at = in ? v : 0;
            const float pair = (e + at)[lane], hv = (hm + at)[lane];
            const float h = in ? hv : 0.0f;  // past the end: a term of 0
            acc[i] += __builtin_amdgcn_fmed3f(pair + h, 0.0f, h);
        }
    }
    const double half_sum = column_sums16(acc, lane & 31);  // chunk (lane & 31) / 2
    const double sum = 2.0 * (half_sum + __shfl_xor(half_sum, 32, 64));
    const uint64_t bits = __double_as_longlong(sum);
    double g = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {  // in chunk order; chunks past the last are 0
        const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(bits), 2 * i);
        const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(bits >> 32), 2 * i);
        g += __longlong_as_double((uint64_t(hi) << 32) | lo);
    }
    if (lane == 0) c.b.part[row] = g;
}

__global__ void __launch_bounds__(256) k_gains_matrix(InstDesc c) {
    gains_matrix_row(c, int64_t(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// Batched: row block on blockIdx.x, 4 candidates of it on blockIdx.y.
__global__ void __launch_bounds__(256)
kb_gains_matrix(const InstDesc* __restrict__ descs, const int64_t* __restrict__ row_pre, int32_t count, int32_t t) {
    const int i = find_slot(row_pre, count, blockIdx.x);
    const InstDesc c = descs[i];
    if (c.t0 + t >= c.k || !matrix_step(c, c.t0 + t)) return;
    const int64_t row = (int64_t(blockIdx.x) - row_pre[i]) * kBlock + blockIdx.y * 4 +
                        __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    gains_matrix_row(c, row);
}

template <int DT>
__global__ void __launch_bounds__(256) k_gains_wide_pairs(GainsArgs ga, int32_t k_pad, float* pairs) {
    gains_wide_body<DT, 4, true>(ga, k_pad, blockIdx.x, pairs);
}

template <int DT, int KS>
__global__ void __launch_bounds__(256) k_gains_wide(GainsArgs ga, int32_t k_pad) {
    gains_wide_body<DT, KS>(ga, k_pad, blockIdx.x);
}

// Batched: workgroups wg_pre[j] .. wg_pre[j+1] serve descriptor slot_inst[j]
// (all candidates, in the same geometry as a solo launch).
template <int DT, int KS>
__global__ void __launch_bounds__(256)
kb_gains_wide(const InstDesc* __restrict__ descs, const int32_t* __restrict__ slot_inst,
              const int64_t* __restrict__ wg_pre, int32_t slots, int64_t first, int32_t t) {
    const int64_t bid = first + blockIdx.x;
    const int j = find_slot(wg_pre, slots, bid);
    const InstDesc c = descs[slot_inst[j]];
    if (c.t0 + t >= c.k || matrix_step(c, c.t0 + t)) return;
    if constexpr (KS == 4) {
        if (pair_matrix(c.n_pad, c.k_pad)) {  // c.b.pairs is null without a matrix
            gains_wide_body<DT, KS, true>(gains_args(c, nullptr, c.n_pad), c.k_pad, bid - wg_pre[j],
                                          c.b.pairs);
            return;
        }
    }
    gains_wide_body<DT, KS>(gains_args(c, nullptr, c.n_pad), c.k_pad, bid - wg_pre[j]);
}

template <int DT, int KS>
void launch_w(const ebc_dataset* ds, const GainsArgs& ga, hipStream_t s) {
    const int64_t ct = 32 * 4 / KS;
    const int64_t tiles = (ga.n_cand + ct - 1) / ct;
    hipLaunchKernelGGL((k_gains_wide<DT, KS>), dim3(unsigned(tiles * ga.v_splits)), dim3(256), 0, s, ga, ds->k_pad);
}

template <int DT>
void launch_w_ks(int32_t ks, const ebc_dataset* ds, const GainsArgs& ga, hipStream_t s) {
    if (ks == 4)
        launch_w<DT, 4>(ds, ga, s);
    else
        launch_w<DT, 1>(ds, ga, s);
}

template <int DT>
void launch_wb(int32_t ks, const InstDesc* descs, const int32_t* slot_inst, const int64_t* wg_pre, int32_t slots,
               int64_t first, int64_t wgs, int32_t t, hipStream_t s) {
    const dim3 g = dim3(unsigned(wgs)), b = dim3(256);
    if (ks == 4)
        hipLaunchKernelGGL((kb_gains_wide<DT, 4>), g, b, 0, s, descs, slot_inst, wg_pre, slots, first, t);
    else
        hipLaunchKernelGGL((kb_gains_wide<DT, 1>), g, b, 0, s, descs, slot_inst, wg_pre, slots, first, t);
}

}  // namespace

hipError_t launch_gains_wide_pairs(const InstDesc& c, hipStream_t s) {
    const dim3 g = dim3(unsigned(c.n_pad / 32 * c.v_splits)), b = dim3(256);
    const GainsArgs ga = gains_args(c, nullptr, c.n_pad);
    switch (c.dt) {
        case EBC_DT_F32: hipLaunchKernelGGL(k_gains_wide_pairs<EBC_DT_F32>, g, b, 0, s, ga, c.k_pad, c.b.pairs); break;
        case EBC_DT_F16: hipLaunchKernelGGL(k_gains_wide_pairs<EBC_DT_F16>, g, b, 0, s, ga, c.k_pad, c.b.pairs); break;
        case EBC_DT_BF16:
            hipLaunchKernelGGL(k_gains_wide_pairs<EBC_DT_BF16>, g, b, 0, s, ga, c.k_pad, c.b.pairs);
            break;
        case EBC_DT_FP8_E4M3:
            hipLaunchKernelGGL(k_gains_wide_pairs<EBC_DT_FP8_E4M3>, g, b, 0, s, ga, c.k_pad, c.b.pairs);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gains_matrix(const InstDesc& c, hipStream_t s) {
    hipLaunchKernelGGL(k_gains_matrix, dim3(unsigned(c.n_pad / 4)), dim3(256), 0, s, c);
    return hipGetLastError();
}

hipError_t launch_gains_matrix_batched(const InstDesc* descs, const int64_t* row_pre, int32_t count,
                                       int64_t total_rows, int32_t t, hipStream_t s) {
    hipLaunchKernelGGL(kb_gains_matrix, dim3(unsigned(total_rows), kBlock / 4), dim3(256), 0, s, descs, row_pre, count, t);
    return hipGetLastError();
}

hipError_t launch_gains_wide(const ebc_dataset* ds, const GainsArgs& ga, hipStream_t s) {
    const int32_t ks = wide_ksplit(ds->n_pad);
    switch (ds->dt) {
        case EBC_DT_F32: launch_w_ks<EBC_DT_F32>(ks, ds, ga, s); break;
        case EBC_DT_F16: launch_w_ks<EBC_DT_F16>(ks, ds, ga, s); break;
        case EBC_DT_BF16: launch_w_ks<EBC_DT_BF16>(ks, ds, ga, s); break;
        case EBC_DT_FP8_E4M3: launch_w_ks<EBC_DT_FP8_E4M3>(ks, ds, ga, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gains_wide_batched(int32_t dt, int32_t ksplit, const InstDesc* descs, const int32_t* slot_inst,
                                     const int64_t* wg_pre, int32_t slots, int64_t first, int64_t wgs, int32_t t,
                                     hipStream_t s) {
    switch (dt) {
        case EBC_DT_F32: launch_wb<EBC_DT_F32>(ksplit, descs, slot_inst, wg_pre, slots, first, wgs, t, s); break;
        case EBC_DT_F16: launch_wb<EBC_DT_F16>(ksplit, descs, slot_inst, wg_pre, slots, first, wgs, t, s); break;
        case EBC_DT_BF16: launch_wb<EBC_DT_BF16>(ksplit, descs, slot_inst, wg_pre, slots, first, wgs, t, s); break;
        case EBC_DT_FP8_E4M3:
            launch_wb<EBC_DT_FP8_E4M3>(ksplit, descs, slot_inst, wg_pre, slots, first, wgs, t, s);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ebc
