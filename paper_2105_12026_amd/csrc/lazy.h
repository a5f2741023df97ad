// Greedy steps after the first: which candidates are scored again.
//
// The gain G[c] = sum_v max(0, m_v - d(v, c)) only shrinks as the minima m_v
// do, so the gain of an earlier step bounds the present one from above
// (Minoux's accelerated greedy; the discrete derivative of a submodular f,
// Sec. 3). Step 0 scores every candidate. A later step scores
//   1. the heads: in each of at most kListHeads stretches of the ground set,
//      the candidate of largest estimate G_old[c] * m_c / m_c(old) (what its
//      own minimum lost since it was scored; only an estimate, it decides
//      nothing but the order of the work);
//   2. the list: every candidate, heads among them, whose last gain reaches
//      the re-score window of the best head. Any other candidate's gain lies
//      below the window.
// The heads are scored again with the list, so that equal candidates get
// equal sums (the two launches cut the ground set differently).
// The window, its float64 re-score and the pick are those of a step that
// scores all candidates: the same candidates enter it. Over a run a candidate
// is scored 1.1 to 1.7 times instead of k times; the rest is launches. 100000 x
// 100 float32, k = 50: 730 -> 37 ms; 200000 x 64 bfloat16, k = 100: 418 -> 25
// ms; 10007 x 50 L1, k = 10: 2.68 -> 1.12 ms.
//
// Bound of the rounding: old and new sums may be cut into chunks differently,
// so a float32 lane sum of t non-negative terms may differ by t * 2^-24 of
// itself; the list takes everything within twice that of the window.
//
// A dataset keeps, in the last chunk of its partial sums (read by step 0
// before they are written): the list (int32 rows) and each row's m at the
// time it was scored (float32); the heads lie in bcnt (at most one per row
// block), which only steps that score every candidate use.
#pragma once

#include "ebc_internal.h"

namespace ebc {

// Heads per step: one candidate tile of the gains kernel.
constexpr int kListHeads = 256;
__host__ __device__ inline int list_heads_max(int dt) { return dt == EBC_DT_F32 ? 128 : kListHeads; }
// Row blocks of a stretch, and the number of stretches (= heads).
__host__ __device__ inline int list_stretch(const InstDesc& c) {
    const int h = list_heads_max(c.dt);
    return (c.nb + h - 1) / h;
}

__host__ __device__ inline int32_t* list_rows(const InstDesc& c) {
    return reinterpret_cast<int32_t*>(c.b.part + int64_t(c.v_splits - 1) * c.n_pad);
}
__host__ __device__ inline float* list_m(const InstDesc& c) {
    return reinterpret_cast<float*>(list_rows(c) + c.n_pad);
}

// Work split of a list of cnt candidates in tiles of ct rows. A few tiles (most
// steps): the ground set is cut finely enough for tiles * splits to fill the
// chip's workgroup slots once. Many tiles: chunks of about kListChunk points,
// long enough that loading a pair's candidates and adding up its sums do not
// count, and many enough that the last round of workgroups does not either.
// Whole units of points: 128 for float32 and L1, whose pairs are bound by their
// arithmetic (against 256: float32, d = 100, 8192 points, 76 -> 65 us a step;
// L1, d = 50, 10007 points, 1.27 -> 1.13 ms for 10 steps; the same above 20000);
// 256, the widest LDS tile, for the matrix-core types. As many splits as the
// partial sums have room for, padded to whole rounds over the 8 XCDs (a padded
// chunk is empty).
__host__ __device__ inline int32_t list_unit(const InstDesc& c) {
    return c.dt == EBC_DT_F32 || c.metric == 1 ? 128 : 256;
}
constexpr int kListSlots = 512;   // 2 workgroups of 4 waves on each of 256 CUs
constexpr int kListChunk = 1024;
struct ListGeom {
    int64_t chunk, stride;
    int32_t tiles, splits;
};
__host__ __device__ inline ListGeom list_geom(const InstDesc& c, int64_t cnt, int32_t ct) {
    ListGeom g;
    g.tiles = int32_t((cnt + ct - 1) / ct);
    g.stride = int64_t(g.tiles) * ct;
    const int32_t unit = list_unit(c);
    const int32_t units = int32_t(c.n_pad / unit);
    const int32_t tiles = g.tiles > 0 ? g.tiles : 1;
    const int32_t cap = int32_t((c.v_splits - 1) * (c.n_pad / ct) / tiles);
    int32_t s = kListSlots / tiles;
    const int32_t fine = units / (kListChunk / unit);
    s = s > fine ? s : fine;
    s = s < cap ? s : cap;
    s = s < units ? s : units;
    s = s < 1 ? 1 : s;
    const int32_t per = (units + s - 1) / s;
    s = (units + per - 1) / per;
    const int32_t up = (s + 7) & ~7;
    g.splits = s >= 8 && up <= cap ? up : s;
    g.chunk = int64_t(per) * unit;
    return g;
}
// Workgroups of a list launch over one instance: one per pair (the scheduler
// balances them, and those past the list's end return at once); a longer list
// than that is walked.
constexpr int kListGridMax = 16384;
inline unsigned list_grid(const InstDesc& c, int32_t part, int32_t ct) {
    const int64_t most = part ? c.n_pad : list_heads_max(c.dt);
    int64_t items = 0;
    // the pairs do not grow monotonically with the count; kListSlots + tiles
    // bounds them for few tiles, the geometry at the full count for many
    const ListGeom g = list_geom(c, most, ct);
    items = int64_t(g.tiles) * (g.splits > 8 ? g.splits : 8) + kListSlots + g.tiles;
    return unsigned(items < kListGridMax ? items : kListGridMax);
}
constexpr int kListGridBatch = 4096;  // batched: pairs of many instances, walked

// Rows and their number: part 0 the heads, part 1 the list. Until their sums
// are added the entries are slots of the grouped order where there is one.
__device__ inline int32_t* list_part(const InstDesc& c, int32_t part) { return part ? list_rows(c) : c.b.bcnt; }
__device__ inline int64_t list_count(const InstDesc& c, int32_t part) {
    return part ? c.b.state->list_len : c.b.state->list_heads;
}

// Gains-kernel arguments of a part of the list, and the number of (tile,
// chunk) pairs; candidate tiles of ct rows.
__device__ inline GainsArgs list_args(const InstDesc& c, int32_t part, int32_t ct, int64_t* items) {
    const int64_t cnt = list_count(c, part);
    const ListGeom g = list_geom(c, cnt, ct);
    GainsArgs a = gains_args(c, list_part(c, part), cnt);
    a.v_splits = g.splits;
    a.chunk = g.chunk;
    a.part_stride = g.stride;
    a.inv = nullptr;  // the entries are slots
    *items = int64_t(g.tiles) * g.splits;
    return a;
}

// Does step `step` of the instance score a list?
__host__ __device__ inline bool list_step(const InstDesc& c, int32_t step) { return c.lazy != 0 && step > 0; }

// Batched list launches: the workgroups walk the (tile, chunk) pairs of every
// instance of a bucket that is at a list step. The pairs of 64 instances at a
// time are counted on the device (the counts are not known to the host; each
// wave does it for itself) and numbered in instance order; workgroup b takes
// pairs b, b + gridDim.x, ... f(gains arguments, pair) runs the kernel body.
template <class F>
__device__ __forceinline__ void list_walk(const InstDesc* __restrict__ descs, const int32_t* __restrict__ slot_inst,
                                          int32_t slots, int32_t t, int32_t part, int32_t ct, F f) {
    const int lane = threadIdx.x & 63;
    int32_t next = blockIdx.x, before = 0;
    for (int32_t s0 = 0; s0 < slots; s0 += 64) {
        int32_t upto = 0;  // pairs of instances s0 .. s0 + lane
        if (s0 + lane < slots) {
            const InstDesc& c = descs[slot_inst[s0 + lane]];
            if (list_step(c, c.t0 + t) && c.t0 + t < c.k) {
                const ListGeom g = list_geom(c, list_count(c, part), ct);
                upto = g.tiles * g.splits;
            }
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t add = __shfl_up(upto, off, 64);
            if (lane >= off) upto += add;
        }
        const int32_t total = __builtin_amdgcn_readlane(upto, 63);
        while (next < before + total) {
            // the same for the whole workgroup: kept scalar
            const int32_t at = next - before;
            const int32_t j = __popcll(__builtin_amdgcn_ballot_w64(upto <= at));
            const int32_t pair = j > 0 ? at - __builtin_amdgcn_readlane(upto, j - 1) : at;
            const InstDesc c = descs[slot_inst[s0 + j]];
            int64_t items;
            f(list_args(c, part, ct, &items), int64_t(pair));
            __syncthreads();  // the body's LDS is free again
            next += gridDim.x;
        }
        before += total;
    }
}

// Candidate tile of the list kernels.
__host__ __device__ inline int32_t list_tile(int32_t dt, int32_t metric) {
    return metric == 1 ? 64 : (dt == EBC_DT_F32 ? kGainsCandTile : 256);
}

}  // namespace ebc
