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
//   3. the recount: where more candidates come near the window of the list's
//      best than are re-scored (kWindowMax), which of them are kept depends on
//      the last bit of every sum. The near ones are scored once more with the
//      chunks of a step that scores all candidates: the same sums, bit for bit,
//      hence the same window. A list of more than half of the points is cut
//      that way from the start. Otherwise (nearly always) the recount's launch
//      finds nothing to do (2.5 us in a solo step, 4.6 in a batch).
// The window, its float64 re-score and the pick are those of a step that
// scores all candidates: the same candidates enter it. What bounds a run: its
// first list still holds 0.93 to 1.0 of all candidates, the later ones add up to
// 0.4 to 2 times their number, and the rest is launches. 100000 x 100 float32,
// k = 50: lists of 1.8 n in all, 729 -> 37 ms; 200000 x 64 bfloat16, k = 100:
// 2.7 n, 429 -> 25 ms; 30011 x 33 FP8, k = 20: 2.1 n, 3.27 -> 1.9 ms; 10007 x 50
// L1, k = 10: 1.3 n, 2.70 -> 1.11 ms.
//
// Bound of the rounding: a float32 lane sum of t non-negative terms is within
// t * 2^-24 of itself (relative), and a lane of a chunk of p points adds p / 32.
// Between a candidate's old sum and the window of a step that scores all lie
// four such sums: the best head's, the one that step would have for it, the
// candidate's old one and the one that step would have. Between the list's sums
// and that step's there are as many. The list, and the recount, take everything
// that far below the window (list_slack).
//
// A dataset keeps its list (int32 rows) and each row's m at the time it was
// scored (float32) in wstage, and its heads in bcnt (at most one per row
// block): only steps that score every candidate use these.
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

__host__ __device__ inline int32_t* list_rows(const InstDesc& c) { return reinterpret_cast<int32_t*>(c.b.wstage); }
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
// Does a list of cnt candidates take the chunks of a step that scores all?
__host__ __device__ inline bool list_full_cut(const InstDesc& c, int64_t cnt) { return 2 * cnt > c.n_pad; }
__host__ __device__ inline ListGeom list_geom(const InstDesc& c, int64_t cnt, int32_t ct, bool full_cut) {
    ListGeom g;
    g.tiles = int32_t((cnt + ct - 1) / ct);
    g.stride = int64_t(g.tiles) * ct;
    if (full_cut) {
        g.splits = c.v_splits;
        g.chunk = c.chunk;
        return g;
    }
    const int32_t unit = list_unit(c);
    const int32_t units = int32_t(c.n_pad / unit);
    const int32_t tiles = g.tiles > 0 ? g.tiles : 1;
    const int32_t cap = int32_t(c.v_splits * (c.n_pad / ct) / tiles);
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
// Half-width of what may lie between a sum and the window of a step that scores
// all, for a best gain g: four float32 sums of the longest chunk any of them has
// (16 terms more for the float64 sums behind them).
__device__ inline double list_slack(const InstDesc& c, double g) {
    const int32_t unit = list_unit(c), units = int32_t(c.n_pad / unit);
    int32_t s = units / (kListChunk / unit);  // fewest chunks of list_geom
    s = s < c.v_splits ? s : c.v_splits;
    s = s < 1 ? 1 : s;
    const int64_t longest = int64_t((units + s - 1) / s) * unit;
    const int64_t p = c.chunk > longest ? c.chunk : longest;
    return 4.0 * (double(p) / 32.0 + 16.0) * 0x1p-24 * fabs(g);
}
// Workgroups of a list launch over one instance: one per pair (the scheduler
// balances them, and those past the list's end return at once); a longer list
// than that is walked.
constexpr int kListGridMax = 16384;
inline unsigned list_grid(const InstDesc& c, int32_t part, int32_t ct) {
    if (part == 2) return kListSlots;  // nearly always empty
    int64_t items = int64_t(c.v_splits) * (c.n_pad / ct);  // what the partial sums have room for
    if (part == 0) {
        const ListGeom g = list_geom(c, list_heads_max(c.dt), ct, false);
        items = int64_t(g.tiles) * (g.splits > 8 ? g.splits : 8) + kListSlots + g.tiles;
    }
    return unsigned(items < kListGridMax ? items : kListGridMax);
}
// Batched: pairs of many instances, walked.
inline unsigned list_grid_batched(int32_t part) { return part == 2 ? kListSlots : 4096; }

// Rows and their number: part 0 the heads, part 1 the list, part 2 the recount.
// Until their sums are added the entries are slots of the grouped order where
// there is one.
__device__ inline int32_t* list_part(const InstDesc& c, int32_t part) { return part ? list_rows(c) : c.b.bcnt; }
__device__ inline int64_t list_count(const InstDesc& c, int32_t part) {
    const DevState* st = c.b.state;
    return part == 0 ? st->list_heads : (part == 1 ? st->list_len : st->list_exact);
}
__device__ inline ListGeom list_part_geom(const InstDesc& c, int32_t part, int64_t cnt, int32_t ct) {
    return list_geom(c, cnt, ct, part == 2 || (part == 1 && list_full_cut(c, cnt)));
}

// Gains-kernel arguments of a part of the list, and the number of (tile,
// chunk) pairs; candidate tiles of ct rows.
__device__ inline GainsArgs list_args(const InstDesc& c, int32_t part, int32_t ct, int64_t* items) {
    const int64_t cnt = list_count(c, part);
    const ListGeom g = list_part_geom(c, part, cnt, ct);
    GainsArgs a = gains_args(c, list_part(c, part), cnt);
    a.v_splits = g.splits;
    a.chunk = g.chunk;
    a.part_stride = g.stride;
    a.inv = nullptr;  // the entries are slots
    *items = int64_t(g.tiles) * g.splits;
    return a;
}

// Does step `step` of the instance score a list?
__host__ __device__ inline bool list_step(const InstDesc& c, int32_t step) { return c.lazy == 1 && step > 0; }

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
                const ListGeom g = list_part_geom(c, part, list_count(c, part), ct);
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
