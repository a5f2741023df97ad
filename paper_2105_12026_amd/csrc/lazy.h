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
// scores all candidates: the same candidates enter it.
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

// Work split of a list of cnt candidates in tiles of ct: enough chunks that
// tiles * splits fills the chip several times (kListItems), chunks of whole
// 256-point units, and partial sums that fit the buffer. Lists are short
// against n (a few tiles) in most steps, so the ground set is cut much finer
// than for a launch over all candidates.
constexpr int kListItems = 4096;   // (tile, chunk) pairs wanted
constexpr int kListUnit = 256;     // points
constexpr int kListGrid = 1024;    // workgroups of a list launch; each walks its share of the pairs
struct ListGeom {
    int64_t tiles, chunk, stride;
    int32_t splits;
};
__host__ __device__ inline ListGeom list_geom(const InstDesc& c, int64_t cnt, int32_t ct) {
    ListGeom g;
    g.tiles = (cnt + ct - 1) / ct;
    g.stride = g.tiles * ct;
    const int64_t units = c.n_pad / kListUnit;
    int64_t s = g.tiles > 0 ? kListItems / g.tiles : 1;
    const int64_t cap = g.stride > 0 ? int64_t(c.v_splits - 1) * c.n_pad / g.stride : 1;
    s = s < units ? s : units;
    s = s < cap ? s : cap;
    s = s < 1 ? 1 : s;
    if (s >= 8) s &= ~int64_t(7);  // whole rounds over the XCDs
    g.chunk = (units + s - 1) / s * kListUnit;
    g.splits = int32_t(s);
    return g;
}

// Rows and their number: part 0 the heads, part 1 the list.
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
    *items = g.tiles * g.splits;
    return a;
}

// Candidate tile of the list kernels.
__host__ __device__ inline int32_t list_tile(int32_t dt, int32_t metric) {
    return metric == 1 ? 64 : (dt == EBC_DT_F32 ? kGainsCandTile : 256);
}

}  // namespace ebc
