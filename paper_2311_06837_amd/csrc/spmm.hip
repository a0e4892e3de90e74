// Masked CSR aggregation, forward and backward (paper section 2.1: h_N(v) = AGGREGATE of the
// neighbours' hidden vectors, a scaled sum; section 6: only the rows the layer's mask keeps).
//
//     Y[v, :] = out_scale[v] * sum_{u in row(v), keep(u)} nbr_scale[u] * X[u, :]      v in rows
//
// Forward: (out_scale, nbr_scale) = (row_scale, col_scale), no filter.  Backward runs the
// same gather over the transposed graph with the scale roles swapped and keep(u) =
// "u was an active row of the forward call" (a dist probe), so no floating-point atomics
// are needed and results are bit-reproducible.
//
// Mapping to CDNA4.  The work is a gather of whole feature rows: HBM/L2 bound, one FMA per
// loaded element, so no MFMA.  A group of LPR lanes (16, 32 or 64) owns one output row and
// spans its feature columns with 16-byte loads, so every neighbour costs one fully coalesced
// row read; 64/LPR rows share a wavefront when rows are narrow.  Neighbour ids are fetched one
// tile ahead, coalesced, filtered, compacted and staged in an LDS tile private to the
// wavefront; the inner loop then reads the tile by broadcast and keeps U x NCH independent
// 16-byte loads in flight per lane.  Groups claim rows dynamically inside a workgroup's chunk.  Rows of more than kHubTiles tiles
// (power-law hubs) are split over all wavefronts of the workgroup and the partial sums are
// reduced through LDS in a fixed order, inside the same launch.
#include "common.h"
#include "scan.h"
#include "spmm_fours.h"
#include "spmm_split.h"
#include <algorithm>
#include <mutex>

namespace gnnhot {

// Independent row loads in flight per lane (a round), and workgroups per CU, when a lane owns one 16-byte chunk of
// the row.  A round must divide the tile (16, 32 or 64 entries): 6, 10 or 12 loads were all slower than 8.  Measured
// as the step time of the 8-level bf16 workload / the sampled-partition workload (ms; rows of 256 and 512 bytes, 10
// to 20 neighbours, partitions numbered by (distance, id)): rounds of 16 at 4 workgroups per CU 17.5 / 23.7, 8 at 6
// 17.5 / 24.2, 8 at 5 or 4 16.5 / 23.4, 4 at 8 19.5 / 24.8 - slots of a round past the end of a tile are wasted issue
// slots of the vector cache, but eight workgroups of short rounds lose more to the caches than they gain.  (On the
// same graph numbered by global id the order is the reverse, 4 at 8 being 18 % faster than 16 at 4: the setting
// follows the numbering the extraction produces.)  Rows of 1 KB (64 lanes per row): 8 at 5 (8 at 6: +2 %).
#ifndef GNN_SPMM_U_NARROW
#define GNN_SPMM_U_NARROW 8
#endif
#ifndef GNN_SPMM_U_WIDE
#define GNN_SPMM_U_WIDE 8
#endif
#ifndef GNN_SPMM_MINB_NARROW
#define GNN_SPMM_MINB_NARROW 5
#endif
#ifndef GNN_SPMM_MINB_WIDE
#define GNN_SPMM_MINB_WIDE 5
#endif

// Rows of the list per lane group in one workgroup, and the length (in tiles of LPR entries) from which a row is
// split over all groups of the workgroup.  A group walks a row alone, tile by tile; with power-law rows one long row
// keeps its group - and the workgroup's registers and LDS - busy long after the other groups have run out of rows
// (simulated on the 8-level workload's graph: the groups of a 64-row workgroup are busy 35 % of its lifetime when only
// rows above 1024 entries are split).  Small chunks let the hardware's workgroup dispatch do the balancing, and a low
// split length bounds what one group can be left with.  Measured as the step time of the 8-level / the
// sampled-partition workload (ms): 4 rows per group and rows split above 1024 entries 16.5 / 23.4; 4 and 16 tiles
// 15.9 / 22.6; 2 and 16 tiles 15.2 / 21.4; 2 and 4 tiles 14.1 / 20.7; 3 and 4..12 tiles 14.0 / 21.4; 1 row per group
// 17.4 / 22.5; 8 or 16 rows per group 21.6 .. 31 / 24.4 .. 28.
#ifndef GNN_SPMM_RPG
#define GNN_SPMM_RPG 2
#endif
constexpr int kRowsPerGroup = GNN_SPMM_RPG;   // largest chunk: this many rows of the list per group
#ifndef GNN_SPMM_HUB_TILES
#define GNN_SPMM_HUB_TILES 4
#endif
constexpr int kHubTiles = GNN_SPMM_HUB_TILES;   // rows of more tiles (of LPR entries) than this are split over the whole workgroup
constexpr int kMaxChunk = 256;                  // rows of the list per workgroup, at most (one descriptor per thread)

// Column-blocked route (dense graphs, gathered matrix far larger than an L2).  The neighbour-id
// range [0, n_cols) is cut into 8 * passes blocks of about as many entries; in pass p workgroup i gathers, for its
// rows, only the neighbours inside block 8p + (i mod 8).  Workgroups are dealt round-robin to the 8
// compute dies, so every die's L2 sees one eighth of the matrix - and with the feature axis walked
// in slabs of 128 bytes per row (row lists, short calls: 256; grid.y, the slow grid axis) that eighth fits: the gathers then
// run at L2 rather than at fabric speed.  Each die leaves a plane of float
// partial sums; a second kernel adds the planes in block order and applies the output scale.
constexpr int kDies = 8;
#ifndef GNN_SPMM_DIE_BYTES
#define GNN_SPMM_DIE_BYTES (8ll << 20)      // target size of one die's share of one slab
#endif
#ifndef GNN_SPMM_BLOCKED_MIN_SLAB
#define GNN_SPMM_BLOCKED_MIN_SLAB (16ll << 20)   // below this slab size the plain route is already cache-resident
#endif
constexpr int kSlabBytes = 256;

struct SpmmArgs {
    const int32_t* row_ptr;
    const int32_t* col_idx;
    const int32_t* rows;      // nullable
    int32_t n_active;
    const void* X;
    int64_t ldx;
    void* Y;
    int64_t ldy;
    int32_t F;
    const float* out_scale;   // nullable, indexed by output row
    const float* nbr_scale;   // nullable, indexed by neighbour
    const int32_t* dist;      // nullable filter: keep u iff 0 <= dist[u] <= max_dist
    int32_t max_dist;
    const uint32_t* edge_keep;  // nullable filter: keep the entry at position p iff bit p is set (layer-wise sampling mask)
    int32_t cut_id;           // -1, or (rows sorted by column): every row ends at its first entry >= cut_id
    int32_t id_limit;         // -1, or (rows in any order): the filter drops the entries >= id_limit
    int32_t accumulate;
    const void* relu_h;       // nullable: the stored result is zeroed where this matrix (same rows and columns as Y) is <= 0
    int64_t ldh;
    int32_t rows_per_group;   // 1..kRowsPerGroup: rows of the list per LPR-lane group in one workgroup
    uint32_t x_row_bytes;     // > 0: X holds fewer than 2^24 rows and less than 4 GB, a row starts every x_row_bytes bytes - the
                              // row kernel then forms a gather address with one 24-bit multiply-add instead of a 64-bit product
    // column-blocked route only
    const int32_t* seg;       // [n_active][n_blocks + 1] cut points of every listed row: block j = [seg[j], seg[j+1])
    const int32_t* seg_end;   // nullable, [n_active][n_blocks]: block j ends here instead (filtered, compacted copy of the ids)
    const float* edge_w;      // with a neighbour scale: the factor of every entry of col_idx, at the same position
    int32_t n_blocks;
    int32_t block0;           // first column block of this pass
    // split route only (spmm_split.h)
    const int32_t* split_on;       // 1: the rows' other entries lie in split_cold, their hot ones are summed in split_plane
    const int32_t* split_cold;
    const SplitRow* split_rows;
    const SplitChunk* split_chunks;
    const float* split_plane;      // a row of split_ld floats per part
    int64_t split_ld;
};

// ---- element access: VE elements per lane-chunk ------------------------------------------
template <int DT, int VE>
struct Elem;

template <>
struct Elem<GNN_F32, 4> {
    static constexpr int VE = 4;
    using Raw = uint4;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return *(const uint4*)((const float*)p + off); }
    static __device__ __forceinline__ void fma(float (&acc)[4], float w, const Raw& r) {
        acc[0] = fmaf(w, __uint_as_float(r.x), acc[0]);
        acc[1] = fmaf(w, __uint_as_float(r.y), acc[1]);
        acc[2] = fmaf(w, __uint_as_float(r.z), acc[2]);
        acc[3] = fmaf(w, __uint_as_float(r.w), acc[3]);
    }
    // h (nullable): activation matrix of the same layout position hoff; what is stored is zeroed where h <= 0.
    // h == p stands for "the value being stored itself": the store applies a ReLU.
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[4], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        float* q = (float*)p + off;
        const float* hq = (const float*)h + hoff;
        if (n_valid >= 4) {
            float4 o = make_float4(v[0], v[1], v[2], v[3]);
            if (accumulate) {
                float4 old = *(const float4*)q;
                o.x += old.x; o.y += old.y; o.z += old.z; o.w += old.w;
            }
            if (h) {
                const float4 m = h == p ? o : *(const float4*)hq;
                o.x = m.x > 0.f ? o.x : 0.f; o.y = m.y > 0.f ? o.y : 0.f; o.z = m.z > 0.f ? o.z : 0.f; o.w = m.w > 0.f ? o.w : 0.f;
            }
            *(float4*)q = o;
        } else {
            for (int e = 0; e < n_valid; ++e) {
                const float t = accumulate ? q[e] + v[e] : v[e];
                q[e] = (h == nullptr || (h == p ? t : hq[e]) > 0.f) ? t : 0.f;
            }
        }
    }
};

template <>
struct Elem<GNN_F32, 1> {
    static constexpr int VE = 1;
    using Raw = float;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return ((const float*)p)[off]; }
    static __device__ __forceinline__ float to_float(Raw r) { return r; }
    static __device__ __forceinline__ void fma(float (&acc)[1], float w, const Raw& r) { acc[0] = fmaf(w, r, acc[0]); }
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[1], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        float* q = (float*)p + off;
        if (n_valid >= 1) {
            const float t = accumulate ? q[0] + v[0] : v[0];
            q[0] = (h == nullptr || (h == p ? t : ((const float*)h)[hoff]) > 0.f) ? t : 0.f;
        }
    }
};

template <>
struct Elem<GNN_BF16, 8> {
    static constexpr int VE = 8;
    using Raw = uint4;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return *(const uint4*)((const uint16_t*)p + off); }
    static __device__ __forceinline__ void fma(float (&acc)[8], float w, const Raw& r) {
        acc[0] = fmaf(w, bf16lo(r.x), acc[0]); acc[1] = fmaf(w, bf16hi(r.x), acc[1]);
        acc[2] = fmaf(w, bf16lo(r.y), acc[2]); acc[3] = fmaf(w, bf16hi(r.y), acc[3]);
        acc[4] = fmaf(w, bf16lo(r.z), acc[4]); acc[5] = fmaf(w, bf16hi(r.z), acc[5]);
        acc[6] = fmaf(w, bf16lo(r.w), acc[6]); acc[7] = fmaf(w, bf16hi(r.w), acc[7]);
    }
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[8], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        uint16_t* q = (uint16_t*)p + off;
        const uint16_t* hq = (const uint16_t*)h + hoff;
        if (n_valid >= 8) {
            float t[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = v[e];
            if (accumulate) {
                uint4 old = *(const uint4*)q;
                t[0] += bf16lo(old.x); t[1] += bf16hi(old.x); t[2] += bf16lo(old.y); t[3] += bf16hi(old.y);
                t[4] += bf16lo(old.z); t[5] += bf16hi(old.z); t[6] += bf16lo(old.w); t[7] += bf16hi(old.w);
            }
            if (h == p) {
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = t[e] > 0.f ? t[e] : 0.f;
            } else if (h) {
                const uint4 m = *(const uint4*)hq;
                t[0] = bf16lo(m.x) > 0.f ? t[0] : 0.f; t[1] = bf16hi(m.x) > 0.f ? t[1] : 0.f;
                t[2] = bf16lo(m.y) > 0.f ? t[2] : 0.f; t[3] = bf16hi(m.y) > 0.f ? t[3] : 0.f;
                t[4] = bf16lo(m.z) > 0.f ? t[4] : 0.f; t[5] = bf16hi(m.z) > 0.f ? t[5] : 0.f;
                t[6] = bf16lo(m.w) > 0.f ? t[6] : 0.f; t[7] = bf16hi(m.w) > 0.f ? t[7] : 0.f;
            }
            uint4 o;
            o.x = pack_bf16(t[0], t[1]); o.y = pack_bf16(t[2], t[3]);
            o.z = pack_bf16(t[4], t[5]); o.w = pack_bf16(t[6], t[7]);
            *(uint4*)q = o;
        } else {
            for (int e = 0; e < n_valid; ++e) {
                const float t = accumulate ? bf16_to_f32(q[e]) + v[e] : v[e];
                q[e] = f32_to_bf16((h == nullptr || (h == p ? t : bf16_to_f32(hq[e])) > 0.f) ? t : 0.f);
            }
        }
    }
};

// two bf16 per lane: narrow rows (up to 32 columns) spread over 16 lanes, so that a tile still holds 16 neighbours
template <>
struct Elem<GNN_BF16, 2> {
    static constexpr int VE = 2;
    using Raw = uint32_t;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return *(const uint32_t*)((const uint16_t*)p + off); }
    static __device__ __forceinline__ void fma(float (&acc)[2], float w, const Raw& r) {
        acc[0] = fmaf(w, bf16lo(r), acc[0]);
        acc[1] = fmaf(w, bf16hi(r), acc[1]);
    }
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[2], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        uint16_t* q = (uint16_t*)p + off;
        const uint16_t* hq = (const uint16_t*)h + hoff;
        for (int e = 0; e < 2; ++e) {
            if (e >= n_valid) break;
            const float t = accumulate ? bf16_to_f32(q[e]) + v[e] : v[e];
            q[e] = f32_to_bf16((h == nullptr || (h == p ? t : bf16_to_f32(hq[e])) > 0.f) ? t : 0.f);
        }
    }
};

// four bf16 per lane (33 to 64 columns over 16 lanes)
template <>
struct Elem<GNN_BF16, 4> {
    static constexpr int VE = 4;
    using Raw = uint2;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return *(const uint2*)((const uint16_t*)p + off); }
    static __device__ __forceinline__ void fma(float (&acc)[4], float w, const Raw& r) {
        acc[0] = fmaf(w, bf16lo(r.x), acc[0]);
        acc[1] = fmaf(w, bf16hi(r.x), acc[1]);
        acc[2] = fmaf(w, bf16lo(r.y), acc[2]);
        acc[3] = fmaf(w, bf16hi(r.y), acc[3]);
    }
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[4], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        uint16_t* q = (uint16_t*)p + off;
        const uint16_t* hq = (const uint16_t*)h + hoff;
        for (int e = 0; e < 4; ++e) {
            if (e >= n_valid) break;
            const float t = accumulate ? bf16_to_f32(q[e]) + v[e] : v[e];
            q[e] = f32_to_bf16((h == nullptr || (h == p ? t : bf16_to_f32(hq[e])) > 0.f) ? t : 0.f);
        }
    }
};

// two floats per lane (17 to 32 columns over 16 lanes)
template <>
struct Elem<GNN_F32, 2> {
    static constexpr int VE = 2;
    using Raw = float2;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return *(const float2*)((const float*)p + off); }
    static __device__ __forceinline__ void fma(float (&acc)[2], float w, const Raw& r) {
        acc[0] = fmaf(w, r.x, acc[0]);
        acc[1] = fmaf(w, r.y, acc[1]);
    }
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[2], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        float* q = (float*)p + off;
        const float* hq = (const float*)h + hoff;
        for (int e = 0; e < 2; ++e) {
            if (e >= n_valid) break;
            const float t = accumulate ? q[e] + v[e] : v[e];
            q[e] = (h == nullptr || (h == p ? t : hq[e]) > 0.f) ? t : 0.f;
        }
    }
};

template <>
struct Elem<GNN_BF16, 1> {
    static constexpr int VE = 1;
    using Raw = uint16_t;
    static __device__ __forceinline__ Raw load(const void* p, int64_t off) { return ((const uint16_t*)p)[off]; }
    static __device__ __forceinline__ float to_float(Raw r) { return bf16_to_f32(r); }
    static __device__ __forceinline__ void fma(float (&acc)[1], float w, const Raw& r) { acc[0] = fmaf(w, bf16_to_f32(r), acc[0]); }
    static __device__ __forceinline__ void store(void* p, int64_t off, const float (&v)[1], int n_valid, bool accumulate,
                                                 const void* h = nullptr, int64_t hoff = 0) {
        uint16_t* q = (uint16_t*)p + off;
        if (n_valid >= 1) {
            const float t = accumulate ? bf16_to_f32(q[0]) + v[0] : v[0];
            q[0] = f32_to_bf16((h == nullptr || (h == p ? t : bf16_to_f32(((const uint16_t*)h)[hoff])) > 0.f) ? t : 0.f);
        }
    }
};

// Float partial sums of the column-blocked route: VE consecutive floats at p[off] (16-byte aligned when VE >= 4).
template <int VE>
__device__ __forceinline__ void store_part(float* p, int64_t off, const float (&v)[VE], int n_valid, bool accumulate) {
    if (VE >= 4 && n_valid == VE) {
#pragma unroll
        for (int q = 0; q < VE / 4; ++q) {
            float4* dst = (float4*)(p + off) + q;
            float4 o = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
            if (accumulate) {
                const float4 old = *dst;
                o.x += old.x; o.y += old.y; o.z += old.z; o.w += old.w;
            }
            *dst = o;
        }
    } else {
#pragma unroll
        for (int k = 0; k < VE; ++k)
            if (k < n_valid) p[off + k] = accumulate ? p[off + k] + v[k] : v[k];
    }
}

// The value the filter tests for the entry at position p with neighbour u: dist[u] (0 without a dist filter),
// or -1 if the layer's edge mask drops the entry.
__device__ __forceinline__ int32_t filter_probe(const SpmmArgs& a, int32_t u, int32_t p) {
    int32_t d = a.dist ? a.dist[u] : 0;
    if (a.edge_keep && !((a.edge_keep[p >> 5] >> (p & 31)) & 1u)) d = -1;
    if (a.id_limit >= 0 && u >= a.id_limit) d = -1;
    return d;
}

// First position in [lo, hi) of a row sorted by column whose entry is >= bound (hi if none).
__device__ __forceinline__ int32_t row_lower_bound(const int32_t* __restrict__ col_idx, int32_t lo, int32_t hi, int64_t bound) {
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if ((int64_t)col_idx[mid] < bound) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Filter (backward: "was u an active row of the forward call"), compact and stage one tile of
// neighbour ids (already in registers: `u` and its `d` = dist[u], valid where `in_row`) into the group's LDS slots.
// Returns how many were kept.
template <int LPR, bool FILTER>
__device__ __forceinline__ int commit_tile(const SpmmArgs& a, bool in_row, int32_t u, int32_t d, int n_in_row, int sub, int sl,
                                           int32_t* s_idx) {
    if (!FILTER) {
        if (in_row) s_idx[sub * LPR + sl] = u;
        return n_in_row;
    }
    const bool keep = in_row && d >= 0 && d <= a.max_dist;  // d = dist[u], fetched by the caller
    const uint64_t group_mask = LPR == 64 ? ~0ull : (((1ull << (LPR & 63)) - 1ull) << (sub * LPR));
    const uint64_t kept = __ballot(keep) & group_mask;
    const uint64_t below = kept & ((1ull << (sub * LPR + sl)) - 1ull);
    if (keep) s_idx[sub * LPR + __popcll(below)] = u;
    return __popcll(kept);
}

// acc += sum over the staged tile.  `cnt` (this group's entries) may differ between the groups
// of a wave; `cnt_max` is uniform over the wave.  Each round issues U x NCH independent row loads
// (plus U broadcast loads of the neighbour scale) before the first multiply-add.  The issue part has
// no branch that depends on a lane: a slot past the group's count repeats the group's last entry (a
// cache hit) and a lane past the row's width reads the row's start; only the multiply-adds are
// predicated.  (With a branch around every load the compiler put a wait for the id's LDS read and
// two mask updates between any two loads: sixteen loads took longer to issue than to arrive.)
template <typename E, int LPR, int NCH, int U>
__device__ __forceinline__ void consume_tile(const SpmmArgs& a, int cnt, int cnt_max, int sub, const int64_t (&col_off)[NCH],
                                             const bool (&col_ok)[NCH], const int32_t* s_idx, float (&acc)[NCH][E::VE]) {
    int64_t col_ld[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) col_ld[c] = col_ok[c] ? col_off[c] : 0;
    uint32_t col_ld_bytes[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) col_ld_bytes[c] = (uint32_t)col_ld[c] * (uint32_t)(sizeof(typename E::Raw) / E::VE);
    const int last = cnt > 0 ? cnt - 1 : 0;
    for (int k = 0; k < cnt_max; k += U) {
        typename E::Raw x[U][NCH];
        float w[U];
        int32_t u[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int32_t staged = s_idx[sub * LPR + (k + j < cnt ? k + j : last)];
            u[j] = cnt > 0 ? staged : 0;   // nothing staged for this group: the slot may hold anything, row 0 always exists
        }
        if (a.nbr_scale) {   // uniform
#pragma unroll
            for (int j = 0; j < U; ++j) w[j] = a.nbr_scale[u[j]];
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) w[j] = 1.f;
        }
        if (a.x_row_bytes) {   // uniform
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t base = __umul24((uint32_t)u[j], a.x_row_bytes);
#pragma unroll
                for (int c = 0; c < NCH; ++c) x[j][c] = *(const typename E::Raw*)((const char*)a.X + (base + col_ld_bytes[c]));
            }
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int64_t base = (int64_t)u[j] * a.ldx;
#pragma unroll
                for (int c = 0; c < NCH; ++c) x[j][c] = E::load(a.X, base + col_ld[c]);
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (k + j < cnt) {
#pragma unroll
                for (int c = 0; c < NCH; ++c)
                    if (col_ok[c]) E::fma(acc[c], w[j], x[j][c]);
            }
        }
    }
}


// One workgroup (4 wavefronts = NG groups of LPR lanes) owns NG * kRowsPerGroup consecutive
// entries of the row list.
//   phase 0  the row descriptors (id, start, end, output scale) of the chunk go to LDS in one
//            coalesced sweep;
//   phase 1  every group streams through rows of the chunk, one LPR-wide tile of neighbours per
//            step; a group that finishes a row claims the next unclaimed one from an LDS counter,
//            so short and long rows mix without idle groups, and the ids of the NEXT tile are
//            fetched while the current tile's rows are being gathered;
//   phase 2  hub rows (more than kHubTiles tiles) are taken one at a time by ALL groups (group q takes
//            tiles q, q+NG, ...); the partial sums meet in LDS and are added in group order.
// Which group handles a row does not change the order of its additions: results are bit-reproducible.
// Workgroups per CU: see the tuning constants at the head of the file.
// SPLIT: the split route's last launch - a row's entries are those the route left over, and its sum starts from its parts.
template <int DT, int VE, int LPR, int NCH, int U, bool FILTER, bool SPLIT>
__global__ __launch_bounds__(256, NCH == 1 ? (LPR == 64 ? GNN_SPMM_MINB_WIDE : GNN_SPMM_MINB_NARROW) : 4) void spmm_rows_kernel(SpmmArgs a) {
    using E = Elem<DT, VE>;
    constexpr int RPW = kWave / LPR;
    constexpr int NG = 4 * RPW;
    constexpr int RPB = NG * kRowsPerGroup < kMaxChunk ? NG * kRowsPerGroup : kMaxChunk;  // largest chunk
    constexpr int W = LPR * NCH * VE;        // feature columns per workgroup (grid.y blocks cover F)
    __shared__ int32_t s_idx_all[4][kWave];
    __shared__ int32_t s_row_v[RPB], s_row_s[RPB], s_row_e[RPB], s_row_hub[RPB], s_row_he[RPB];
    __shared__ float s_row_sc[RPB];
    __shared__ int32_t s_row_part[SPLIT ? RPB : 1], s_row_np[SPLIT ? RPB : 1], s_row_nc[SPLIT ? RPB : 1];
    __shared__ int32_t s_next;
    __shared__ float s_red[NG][W];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int sub = lane / LPR, sl = lane % LPR;
    const int gi = wave * RPW + sub;
    int32_t* s_idx = s_idx_all[wave];
    const bool split = SPLIT && *a.split_on != 0;     // uniform
    const int32_t* const ids = split ? a.split_cold : a.col_idx;

    // ---- phase 0
    const int rpb = NG * a.rows_per_group;
    const int64_t chunk0 = (int64_t)blockIdx.x * rpb;
    const int n_chunk = (int)(((int64_t)a.n_active - chunk0) < rpb ? ((int64_t)a.n_active - chunk0) : rpb);
    if ((int)threadIdx.x < n_chunk) {
        const int r = threadIdx.x;
        const int32_t v = a.rows ? a.rows[chunk0 + r] : (int32_t)(chunk0 + r);
        const int32_t s = a.row_ptr[v];
        int32_t e = a.row_ptr[v + 1];
        if (a.cut_id >= 0 && !split) e = row_lower_bound(a.col_idx, s, e, a.cut_id);   // the entries past it can never pass the filter
        int32_t own = e - s;
        bool hub = own > kHubTiles * LPR;
        if (split) {
            // a row that reaches into another chunk of entries is taken by the whole workgroup, whatever its length
            SplitRow d = {0, 0, 0};
            if (e > s) d = a.split_rows[v];
            own = d.n_cold;
            hub = own > kHubTiles * LPR || (e > s && (uint32_t)s / kSplitChunk != (uint32_t)(e - 1) / kSplitChunk);
            s_row_part[r] = d.part;
            s_row_np[r] = d.n_parts;
            s_row_nc[r] = own;
        }
        s_row_v[r] = v;
        s_row_s[r] = s;
        s_row_e[r] = hub ? s : s + own;
        s_row_he[r] = e;
        s_row_hub[r] = hub ? 1 : 0;
        s_row_sc[r] = a.out_scale ? a.out_scale[v] : 1.f;
    }
    if (threadIdx.x == 0) s_next = NG;
    __syncthreads();

    int64_t col_off[NCH];
    bool col_ok[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        col_off[c] = (int64_t)blockIdx.y * W + (int64_t)(sl + c * LPR) * VE;
        col_ok[c] = col_off[c] < a.F;
    }
    float acc[NCH][VE];
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int k = 0; k < VE; ++k) acc[c][k] = 0.f;
    float parts[SPLIT ? NCH : 1][SPLIT ? VE : 1];     // sum of the row's parts: fetched when the row begins, added when it ends
    auto add_part = [&](float (&to)[NCH][VE], int64_t part) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (!col_ok[c]) continue;
            const float* q = a.split_plane + part * a.split_ld + col_off[c];
#pragma unroll
            for (int k = 0; k < VE; k += 4) {
                const FourRaw t = __builtin_nontemporal_load((const FourRaw*)(q + k));
                to[c][k] += __uint_as_float(t[0]); to[c][k + 1] += __uint_as_float(t[1]); to[c][k + 2] += __uint_as_float(t[2]); to[c][k + 3] += __uint_as_float(t[3]);
            }
        }
    };
    auto begin_row = [&](int j, bool valid) {
        if constexpr (SPLIT) {
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int k = 0; k < VE; ++k) parts[c][k] = 0.f;
            if (split && valid && !s_row_hub[j]) {
                const int np = s_row_np[j];
                for (int k = 0; k < np; ++k) add_part(parts, (int64_t)s_row_part[j] + k);
            }
        }
    };

    // ---- phase 1
    // Tile descriptors (row slot j, position p, row end e, valid flag) of the current tile and of the
    // two tiles after it: ids are fetched two tiles ahead and their dist values (backward filter) one
    // tile ahead, so neither latency is paid between two gathers.
    auto advance = [&](int j, uint32_t p, uint32_t e, bool hv, int& jo, uint32_t& po, uint32_t& eo, bool& ho) {   // (past a row's end, a position may not fit an int32_t)
        const bool done = hv && p + LPR >= e;
        int got = 0;
        if (done && sl == 0) got = atomicAdd(&s_next, 1);
        got = __shfl(got, sub * LPR, kWave);  // executed by every lane of the wave
        jo = j; po = p + LPR; eo = e; ho = hv;
        if (done) {
            jo = got;
            ho = jo < n_chunk;
            po = ho ? s_row_s[jo] : 0;
            eo = ho ? s_row_e[jo] : 0;
        }
    };
    int jc = gi;
    bool have = jc < n_chunk;
    uint32_t pc = 0, ec = 0;
    if (have) {
        pc = s_row_s[jc];
        ec = s_row_e[jc];
    }
    begin_row(jc, have);
    int jn;
    uint32_t pn, en;
    bool have_n;
    advance(jc, pc, ec, have, jn, pn, en, have_n);
    int32_t u_c = (have && pc + sl < ec) ? ids[pc + sl] : 0;
    int32_t u_n = (have_n && pn + sl < en) ? ids[pn + sl] : 0;
    int32_t d_c = 0;
    if (FILTER) d_c = (have && pc + sl < ec) ? filter_probe(a, u_c, pc + sl) : -1;
    while (__ballot(have) != 0ull) {  // uniform over the wave
        const bool row_done = have && pc + LPR >= ec;
        int jnn;
        uint32_t pnn, enn;
        bool have_nn;
        advance(jn, pn, en, have_n, jnn, pnn, enn, have_nn);
        const int32_t u_nn = (have_nn && pnn + sl < enn) ? ids[pnn + sl] : 0;  // two tiles ahead
        int32_t d_n = 0;
        if (FILTER) d_n = (have_n && pn + sl < en) ? filter_probe(a, u_n, pn + sl) : -1;  // one tile ahead

        int left = have ? (int)(ec - pc) : 0;
        left = left < 0 ? 0 : (left < LPR ? left : LPR);
        wave_lds_sync();  // the previous tile has been consumed
        const int cnt = commit_tile<LPR, FILTER>(a, sl < left, u_c, d_c, left, sub, sl, s_idx);
        int cnt_max = cnt;
#pragma unroll
        for (int d = LPR; d < kWave; d <<= 1) cnt_max = max(cnt_max, __shfl_xor(cnt_max, d, kWave));
        wave_lds_sync();
        consume_tile<E, LPR, NCH, U>(a, cnt, cnt_max, sub, col_off, col_ok, s_idx, acc);

        if (row_done) {
            if (!s_row_hub[jc]) {
                const int32_t v = s_row_v[jc];
                const float sc = s_row_sc[jc];
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    if (col_ok[c]) {
                        float o[VE];
#pragma unroll
                        for (int k = 0; k < VE; ++k) {
                            if constexpr (SPLIT) acc[c][k] += parts[c][k];
                            o[k] = acc[c][k] * sc;
                        }
                        const int64_t rest = (int64_t)a.F - col_off[c];
                        E::store(a.Y, (int64_t)v * a.ldy + col_off[c], o, rest >= VE ? VE : (int)rest, a.accumulate != 0, a.relu_h,
                                 (int64_t)v * a.ldh + col_off[c]);
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int k = 0; k < VE; ++k) acc[c][k] = 0.f;
        }
        if (row_done) begin_row(jn, have_n);
        jc = jn; pc = pn; ec = en; have = have_n;
        jn = jnn; pn = pnn; en = enn; have_n = have_nn;
        u_c = u_n; u_n = u_nn; d_c = d_n;
    }

    // ---- phase 2
    __syncthreads();
    for (int q = 0; q < n_chunk; ++q) {
        if (!s_row_hub[q]) continue;  // uniform over the workgroup
        const int32_t hv = s_row_v[q];
        const int32_t hs = s_row_s[q], he = s_row_he[q];
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int k = 0; k < VE; ++k) acc[c][k] = 0.f;
        // entries lo .. hi: the wave's RPW groups take consecutive LPR-wide tiles of every 64-entry stretch (a macro: as a lambda, or as one
        // loop for both forms, the compiler keeps other values in registers: 602 columns, 66 870 rows of 36, 816 -> 831 us)
#define GNN_HUB_WALK(lo_, hi_)                                                                                          \
        for (int64_t base = (int64_t)(lo_) + (int64_t)wave * kWave; base < (hi_); base += 4 * kWave) {                  \
            const int64_t p0 = base + sub * LPR;                                                                        \
            int left = (int)((int64_t)(hi_)-p0 < 0 ? 0 : ((int64_t)(hi_)-p0 < LPR ? (int64_t)(hi_)-p0 : LPR));         \
            const int32_t u = sl < left ? ids[p0 + sl] : 0;                                                             \
            int32_t d = 0;                                                                                              \
            if (FILTER) d = sl < left ? filter_probe(a, u, (int32_t)(p0 + sl)) : -1;                                    \
            wave_lds_sync();                                                                                            \
            const int cnt = commit_tile<LPR, FILTER>(a, sl < left, u, d, left, sub, sl, s_idx);                         \
            int cnt_max = cnt;                                                                                          \
            _Pragma("unroll") for (int w = LPR; w < kWave; w <<= 1) cnt_max = max(cnt_max, __shfl_xor(cnt_max, w, kWave)); \
            wave_lds_sync();                                                                                            \
            consume_tile<E, LPR, NCH, U>(a, cnt, cnt_max, sub, col_off, col_ok, s_idx, acc);                            \
        }
        if constexpr (!SPLIT) {
            GNN_HUB_WALK(hs, he)
        } else {
            // a row of the split route: chunk by chunk, its parts (one of every NG to a group) and its other entries there
            int64_t lo = hs, hi = he, chunk = 0;
            if (split) {
                chunk = (uint32_t)hs / kSplitChunk;
                hi = lo + s_row_nc[q];
                for (int k = gi; k < s_row_np[q]; k += NG) add_part(acc, (int64_t)s_row_part[q] + k);
            }
            for (;;) {
                GNN_HUB_WALK(lo, hi)
                ++chunk;
                if (!split || chunk * kSplitChunk >= he) break;      // uniform
                const SplitChunk d = a.split_chunks[chunk];
                lo = chunk * kSplitChunk;
                hi = lo + d.head_cold;
                for (int k = gi; k < d.head_parts; k += NG) add_part(acc, (int64_t)d.part0 + k);
            }
        }
#undef GNN_HUB_WALK
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int k = 0; k < VE; ++k) s_red[gi][(sl + c * LPR) * VE + k] = acc[c][k];
        __syncthreads();
        const float sc = s_row_sc[q];
        for (int col = threadIdx.x; col < W; col += 256) {
            const int64_t gcol = (int64_t)blockIdx.y * W + col;
            if (gcol < a.F) {
                float t = 0.f;
#pragma unroll
                for (int r = 0; r < NG; ++r) t += s_red[r][col];
                float o[1] = {t * sc};
                Elem<DT, 1>::store(a.Y, (int64_t)hv * a.ldy + gcol, o, 1, a.accumulate != 0, a.relu_h, (int64_t)hv * a.ldh + gcol);
            }
        }
        __syncthreads();
    }
}


// ---- edge-balanced kernel ------------------------------------------------------------------
// One workgroup owns up to kStreamMaxRows consecutive entries of the row list, but the work is split
// by EDGES, not by rows: the rows' neighbour lists are treated as one concatenated stream, taken in equal pieces of
// at most kStreamPiece edges, and of a piece each of the NG lane groups takes a contiguous stretch.  A row
// that lies inside one stretch is summed and stored by that group; of a row cut by stretch boundaries the
// groups behind its first one leave their sums ("heads") in LDS, and after a barrier the first one adds them in
// stream order and stores the row, or hands the sum to the next piece.  So power-law rows cost no imbalance inside the
// workgroup, and the result is a fixed-order sum (bit-reproducible).
// It serves the column-blocked route of row lists and of short calls (others: spmm_fours.h, fours_pay): the workgroup id carries (chunk, die) = (id / 8, id % 8);
// every row is cut to the die's column block through `seg`, and the unscaled float sums go to plane `die` of the partial buffer
// (a.Y, row index = position in the row list), not to the output matrix.
//
// Beside the L2 misses of a 7.4 MB block every instruction per edge counts: a CU takes 16 clocks for a 1 KB load, the time
// of 16 vector instructions.  Hence ids are staged for a whole piece at once (one search per lane, then steps along the
// row ends; the next piece's ids are fetched while this one is gathered), row starts are a bit per edge, tested for the
// whole wavefront by scalar instructions, and a load's address is one addition to a staged dword.  114 M edges of 233 000 rows,
// 256 columns, the whole call: 6.2 ms in fp32, 3.7 in bf16.  Pieces of 4096 edges, 8 loads in flight, 5 or 7 workgroups per CU, non-temporal
// id loads: all within 2 % or slower.
constexpr int kStreamMaxRows = 256;
constexpr int kStreamLoads = 4;          // row loads in flight per lane
constexpr int kStreamPiece = 2048;       // edges staged in LDS at a time
constexpr int kStreamWgEdges = 8192;     // edges one workgroup aims for when the host picks its row count

// OFF32: the gathered matrix spans less than 4 GB, so a row's byte offset is a dword beside a scalar base.
template <int DT, int VE, int LPR, int U, bool SCALED, bool OFF32>
__global__ __launch_bounds__(256, SCALED ? 4 : 6) void spmm_stream_kernel(SpmmArgs a) {
    using E = Elem<DT, VE>;
    constexpr int RPW = kWave / LPR;
    constexpr int NG = 4 * RPW;
    constexpr int W = LPR * VE;              // feature columns per workgroup (grid.y blocks cover F)
    constexpr int kPiece = kStreamPiece;
    constexpr int kPad = kPiece / NG + 8;    // a group that ends early reads on to the common length of a stretch
    constexpr int kIds = kPiece / 256;       // ids a lane fetches for a piece
    static_assert(8 % U == 0 && kPiece % (NG * 8) == 0, "a stretch is a whole number of rounds");
    __shared__ int32_t s_delta[kStreamMaxRows], s_voff[kStreamMaxRows + 1], s_row[kStreamMaxRows];
    __shared__ uint32_t s_empty[kStreamMaxRows / 32];
    __shared__ __attribute__((aligned(16))) uint32_t s_ent[kPiece + kPad];                       // row offset of every staged edge
    __shared__ __attribute__((aligned(16))) float s_w[SCALED ? kPiece + kPad : 4];               // its scale factor
    __shared__ uint32_t s_flag[(kPiece + kPad) / 32 + 3];                                        // bit: the edge begins a row
    __shared__ __attribute__((aligned(16))) float s_head[NG][W], s_run[2][W];
    __shared__ int32_t s_head_row[NG], s_run_row[2];
    __shared__ int s_scan[4];
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int sub = lane / LPR, sl = lane % LPR;
    const int gi = wave * RPW + sub;

    // ---- the rows with edges in this block, and the exclusive prefix of their lengths
    const int rpw = a.rows_per_group;  // rows of the list per workgroup, <= kStreamMaxRows
    const int die = (int)(blockIdx.x % kDies);
    const int64_t chunk0 = (int64_t)(blockIdx.x / kDies) * rpw;
    const int n_chunk = (int)(((int64_t)a.n_active - chunk0) < rpw ? ((int64_t)a.n_active - chunk0) : rpw);
    float* const part = (float*)a.Y + ((int64_t)die * a.n_active + chunk0) * a.ldy;
    int len = 0, first = 0;
    if (tid < n_chunk) {
        const int64_t v = chunk0 + tid;
        const int32_t* cut = a.seg + v * (a.n_blocks + 1) + a.block0 + die;
        first = cut[0];
        const int32_t e = a.seg_end ? a.seg_end[v * a.n_blocks + a.block0 + die] : cut[1];
        len = e - first;
    }
    int n_edges, n_rows;
    const int voff = block_exclusive_scan<256>(len, s_scan, &n_edges);
    const int slot = block_exclusive_scan<256>(len > 0 ? 1 : 0, s_scan, &n_rows);
    if (len > 0) {
        s_voff[slot] = voff;
        s_delta[slot] = first - voff;
        s_row[slot] = tid;
    }
    if (tid == 0) s_voff[n_rows] = n_edges;
    if (tid < 2) s_run_row[tid] = -1;
    const uint64_t empty = __ballot(tid < n_chunk && len == 0);
    if (lane < 2) s_empty[wave * 2 + lane] = (uint32_t)(empty >> (32 * lane));
    __syncthreads();

    const int64_t col_off = (int64_t)blockIdx.y * W + (int64_t)sl * VE;
    const bool col_ok = col_off < a.F;
    const int n_valid = (int64_t)a.F - col_off >= VE ? VE : (int)((int64_t)a.F - col_off);
    // the slab's first column, and a lane's 16 bytes in it (bytes 0 for the lanes past F, whose sums are never stored); a
    // neighbour's row then adds its offset: bytes, or 16-byte units where a dword of bytes does not reach
    constexpr int ES = DT == GNN_F32 ? 4 : 2;
    const char* const x_slab = (const char*)a.X + (int64_t)blockIdx.y * W * ES;
    const uint32_t lane_off = col_ok ? (uint32_t)(sl * 16) : 0u;
    const uint32_t row_units = (uint32_t)(OFF32 ? a.ldx * ES : a.ldx * ES / 16);
    // slot of the row that holds stream position t
    auto row_of = [&](int t) {
        int x = 0, y = n_rows;
        while (y - x > 1) {
            const int m = (x + y) >> 1;
            if (s_voff[m] <= t) x = m;
            else y = m;
        }
        return x;
    };
    auto store_row = [&](int row, const float (&v)[VE]) {
        if (col_ok) store_part<VE>(part, (int64_t)s_row[row] * a.ldy + col_off, v, n_valid, a.accumulate != 0);
    };

    const int n_pieces = (n_edges + kPiece - 1) / kPiece;
    const int piece = n_pieces > 0 ? (((n_edges + n_pieces - 1) / n_pieces) + 7) / 8 * 8 : 1;   // equal pieces
    // a piece's ids: a wave takes a stretch of its own, 64 consecutive edges a step; fetched while the piece before is gathered
    uint32_t u[kIds];
    float w[kIds];
    uint32_t begins = 0;     // bit i: this lane's i-th edge begins a row
    auto fetch = [&](int t0) {
        const int n = n_edges - t0 < piece ? n_edges - t0 : piece;
        const int steps = (n + 255) / 256;
        const int k = wave * steps * kWave + lane;
        int x = 0, begin = 0, end = 0, delta = 0;
        if (k < n) {
            x = row_of(t0 + k);
            begin = s_voff[x];
            end = s_voff[x + 1];
            delta = s_delta[x];
        }
        begins = 0;
#pragma unroll
        for (int i = 0; i < kIds; ++i) {
            const int t = t0 + k + i * kWave;
            int32_t p = 0;
            if (k + i * kWave < n && i < steps) {
                if (t >= end) {
                    do {
                        begin = end;
                        end = s_voff[++x + 1];
                    } while (t >= end);
                    delta = s_delta[x];
                }
                if (t == begin) begins |= 1u << i;
                p = t + delta;
            }
            u[i] = (uint32_t)a.col_idx[p];
            w[i] = SCALED ? a.edge_w[p] : 1.f;
        }
    };
    if (n_edges > 0) fetch(0);
    for (int t0 = 0, turn = 0; t0 < n_edges; t0 += piece, turn ^= 1) {
        const int n = n_edges - t0 < piece ? n_edges - t0 : piece;
        const int per = ((n + NG - 1) / NG + 7) / 8 * 8;    // edges of a group's stretch
        {
            const int steps = (n + 255) / 256;
            const int k = wave * steps * kWave + lane;
#pragma unroll
            for (int i = 0; i < kIds; ++i) {
                if (i < steps) {        // uniform
                    const int q = k + i * kWave;
                    if (q < n) {
                        s_ent[q] = u[i] * row_units;
                        if (SCALED) s_w[q] = w[i];
                    }
                    const uint64_t b = __ballot((begins >> i) & 1u);
                    if (lane < 2) s_flag[((q - lane) >> 5) + lane] = (uint32_t)(b >> (32 * lane));
                }
            }
            for (int q = n + tid; q < n + per; q += 256) s_ent[q] = 0;   // a valid row, never added
        }
        __syncthreads();     // (also: the cut rows of the piece before have been read)
        if (t0 + piece < n_edges) fetch(t0 + piece);
        const int lo = gi * per < n ? gi * per : n;
        const int cnt = n - lo < per ? n - lo : per;        // this group's stretch: edges lo .. lo + cnt of the piece
        const int at = cnt > 0 ? lo : 0;
        int cur = 0, head_row = -1;
        bool cut = false;          // the accumulators' row began in an earlier stretch
        float acc[VE];
#pragma unroll
        for (int k = 0; k < VE; ++k) acc[k] = 0.f;
        if (cnt > 0) {
            cur = row_of(t0 + lo);
            cut = s_voff[cur] < t0 + lo;
        }
        auto end_row = [&]() {     // the accumulators' row has ended inside this stretch
            if (cut) {
                head_row = cur;
#pragma unroll
                for (int k = 0; k < VE; ++k) s_head[gi][sl * VE + k] = acc[k];
            } else {
                store_row(cur, acc);
            }
        };
        for (int k1 = 0; k1 < per; k1 += 32) {
            // bit k of `starts`: edge k1 + k of this group's stretch begins a row; `any`: of some group of the wave
            const int q = at + k1;
            uint32_t starts = __builtin_amdgcn_alignbit(s_flag[(q >> 5) + 1], s_flag[q >> 5], (uint32_t)q & 31u);
            if (k1 == 0) starts &= ~1u;                     // the stretch's first edge continues the accumulators' row
            const int left = per - k1 < 32 ? per - k1 : 32;
            uint32_t any = starts;
#pragma unroll
            for (int d = LPR; d < kWave; d <<= 1) any |= __shfl_xor(any, d, kWave);
            any = __builtin_amdgcn_readfirstlane(any);
#pragma unroll 1
            for (int k0 = 0; k0 < left; k0 += U) {
                // The loads are unconditional (past the group's count lies row 0 or another group's edge, a column past F
                // reads the slab's first column: valid addresses, the values are never used): with branches around them
                // the compiler waits for every load before issuing the next one.
                typename E::Raw x[U];
                float wt[U];
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const uint32_t off = s_ent[q + k0 + j];
                    wt[j] = SCALED ? s_w[q + k0 + j] : 1.f;
                    if (OFF32) x[j] = *(const typename E::Raw*)(x_slab + (off + lane_off));
                    else x[j] = *(const typename E::Raw*)(x_slab + (((uint64_t)off << 4) + lane_off));
                }
                // the common round: all groups have its edges and none of them begins a row (scalar test)
                const bool full = __ballot(cnt < k1 + k0 + U) == 0ull;
                if (full && ((any >> k0) & ((1u << U) - 1u)) == 0u) {
#pragma unroll
                    for (int j = 0; j < U; ++j) E::fma(acc, wt[j], x[j]);
                } else {
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        if (k1 + k0 + j < cnt) {
                            if ((starts >> (k0 + j)) & 1u) {
                                end_row();
                                cut = false;
                                ++cur;
#pragma unroll
                                for (int k = 0; k < VE; ++k) acc[k] = 0.f;
                            }
                            E::fma(acc, wt[j], x[j]);
                        }
                    }
                }
            }
        }
        bool tail = false;         // the accumulators' row goes on in the next stretch
        if (cnt > 0) {
            tail = !cut && s_voff[cur + 1] > t0 + lo + cnt;
            if (!tail) end_row();
        }
        if (sl == 0) s_head_row[gi] = head_row;
        __syncthreads();
        // ---- rows cut by stretch boundaries: the group where the row began (group 0 for the row that came out of the piece
        // before) adds the heads of the groups behind it, in stream order
        int row = tail ? cur : -1, g = gi + 1;
        for (int pass = 0; pass < 2; ++pass) {
            if (pass == 1) {
                if (gi != 0) break;
                row = s_run_row[turn];
                g = 0;
#pragma unroll
                for (int k = 0; k < VE; ++k) acc[k] = s_run[turn][sl * VE + k];
            }
            if (row < 0) continue;
            for (; g < NG && s_head_row[g] == row; ++g)
#pragma unroll
                for (int k = 0; k < VE; ++k) acc[k] += s_head[g][sl * VE + k];
            if (s_voff[row + 1] > t0 + n) {      // goes on in the next piece
#pragma unroll
                for (int k = 0; k < VE; ++k) s_run[turn ^ 1][sl * VE + k] = acc[k];
                if (sl == 0) s_run_row[turn ^ 1] = row;
            } else {
                store_row(row, acc);
            }
        }
        if (gi == 0 && sl == 0) s_run_row[turn] = -1;
    }
    // ---- rows without any edge are zero (they never show up in the stream)
    if (!a.accumulate) {
        float zero[VE];
#pragma unroll
        for (int k = 0; k < VE; ++k) zero[k] = 0.f;
        for (int r = gi; r < n_chunk; r += NG) {
            if (!((s_empty[r >> 5] >> (r & 31)) & 1u) || !col_ok) continue;
            store_part<VE>(part, (int64_t)r * a.ldy + col_off, zero, n_valid, false);
        }
    }
}

template <int DT, int VE, int LPR>
static int32_t launch_stream(const SpmmArgs& a, bool off32, hipStream_t stream) {
    constexpr int U = kStreamLoads;
    constexpr int W = LPR * VE;
    constexpr bool S = DT != GNN_F32;     // (fp32 gathers from rows that are scaled already)
    const int64_t n_chunks = ((int64_t)a.n_active + a.rows_per_group - 1) / a.rows_per_group;
    dim3 grid((unsigned)(n_chunks * kDies), (unsigned)((a.F + W - 1) / W));
    if (off32) {
        if (S && a.edge_w) spmm_stream_kernel<DT, VE, LPR, U, S, true><<<grid, 256, 0, stream>>>(a);
        else spmm_stream_kernel<DT, VE, LPR, U, false, true><<<grid, 256, 0, stream>>>(a);
    } else {
        if (S && a.edge_w) spmm_stream_kernel<DT, VE, LPR, U, S, false><<<grid, 256, 0, stream>>>(a);
        else spmm_stream_kernel<DT, VE, LPR, U, false, false><<<grid, 256, 0, stream>>>(a);
    }
    GNN_LAUNCH_CHECK("spmm_stream_kernel");
    return GNN_OK;
}

template <int DT, int VE, int LPR, int NCH, bool FILTER, bool SPLIT = false>
static int32_t launch_rows(const SpmmArgs& a, hipStream_t stream) {
    constexpr int U = NCH == 1 ? (LPR < 16 ? 4 : (LPR < 64 ? GNN_SPMM_U_NARROW : GNN_SPMM_U_WIDE)) : (NCH == 2 ? 4 : (NCH == 3 ? 3 : 2));
    constexpr int NG = 4 * (kWave / LPR);
    constexpr int W = LPR * NCH * VE;
    // chunk size: as large as possible (better balance inside a workgroup) while the launch still
    // has about 16 workgroups per CU
    SpmmArgs b = a;
    int rpg = (int)((int64_t)a.n_active / ((int64_t)NG * 4096));
    constexpr int kMaxRpg = kRowsPerGroup * NG <= kMaxChunk ? kRowsPerGroup : kMaxChunk / NG;
    b.rows_per_group = rpg < 1 ? 1 : (rpg > kMaxRpg ? kMaxRpg : rpg);
    const int rpb = NG * b.rows_per_group;
    dim3 grid((unsigned)(((int64_t)a.n_active + rpb - 1) / rpb), (unsigned)((a.F + W - 1) / W));
    spmm_rows_kernel<DT, VE, LPR, NCH, U, FILTER, SPLIT><<<grid, 256, 0, stream>>>(b);
    GNN_LAUNCH_CHECK("spmm_rows_kernel");
    return GNN_OK;
}

// Column-block boundaries: bounds[j], j = 0 .. n_blocks, split the gathered neighbour ids [0, n_src) so that every block holds
// about the same number of the call's entries (with a dist filter: of those that pass it).  The die whose block has the
// most entries ends last, and the others wait: with eight equally long blocks of a partition numbered by (distance, id), whose
// first block - the targets - holds 1.20 times its share of the entries, a call over 114 M entries (233 000 rows of 256 floats) took 7.33 ms
// or 7.01, as that block's die had an even number or an odd one (workgroup 0 of a launch goes to a die that depends on the
// hardware queue behind the stream); cut like this 6.25 to 6.32 on every queue (bf16 4.43 / 4.26, now 3.78; vertices renamed at random, where
// equal blocks are equal shares, 6.21 -> 6.23).
// 131 072 entries, one at a hashed place in each of as many equal stretches, are counted into 2048 bins of ids; the share of a
// bin is that of its samples, but at least half its share of the (active) ids: a block of rare ids outgrows the L2 otherwise.
// The samples are random reads all over the entries, 1.5 ns apart for a single workgroup (65 536 of them 0.1 ms): 512
// workgroups fetch them, one counts.  The counts are integers, so the same call cuts at the same ids.
constexpr int kBoundBins = 2048, kBoundSamples = 131072, kMaxFourBlocks = 512;

__device__ __forceinline__ int64_t bound_sample(int i, int64_t n) {      // the i-th stretch's place of n
    uint32_t h = (uint32_t)i * 2654435761u;
    h = (h ^ (h >> 15)) * 2246822519u;
    h ^= h >> 13;
    return ((int64_t)i * n + (int64_t)(((uint64_t)h * (uint64_t)n) >> 32)) / kBoundSamples;
}

// bins[i]: bin of the i-th sampled entry, kBoundBins if it is not gathered; with dist, bins[kBoundSamples + i]: of the i-th sampled id
__global__ __launch_bounds__(256) void spmm_samples_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                            int32_t n_rows, const int32_t* __restrict__ dist, int32_t max_dist, int32_t n_src,
                                                            uint16_t* __restrict__ bins) {
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    const int32_t width = (n_src + kBoundBins - 1) / kBoundBins, first = row_ptr[0];
    const int64_t m = (int64_t)row_ptr[n_rows] - first;
    int32_t u = m > 0 ? col_idx[first + bound_sample(i, m)] : n_src, v = (int32_t)bound_sample(i, n_src);
    if (dist) {
        const int32_t du = dist[u < n_src ? u : 0], dv = dist[v];
        if (du < 0 || du > max_dist) u = n_src;
        if (dv < 0 || dv > max_dist) v = n_src;
        bins[kBoundSamples + i] = (uint16_t)(v < n_src ? v / width : kBoundBins);
    }
    bins[i] = (uint16_t)(u < n_src ? u / width : kBoundBins);
}

__global__ __launch_bounds__(1024) void spmm_bounds_kernel(const uint16_t* __restrict__ bins, bool filtered, int32_t n_src, int32_t n_blocks,
                                                            int32_t* __restrict__ bounds) {
    __shared__ int32_t s_e[kBoundBins + 1], s_v[kBoundBins + 1], s_cum[kBoundBins + 1], s_cut[kMaxFourBlocks];
    __shared__ int s_part[16];
    constexpr int kPer = kBoundBins / 1024, kLoads = kBoundSamples / 1024 / 8;
    const int tid = (int)threadIdx.x;
    const int32_t width = (n_src + kBoundBins - 1) / kBoundBins;
    for (int b = tid; b <= kBoundBins; b += 1024) s_e[b] = s_v[b] = 0;
    __syncthreads();
    auto count = [&](int32_t* to, const uint16_t* from) {
        uint4 x[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) x[k] = ((const uint4*)from)[k * 1024 + tid];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const uint32_t w[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                atomicAdd(&to[w[j] & 0xffffu], 1);
                atomicAdd(&to[w[j] >> 16], 1);
            }
        }
    };
    count(s_e, bins);
    if (filtered) count(s_v, bins + kBoundSamples);
    __syncthreads();
    int32_t e[kPer], v[kPer], all_e, all_v, sum_e = 0, sum_v = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int b = tid * kPer + k;
        e[k] = s_e[b];
        v[k] = s_v[b];
        sum_e += e[k];
        sum_v += v[k];
    }
    block_exclusive_scan<1024>(sum_e, s_part, &all_e);
    block_exclusive_scan<1024>(sum_v, s_part, &all_v);
    int32_t mass[kPer], sum = 0, total;      // of a bin, in 2^-28ths of all: less than 2^29 together
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t lo = (int64_t)(tid * kPer + k) * width, ids = lo >= n_src ? 0 : (n_src - lo < width ? n_src - lo : width);
        const float share_v = all_v > 0 ? (float)v[k] / (float)all_v : (float)ids / (float)n_src;
        const float share_e = all_e > 0 ? (float)e[k] / (float)all_e : 0.f;
        mass[k] = (int32_t)(fmaxf(share_e, share_v * 0.5f) * 268435456.f);
        sum += mass[k];
    }
    int32_t at = block_exclusive_scan<1024>(sum, s_part, &total);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        s_cum[tid * kPer + k] = at;
        at += mass[k];
    }
    if (tid == 0) {
        s_cum[kBoundBins] = total;
        bounds[0] = 0;
        bounds[n_blocks] = n_src;
    }
    __syncthreads();
    for (int j = 1 + tid; j < n_blocks; j += 1024) {
        const int32_t want = (int32_t)((int64_t)j * total / n_blocks);      // < total: some bin holds it
        int x = 0, y = kBoundBins;
        while (y - x > 1) {
            const int h = (x + y) >> 1;
            if (s_cum[h] <= want) x = h;
            else y = h;
        }
        const int64_t at_id = (int64_t)x * width + (int64_t)(want - s_cum[x]) * width / (s_cum[x + 1] > s_cum[x] ? s_cum[x + 1] - s_cum[x] : 1);
        bounds[j] = (int32_t)(at_id < n_src ? at_id : n_src);
        if (n_blocks <= kMaxFourBlocks) s_cut[j] = bounds[j];
    }
    __syncthreads();
    // an id's place in its block has 16 bits: at most kBlockIds of them (on average a block holds half as many)
    if (tid == 0 && n_blocks <= kMaxFourBlocks) {
        int64_t last = 0;
        for (int j = 1; j < n_blocks; ++j) {
            const int64_t least = (int64_t)n_src - (int64_t)(n_blocks - j) * kBlockIds;
            last = std::min(std::max((int64_t)s_cut[j], least), last + kBlockIds);
            bounds[j] = (int32_t)last;
        }
    }
}

// Cut points of every listed row at the column-block boundaries (rows sorted by column): seg[r][j] = first position
// of row r whose column is >= the j-th boundary; seg[r][0] = start,
// seg[r][n_blocks] = end - or, with limit < n_cols, the first position whose column is >= limit (the entries past it
// are never gathered), and no boundary lies above limit.
__global__ __launch_bounds__(256) void spmm_seg_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                        const int32_t* __restrict__ rows, int32_t n_active, int32_t n_blocks,
                                                        const int32_t* __restrict__ bounds, int32_t limit, int32_t n_cols,
                                                        int32_t* __restrict__ seg) {
    const int64_t total = (int64_t)n_active * (n_blocks + 1);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = (int32_t)(i / (n_blocks + 1)), j = (int32_t)(i % (n_blocks + 1));
        const int32_t v = rows ? rows[r] : r;
        int32_t lo = row_ptr[v], hi = row_ptr[v + 1];
        if (j == n_blocks) {
            lo = limit < n_cols ? row_lower_bound(col_idx, lo, hi, limit) : hi;
        } else if (j > 0) {
            lo = row_lower_bound(col_idx, lo, hi, bounds[j]);
        }
        seg[i] = lo;
    }
}

// Per-edge preparation of the column-blocked route, done once per call instead of once per feature slab: every
// (row, block) segment is copied to `ids` at its own position - with a dist filter (backward) the neighbours that
// fail the test are squeezed out, seg_end[r][j] = where the kept ones end - and with a neighbour scale the factor of
// every kept neighbour goes to `w` at the same position (the random 4-byte gathers of the scale vector happen here,
// once; the stream kernel then reads ids and factors coalesced).  One group of 16 lanes per segment.
__global__ __launch_bounds__(256) void spmm_prepare_kernel(const int32_t* __restrict__ col_idx, const int32_t* __restrict__ seg,
                                                            const int32_t* __restrict__ dist, int32_t max_dist,
                                                            const float* __restrict__ nbr_scale, int64_t n_segments, int32_t n_blocks,
                                                            int32_t* __restrict__ ids, float* __restrict__ w, int32_t* __restrict__ seg_end) {
    constexpr int LPG = 16;
    const int lane = lane_id(), sub = lane / LPG, sl = lane % LPG;
    const int64_t groups = (int64_t)gridDim.x * (blockDim.x / LPG);
    for (int64_t sgm = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / LPG; sgm < n_segments; sgm += groups) {
        const int64_t r = sgm / n_blocks;
        const int32_t j = (int32_t)(sgm % n_blocks);
        const int32_t lo = seg[r * (n_blocks + 1) + j], hi = seg[r * (n_blocks + 1) + j + 1];
        int32_t out = lo;
        // kT tiles of 16 entries per step: all their id loads go out together, then all dist / scale loads, so a
        // typical segment (a few tiles) pays each memory latency once instead of once per tile
        constexpr int kT = 4;
        for (uint32_t p = lo; p < (uint32_t)hi; p += kT * LPG) {
            int32_t u[kT], d[kT];
            float f[kT];
            bool valid[kT];
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                valid[t] = p + t * LPG + sl < (uint32_t)hi;
                u[t] = valid[t] ? col_idx[p + t * LPG + sl] : 0;
            }
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                d[t] = dist ? dist[u[t]] : 0;          // u = 0 where the lane has no entry: a valid index
                f[t] = nbr_scale ? nbr_scale[u[t]] : 1.f;
            }
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                const bool keep = valid[t] && d[t] >= 0 && d[t] <= (dist ? max_dist : 0);
                const uint64_t kept = (__ballot(keep) >> (sub * LPG)) & 0xffffull;
                if (keep) {
                    const int32_t q = out + __popcll(kept & ((1ull << sl) - 1ull));
                    ids[q] = u[t];
                    if (nbr_scale) w[q] = f[t];
                }
                out += __popcll(kept);
            }
        }
        if (sl == 0) seg_end[sgm] = out;
    }
}

// Y[v, c] (+)= out_scale[v] * (plane 0 + plane 1 + ... + plane 7)[r, c], v = rows[r]: planes added in die order.
// One thread per four columns; part rows are 16-byte aligned, and so are the rows of Y (vector route only).
template <int DT>
__global__ __launch_bounds__(256) void spmm_sum_parts_kernel(const float* __restrict__ part, int64_t ldp, const int32_t* __restrict__ rows,
                                                              int32_t n_active, int32_t F, void* __restrict__ Y, int64_t ldy,
                                                              const float* __restrict__ out_scale, int32_t accumulate, const void* __restrict__ relu_h, int64_t ldh) {
    const int32_t f4 = (F + 3) / 4;
    const int64_t total = (int64_t)n_active * f4;
    const int64_t plane = (int64_t)n_active * ldp;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = (int32_t)(i / f4), c = (int32_t)(i % f4) * 4;
        const int32_t v = rows ? rows[r] : r;
        float4 t = *(const float4*)(part + (int64_t)r * ldp + c);
#pragma unroll
        for (int d = 1; d < kDies; ++d) {
            const float4 q = *(const float4*)(part + d * plane + (int64_t)r * ldp + c);
            t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
        }
        const float sc = out_scale ? out_scale[v] : 1.f;
        float o[4] = {t.x * sc, t.y * sc, t.z * sc, t.w * sc};
        const int n_valid = F - c >= 4 ? 4 : F - c;
        const int64_t off = (int64_t)v * ldy + c;
        // the stored value is zeroed where relu_h (same rows and columns as Y) is <= 0; relu_h == Y: where it is <= 0 itself
        const bool self = relu_h == (const void*)Y;
        bool pass[4] = {true, true, true, true};
        // (rows of relu_h and Y start on 16 bytes: the columns up to the next multiple of four are there)
        using E = Elem<DT, 4>;
        if (relu_h && !self) {
            float h[4] = {0.f, 0.f, 0.f, 0.f};
            E::fma(h, 1.f, E::load(relu_h, (int64_t)v * ldh + c));
#pragma unroll
            for (int k = 0; k < 4; ++k) pass[k] = h[k] > 0.f;
        }
        if (accumulate) {
            float y[4] = {0.f, 0.f, 0.f, 0.f};
            E::fma(y, 1.f, E::load(Y, off));
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] += y[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = (self ? o[k] > 0.f : pass[k]) ? o[k] : 0.f;
        if (DT == GNN_F32) {
            float* y = (float*)Y + off;
            if (n_valid == 4) *(float4*)y = make_float4(o[0], o[1], o[2], o[3]);
            else
                for (int k = 0; k < n_valid; ++k) y[k] = o[k];
        } else {
            uint16_t* y = (uint16_t*)Y + off;
            if (n_valid == 4) *(uint2*)y = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
            else
                for (int k = 0; k < n_valid; ++k) y[k] = f32_to_bf16(o[k]);
        }
    }
}

// Y[v, 0:F] = bias[0:F] for the listed rows: the starting value of an aggregation that has no self term under it.
template <int DT>
__global__ __launch_bounds__(256) void spmm_bias_rows_kernel(const int32_t* __restrict__ rows, int32_t n_active, const float* __restrict__ bias,
                                                              void* __restrict__ Y, int64_t ldy, int32_t F) {
    const int64_t total = (int64_t)n_active * F;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t i = (int32_t)(t / F), c = (int32_t)(t % F);
        const int64_t v = rows ? (int64_t)rows[i] : i;
        if (DT == GNN_F32) ((float*)Y)[v * ldy + c] = bias[c];
        else ((uint16_t*)Y)[v * ldy + c] = f32_to_bf16(bias[c]);
    }
}

// Xs[u, 0:F] = scale[u] * X[u, 0:F] for every row of the gathered matrix (16-byte aligned rows): with a neighbour scale
// the column-blocked route gathers from this copy, so its inner loop needs no per-edge factor.
template <int DT>
__global__ __launch_bounds__(256) void spmm_scale_rows_kernel(const void* __restrict__ X, int64_t ldx, int32_t n_rows, int32_t F,
                                                              const float* __restrict__ scale, void* __restrict__ Xs) {
    using E = Elem<DT, DT == GNN_F32 ? 4 : 8>;
    constexpr int VE = E::VE;
    const int vpr = (F + VE - 1) / VE;
    const int64_t total = (int64_t)n_rows * vpr;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = t / vpr;
        const int64_t off = u * ldx + (t % vpr) * VE;
        float acc[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) acc[e] = 0.f;
        E::fma(acc, scale[u], E::load(X, off));
        E::store(Xs, off, acc, VE, false);
    }
}

// ---- does workgroup i run on compute die i mod 8? --------------------------------------------------------------
// The column-blocked route rests on it (correctness does not: with another dispatch order the sums are the same, only
// the reason for the route is gone).  Checked once per device, at the first call that would take the route: a 16 x 4
// grid of one-wave workgroups records the die (XCC) id each of them ran on; the route is taken only if the first eight
// ids are eight different dies and workgroup i (in dispatch order: x fastest) repeats the die of workgroup i mod 8.
constexpr int kProbeX = 16, kProbeY = 4;
static __device__ int32_t g_die_probe[kProbeX * kProbeY];

__global__ __launch_bounds__(64) void die_probe_kernel(int32_t* __restrict__ out) {
    uint32_t x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));   // bits 3:0: the die this wavefront runs on
    if (threadIdx.x == 0) out[blockIdx.y * gridDim.x + blockIdx.x] = (int32_t)(x & 0xfu);
}

static int32_t probe_die_ids(int32_t* ids_host) {
    void* p = nullptr;
    GNN_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(g_die_probe)));
    die_probe_kernel<<<dim3(kProbeX, kProbeY), 64, 0, (hipStream_t)0>>>((int32_t*)p);
    GNN_LAUNCH_CHECK("die_probe_kernel");
    GNN_HIP(hipMemcpy(ids_host, p, sizeof(int32_t) * kProbeX * kProbeY, hipMemcpyDeviceToHost));   // waits for the kernel
    return GNN_OK;
}

static bool die_ids_round_robin(const int32_t* ids) {
    uint32_t seen = 0;
    for (int i = 0; i < kDies; ++i) {
        if (ids[i] < 0 || ids[i] >= kDies) return false;
        seen |= 1u << ids[i];
    }
    if (seen != (1u << kDies) - 1u) return false;
    for (int i = kDies; i < kProbeX * kProbeY; ++i)
        if (ids[i] != ids[i % kDies]) return false;
    return true;
}

// 1: the mapping holds on the current device, 0: it does not (or could not be probed); probed at the first question.  `capturing`
// (nullable): a stream whose capture the probe would end - not probed then, and asked again next time.
static int die_mapping_holds(const hipStream_t* capturing = nullptr) {
    static std::mutex mu;
    static int state[64];   // per device: 0 unknown, 1 holds, 2 does not
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lock(mu);
    if (state[dev] == 0 && capturing != nullptr) {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(*capturing, &status) != hipSuccess || status != hipStreamCaptureStatusNone) return 0;
    }
    if (state[dev] == 0) {
        int32_t ids[kProbeX * kProbeY];
        state[dev] = (probe_die_ids(ids) == GNN_OK && die_ids_round_robin(ids)) ? 1 : 2;
    }
    return state[dev] == 1;
}

// The column-blocked route's shape for one call; passes == 0: the route does not apply.
struct BlockedPlan {
    int passes = 0;
    int n_blocks = 0;
    int64_t ldp = 0;          // leading dimension of a partial plane, in floats
    size_t seg_bytes = 0, part_bytes = 0;
    size_t end_bytes = 0, ids_bytes = 0;   // with a filter (stream kernel, bf16: or a neighbour scale): segment ends and the (compacted) copy of the ids
    size_t xs_bytes = 0;                   // fours: the gathered rows slab by slab; stream kernel, fp32 with a neighbour scale: the rows scaled
    size_t w_bytes = 0;                    // bf16 with a neighbour scale: the factor of every copied id, fours: of every place
    bool off32 = false;       // the gathered matrix spans less than 4 GB
    int32_t n_rows = 0, n_cols = 0;
    int32_t limit = 0;        // neighbour ids >= limit are never gathered (n_cols without a source prefix)
    int32_t rows_per_wg = 0;
    bool fours = false;       // the entries are laid out as streams of fours (spmm_fours.h)
    size_t at_bytes = 0, places = 0, before_bytes = 0;
    size_t bounds_bytes = 0, sample_bytes = 0;  // the column-block boundaries, and the samples they come from
};

// Entries of a row in a block, on average, from which the route is taken: its planes and cut points cost the same whatever the rows hold.
// fp32 has one line, 8: whole rows, with the split route where it applies, cross it at 8 to 13 on power-law graphs and below 8 on graphs
// with uniform ends (256 columns, 70 entries a row 1700 / 1500, uniform 1582 / 2347; with a dist filter not below 20).  In bfloat16 a row is half as
// long and the planes are not, so the line depends on what a call adds to an entry: over many rows no call above it was some 5 % slower than whole rows.
// Time of the route over that of whole rows, eight blocks, 130 000 and 240 000 vertices, power-law graphs (uniform ends), by entries a row:
//   fours         32 columns 100 1.10 1.14, 120 1.03 1.04 (0.99 0.81); 64 80 0.94 1.06, 100 0.96 0.98; 128 100 1.20 1.14 (0.88 0.90), 120 1.09 1.03, 140 0.88 0.94;
//                 256 80 1.07 1.26 (0.87 1.01), 100 1.00 1.06, 120 0.88 0.85; 602 72 1.01 1.11, 80 1.04 1.02, 90 0.87 0.91
//     a factor    32 400 1.17 1.00, 600 1.02 1.01; 64 200 0.97 1.02 (1.14 1.03), 300 0.99 0.92; 128 140 1.01 1.07, 170 1.02 1.01; 256 100 1.08 1.05; 602 80 1.03 1.03
//     dist filter 32 600 1.03 1.04 (1.15 1.08); 64 200 0.94 0.92 (1.21 1.15), 260 0.89 0.83 (1.04 0.97); 128 260 1.06 0.99, 300 1.05 0.94; 256 170 1.15 1.05, 200 1.08
//                 0.92; 602 120 1.18 1.00, 140 0.98 0.88
//     both        32 600 1.14 1.13 (1.21 1.12); 64 400 1.07 0.94 (1.18 1.04), 600 0.94 0.96; 128 600 1.05 0.93; 256 200 1.09 0.97; 602 120 1.16 0.97, 140 0.96 0.86
//   stream kernel (row lists; here half of the rows)
//                 32 300 1.12 1.21, 400 1.08 1.04; 64 260 0.96 0.96 (1.12 1.07), 400 0.91 0.96 (1.06 0.96); 128 140 1.07 1.14, 170 1.02 1.02; 256 120 1.14 1.09, 140 0.99
//                 0.91; 602 100 1.04 1.00 (1.04 1.11), 120 0.87 0.89
//     a factor    64 600 1.49 1.50; 128 300 1.14 1.04, 400 1.03 0.86; 256 140 1.16 1.05, 170 1.05 0.95; 602 100 1.15 1.09, 120 0.98 0.99
//     dist filter 32 600 1.17 1.18; 64 600 0.96 0.96 (1.16 1.11); 128 400 1.10 0.97, 600 0.93 0.88; 256 300 1.09 0.88; 602 140 1.01 1.14, 200 0.98 0.90
//     both        64 600 1.19 1.20; 128 600 1.09 0.97; 256 300 1.18 0.94, 400 1.03 0.85; 602 140 1.08 1.20, 200 1.06 0.94
// A call over few rows: whole rows take some 100 us however few they are on a power-law graph (a hub's row), not on one with uniform ends.
// Route over whole rows, power-law (uniform) of 130 000 and 240 000 vertices, by rows asked for and entries a row; stream kernel
//   64 columns 8000 of 80 0.66 0.69 (1.04 1.02), 16 000 of 100 0.94 0.78 (1.46 1.45), 32 000 of 100 1.04 0.95 (1.07 1.10); 128 8000 of 80 0.65 0.66 (1.03 1.08), 32 000 of
//   100 0.98 0.89 (1.00 1.12); 256 8000 of 100 0.80 0.54 (1.56 1.61), of 140 0.73 0.59 (1.22 1.34), 32 000 of 100 1.11 1.07 (1.09 1.24); 602 8000 of 100 0.82 0.45 (1.44
//   1.55); a factor, 64 16 000 of 140 1.02 0.96 (1.91 1.93), 256 8000 of 100 1.02 0.69 (1.77 1.80)
// fours 32 columns 32 000 of 120 0.92 0.88 (1.08 1.07); 64 32 000 of 80 0.98 0.75 (0.86 0.91); a factor, 32 32 000 of 120 0.98 0.97 (1.20 1.21); 64 32 000 of 100 0.96 0.90
//   (1.06 1.13).  Rows of 32 bytes gain little (16 columns, 10 800 rows of 150 0.90) and lose more (9400 of 136, uniform, 2.2): as calls over many
// rows.  With a dist filter uniform ends lose more by the route (2 to 3 times up to 200 entries) than power-law graphs gain: one line.
constexpr int32_t kBlockedFewRows = 20000, kBlockedSomeRows = 48000;

static int blocked_min_segment(bool f32, bool fours, bool filter, bool scaled, int32_t n_active, int32_t F) {
    if (f32) return 8;
    constexpr int kNever = 1 << 20;      // no length measured, up to 600 entries, was faster
    const int width = F <= 32 ? 0 : F <= 64 ? 1 : F <= 128 ? 2 : F <= 256 ? 3 : 4;
    static const int filtered[2][2][5] = {{{kNever, 80, 52, 40, 22}, {kNever, kNever, 76, 48, 24}}, {{80, 32, 36, 26, 17}, {kNever, 64, 72, 28, 17}}};
    static const int line[3][2][2][5] = {{{{8, 8, 8, 13, 12}, {25, 17, 17, 13, 12}}, {{13, 8, 8, 8, 8}, {17, 14, 17, 8, 8}}},
                                         {{{21, 12, 12, 13, 12}, {kNever, kNever, 21, 19, 12}}, {{13, 8, 8, 8, 8}, {17, 14, 17, 8, 8}}},
                                         {{{48, 40, 22, 17, 14}, {kNever, kNever, 48, 21, 15}}, {{15, 10, 16, 13, 10}, {64, 32, 20, 13, 10}}}};
    if (filter) return filtered[fours][scaled][width];
    return line[F <= 16 ? 2 : n_active <= kBlockedFewRows ? 0 : n_active <= kBlockedSomeRows ? 1 : 2][fours][scaled][width];
}

// Streams of fours or the stream kernel, for a call without a row list.  The fours pay for a copy of the gathered rows (without a neighbour
// scale or in bfloat16 the stream kernel makes none) and take chunks of at least 16 rows, of which short calls fill no stage; what
// they save grows with the call's entries, and least of all where the stream kernel has a single slab and stages its ids once, too.  Rows that one
// line holds are half a slab of the stream kernel.  us, stream / fours, power-law graphs and, in brackets, uniform ends, by rows asked for:
//   fp32, 256 columns: 233 000 ids, 490 entries a row, 4096 rows 185 / 289, 16 000 502 / 572, 32 000 957 / 916, 64 000 1842 / 1631; 150 000 ids,
//     160 entries, 4096 94 / 170, 32 000 433 / 476, 64 000 799 / 750 (400 entries, 4096 136 / 165, 16 000 394 / 414, 32 000 777 / 734)
//     with a neighbour scale: 490 entries 4096 291 / 289, 64 000 1928 / 1631; 160 4096 149 / 171, 32 000 486 / 476 (400, 4096 191 / 168)
//   fp32, 64 columns: 150 000 ids, 160 entries, 16 000 84 / 107, 64 000 218 / 221, all 502 / 438 (233 000 ids, 100 entries, 64 000 201 / 185)
//   bf16, 256 columns: 490 entries 4096 128 / 152, 32 000 605 / 534; 160 8000 109 / 164, 32 000 315 / 289; scaled 490 8000 251 / 280, 16 000 436 / 411
//   one line, 490 entries: bf16, 64 columns 4096 84 / 70, scaled 120 / 81; (100 entries, 8000 54 / 71, 32 000 106 / 96, scaled 8000 68 / 81, 16 000 98 / 88).
// Over 1780 calls (70 000 to 400 000 ids, 100 to 490 entries, 32 to 602 columns, 4096 rows to all) the lines below are 1.01 times as slow
// as the faster form on average and 1.24 at most; fours for all of them 1.21 (fp32), 1.05 (scaled), 1.14 and 1.10 (bf16), up to 2.7.
// Two passes have twice the segments: fp32, 256 columns, 300 000 ids of 140 32 000 rows 0.79 (stream over fours), 64 000 0.94, 128 000 1.07; 500 000 64 000 0.89,
// 128 000 1.05; bf16 32 000 0.91, 64 000 1.04; 32 columns 16 000 0.88, 32 000 1.06: twice the lines.
static bool fours_pay(int64_t n_active, int64_t avg_row, int64_t n_src, int64_t row_bytes_used, int passes, bool f32, bool scaled) {
    const int64_t rows = n_active / passes, entries = rows * avg_row;
    if (row_bytes_used <= kFourBytes) return entries >= (scaled ? 1000000 : 2000000);
    if (f32 && row_bytes_used <= kSlabBytes) return rows >= n_src / (scaled ? 6 : 3) && entries >= (scaled ? 4000000 : 6000000);
    return rows >= n_src / (scaled ? 16 : 10) && entries >= (scaled ? 4000000 : 6000000);
}

static BlockedPlan plan_blocked(const gnn_csr* g, bool listed, bool copies, int32_t n_active, int32_t F, int64_t row_bytes, bool vec_ok, bool filter,
                                bool scaled, bool f32, int32_t src_prefix) {
    BlockedPlan p;
    // with a source prefix only the rows [0, src_prefix) of the gathered matrix are ever read
    const int32_t n_src = (src_prefix >= 0 && src_prefix < g->n_cols) ? src_prefix : g->n_cols;
    // the stream kernel addresses the gathered matrix with 32-bit offsets in 16-byte units: 64 GB at most
    if ((int64_t)g->n_cols * row_bytes >= ((int64_t)1 << 36)) return p;
    if (!vec_ok || !(g->flags & GNN_CSR_SORTED_COLUMNS) || g->n_rows <= 0 || n_active < 4096) return p;
    if (g->edge_keep != nullptr) return p;  // the per-layer edge mask is only known to the one-launch route
    const int64_t slab = (int64_t)n_src * kSlabBytes;
    if (slab < (int64_t)GNN_SPMM_BLOCKED_MIN_SLAB) return p;
    const int passes = (int)((slab + kDies * (int64_t)GNN_SPMM_DIE_BYTES - 1) / (kDies * (int64_t)GNN_SPMM_DIE_BYTES));
    const int n_blocks = kDies * passes;
    // average kept length of a row: its entries spread over the id range like the vertices do
    const int64_t avg_row = (int64_t)((double)g->nnz / g->n_rows * ((double)n_src / g->n_cols));
    // Streams of fours: not for a row list, which may name a row twice (how many entries it has is not known here).
    p.fours = !listed && n_blocks <= kMaxFourBlocks && fours_pay(n_active, avg_row, n_src, (int64_t)F * (f32 ? 4 : 2), passes, f32, scaled);
    if (avg_row < (int64_t)blocked_min_segment(f32, p.fours, filter, scaled, n_active, F) * n_blocks) return p;
    p.fours = p.fours && copies;
    if (!die_mapping_holds()) return p;     // workgroup i is not on die i mod 8 here: the route has lost its reason
    p.passes = passes;
    p.n_blocks = n_blocks;
    const int64_t avg_seg = avg_row / n_blocks;
    p.off32 = (int64_t)g->n_cols * row_bytes < ((int64_t)1 << 32);
    p.limit = n_src;
    p.ldp = ((int64_t)F + 7) / 8 * 8;
    p.seg_bytes = (size_t)n_active * (n_blocks + 1) * sizeof(int32_t);
    p.part_bytes = (size_t)kDies * n_active * p.ldp * sizeof(float);
    // A neighbour scale: fp32 gathers from a copy of the matrix with scaled rows (one rounding more per element,
    // far inside the fp32 tolerance); bf16 would lose too much in a rounded copy and keeps a factor per edge.
    const int64_t rows = (p.fours ? kFourEdges : kStreamWgEdges) / std::max<int64_t>(avg_seg, 1), cap = (int64_t)n_active * kDies / 4096;
    p.rows_per_wg = (int32_t)std::min<int64_t>(std::max<int64_t>(std::min(rows, cap), 16), p.fours ? kFourMaxRows : kStreamMaxRows);
    if (p.fours) {
        const int64_t n_chunks = ((int64_t)n_active + p.rows_per_wg - 1) / p.rows_per_wg;
        p.at_bytes = (size_t)(n_chunks * n_blocks) * sizeof(uint2);
        p.places = four_places(g->nnz, n_active, n_chunks, n_blocks);
        p.before_bytes = (size_t)(n_chunks * n_blocks) * kFourGroups * sizeof(uint16_t);
        if (scaled && !f32) p.w_bytes = p.places * 32 * sizeof(float4);
    }
    if (filter || (scaled && !f32 && !p.fours)) {
        p.end_bytes = (size_t)n_active * n_blocks * sizeof(int32_t);
        p.ids_bytes = (size_t)g->nnz * sizeof(int32_t);
    }
    if (p.fours) p.xs_bytes = (size_t)(((int64_t)F * (f32 ? 4 : 2) + kFourBytes - 1) / kFourBytes) * n_src * kFourBytes;
    else if (scaled && f32) p.xs_bytes = (size_t)n_src * (size_t)row_bytes;
    if (scaled && !f32 && !p.fours) p.w_bytes = (size_t)g->nnz * sizeof(float);
    p.bounds_bytes = ((size_t)n_blocks + 1) * sizeof(int32_t);
    p.sample_bytes = (size_t)kBoundSamples * (filter ? 2 : 1) * sizeof(uint16_t);
    p.n_rows = g->n_rows;
    p.n_cols = g->n_cols;
    return p;
}

// Bytes of the arrays that run_blocked lays out.
static size_t blocked_bytes(const BlockedPlan& p) {
    if (p.passes == 0) return 0;
    WsCarver measure(nullptr);
    measure.take<char>(p.seg_bytes);
    measure.take<char>(p.part_bytes);
    if (p.end_bytes) {
        measure.take<char>(p.end_bytes);
        measure.take<char>(p.ids_bytes);
    }
    if (p.xs_bytes) measure.take<char>(p.xs_bytes);
    if (p.w_bytes) measure.take<char>(p.w_bytes);
    measure.take<char>(p.at_bytes);
    measure.take<uint2>(p.places * 32);
    measure.take<uint32_t>(p.places);
    measure.take<char>(p.before_bytes);
    measure.take<char>(p.bounds_bytes);
    measure.take<char>(p.sample_bytes);
    return measure.used;
}

template <int DT, bool FILTER>
static int32_t run_blocked(const SpmmArgs& a, const BlockedPlan& p, void* ws, hipStream_t stream) {
    constexpr int VE = DT == GNN_F32 ? 4 : 8;
    WsCarver carve(ws);
    int32_t* seg = carve.take<int32_t>(p.seg_bytes / sizeof(int32_t));
    float* part = carve.take<float>(p.part_bytes / sizeof(float));
    const bool prescale = a.nbr_scale != nullptr && DT == GNN_F32, per_edge = a.nbr_scale != nullptr && DT != GNN_F32;
    const bool prepare = FILTER || (per_edge && !p.fours);
    int32_t* seg_end = prepare ? carve.take<int32_t>(p.end_bytes / sizeof(int32_t)) : nullptr;
    int32_t* ids = prepare ? carve.take<int32_t>(p.ids_bytes / sizeof(int32_t)) : nullptr;
    char* xs = p.xs_bytes ? carve.take<char>(p.xs_bytes) : nullptr;
    float* edge_w = per_edge ? carve.take<float>(p.w_bytes / sizeof(float)) : nullptr;
    FourArgs f = {};
    f.at = carve.take<uint2>(p.at_bytes / sizeof(uint2));
    f.stream = carve.take<uint2>(p.places * 32);
    f.ends = carve.take<uint32_t>(p.places);
    f.before = carve.take<uint16_t>(p.before_bytes / sizeof(uint16_t));
    int32_t* bounds = carve.take<int32_t>(p.bounds_bytes / sizeof(int32_t));
    uint16_t* bins = carve.take<uint16_t>(p.sample_bytes / sizeof(uint16_t));
    const int32_t* dist = FILTER ? a.dist : nullptr;
    spmm_samples_kernel<<<kBoundSamples / 256, 256, 0, stream>>>(a.row_ptr, a.col_idx, a.rows ? p.n_rows : a.n_active, dist, a.max_dist, p.limit, bins);
    GNN_LAUNCH_CHECK("spmm_samples_kernel");
    spmm_bounds_kernel<<<1, 1024, 0, stream>>>(bins, dist != nullptr, p.limit, p.n_blocks, bounds);
    GNN_LAUNCH_CHECK("spmm_bounds_kernel");
    spmm_seg_kernel<<<grid_for((int64_t)a.n_active * (p.n_blocks + 1), 256, 1 << 16), 256, 0, stream>>>(
        a.row_ptr, a.col_idx, a.rows, a.n_active, p.n_blocks, bounds, p.limit, p.n_cols, seg);
    GNN_LAUNCH_CHECK("spmm_seg_kernel");
    SpmmArgs b = a;
    if (prescale && !p.fours) {
        // the neighbour scale is applied once per row of the gathered matrix, not once per edge and slab
        spmm_scale_rows_kernel<DT><<<grid_for((int64_t)p.limit * ((a.F + VE - 1) / VE), 256, 1 << 16), 256, 0, stream>>>(
            a.X, a.ldx, p.limit, a.F, a.nbr_scale, xs);
        GNN_LAUNCH_CHECK("spmm_scale_rows_kernel");
        b.X = xs;
        b.nbr_scale = nullptr;
    }
    if (prepare) {
        const int64_t n_segments = (int64_t)a.n_active * p.n_blocks;
        spmm_prepare_kernel<<<grid_for(n_segments * 16, 256, 1 << 18), 256, 0, stream>>>(
            a.col_idx, seg, FILTER ? a.dist : nullptr, a.max_dist, per_edge && !p.fours ? a.nbr_scale : nullptr, n_segments, p.n_blocks, ids,
            edge_w, seg_end);
        GNN_LAUNCH_CHECK("spmm_prepare_kernel");
        b.col_idx = ids;
        b.seg_end = seg_end;
        b.edge_w = edge_w;
        b.dist = nullptr;
    }
    b.seg = seg;
    b.n_blocks = p.n_blocks;
    b.Y = part;
    b.ldy = p.ldp;
    b.out_scale = nullptr;
    if (p.fours) {
        f.row_ptr = a.row_ptr; f.ids = b.col_idx; f.seg = seg; f.seg_end = b.seg_end; f.bounds = bounds;
        f.n_active = a.n_active; f.n_blocks = p.n_blocks; f.rows_per_wg = p.rows_per_wg;
        f.X = a.X; f.ldx = a.ldx; f.F = a.F; f.n_src = p.limit; f.slabs = xs;
        f.nbr_scale = a.nbr_scale; f.w = (float4*)edge_w;
        f.part = part; f.ldp = p.ldp;
        const unsigned n_chunks = (unsigned)(((int64_t)a.n_active + p.rows_per_wg - 1) / p.rows_per_wg);
        if (per_edge) spmm_fours_kernel<true><<<n_chunks * (unsigned)p.n_blocks, 256, 0, stream>>>(f);
        else spmm_fours_kernel<false><<<n_chunks * (unsigned)p.n_blocks, 256, 0, stream>>>(f);
        GNN_LAUNCH_CHECK("spmm_fours_kernel");
        constexpr int W = kFourBytes / (DT == GNN_F32 ? 4 : 2);
        spmm_slabs_kernel<DT><<<grid_for((int64_t)p.limit * ((a.F + W - 1) / W * 8), 256, 1 << 16), 256, 0, stream>>>(f);
        GNN_LAUNCH_CHECK("spmm_slabs_kernel");
        const dim3 grid(n_chunks * kDies, (unsigned)((a.F + W - 1) / W));
        for (int pass = 0; pass < p.passes; ++pass) {
            f.block0 = pass * kDies;
            f.accumulate = pass > 0;
            if (DT != GNN_F32 && per_edge) spmm_four_sums_kernel<DT, DT != GNN_F32><<<grid, 256, 0, stream>>>(f);
            else spmm_four_sums_kernel<DT, false><<<grid, 256, 0, stream>>>(f);
            GNN_LAUNCH_CHECK("spmm_four_sums_kernel");
        }
    } else {
        b.rows_per_group = p.rows_per_wg;
        for (int pass = 0; pass < p.passes; ++pass) {
            b.block0 = pass * kDies;
            b.accumulate = pass > 0;
            GNN_CHECK((launch_stream<DT, VE, kSlabBytes / 16>(b, p.off32, stream)));
        }
    }
    spmm_sum_parts_kernel<DT><<<grid_for((int64_t)a.n_active * ((a.F + 3) / 4), 256, 1 << 16), 256, 0, stream>>>(
        part, p.ldp, a.rows, a.n_active, a.F, a.Y, a.ldy, a.out_scale, a.accumulate, a.relu_h, a.ldh);
    GNN_LAUNCH_CHECK("spmm_sum_parts_kernel");
    return GNN_OK;
}

// The split route's shape for one call; n_chunks == 0: the route does not apply.
struct SplitPlan {
    int64_t n_chunks = 0, n_parts = 0;
    int32_t n_slabs = 0, n_nbr = 0;
};

// Where the line lies (power-law graphs, call with / without the route, us): what the route costs - moving the entries once, a
// part written and read once per row - has to be made up for by the rows' hot entries, so it takes long rows
//   256 columns: 2.4 M rows of 12 4385 / 4232, of 25 8190 / 8158; 1 M of 24 2796 / 3118, of 50 5311 / 6492; 400 k of 120 4277 / 6243
// of several cache lines
//   1 M rows of 50: 48 columns 1591 / 1403, 64 1890 / 2045, 100 2730 / 3124, 128 3100 / 3927, 602 14129 / 16556
//   300 k rows of 50: 48 465 / 374, 64 492 / 449, 100 759 / 847, 128 807 / 981, 602 3201 / 4796
// in fp32 (bf16 parts are floats all the same: 1 M rows of 50, 256 columns 3565 / 3052, 512 columns 6752 / 6687), out of a matrix
// that the L2s of all dies (32 MB) do not hold
//   100 k rows of 60: 100 columns 285 / 298, 256 494 / 671.
// The neighbours are looked through and the table is copied however few rows a call asks for, and a source prefix shortens the rows, so
// the call's own share counts (1.2 M rows of 51; a call over the first rows, in random order / numbered by distance, where they are the longer ones)
//   256 columns: 0.4 % of the rows (0.25 GB) 222 / 221, 331 / 378; 1 % 283 / 332, 477 / 579; 10 % 938 / 1177, 2766 / 3740
//   100 columns: 1 % (0.25 GB) 172 / 163, 301 / 340; 2 % (0.5 GB) 214 / 207, 438 / 536; 5 % 320 / 344, 843 / 1058
//   300 k rows of 51, 128 columns: 5 % (0.39 GB) 120 / 109, 210 / 245; 10 % 154 / 160, 333 / 405
// and of the neighbours (a source prefix; it stands for rows of the forward call, so the numbering by distance decides)
//   256 columns: 5 % 1146 / 1077, 1630 / 1558; 12.5 % (6 entries a row) 1514 / 1435, 3051 / 3567; 25 % (13) 2218 / 2142, 3494 / 4408; 50 % 3660 / 4343, 4479 / 5984
//   100 columns: 25 % 1195 / 1131, 2061 / 2052; 50 % (26) 2162 / 2245, 2573 / 2857
//   300 k rows of 51, 256 columns: 12.5 % 356 / 357, 681 / 681; 25 % 543 / 492, 802 / 860; with 10 % of the rows and 50 % 178 / 156, 372 / 517.
static SplitPlan plan_split(const gnn_csr* g, const int32_t* rows, int32_t n_active, int32_t F, int32_t dtype, int64_t row_bytes, bool vec_ok,
                            bool filter, int32_t cut_id, hipStream_t stream) {
    SplitPlan p;
    if (dtype != GNN_F32 || rows != nullptr || !vec_ok || filter || n_active < 4096 || F <= 3 * kSplitCols) return p;
    const int32_t n_src = cut_id >= 0 ? cut_id : g->n_cols;
    if (g->nnz / g->n_rows < 40 || n_src * row_bytes < (48ll << 20) || g->nnz * row_bytes < (1ll << 30)) return p;
    const double row_share = (double)n_active / g->n_rows, src_share = (double)n_src / g->n_cols;
    if ((double)g->nnz / g->n_rows * src_share < (F > 4 * kSplitCols ? 6 : 20)) return p;
    if ((double)g->nnz * row_bytes * row_share * src_share * src_share < 4e8) return p;
    p.n_nbr = n_src < g->n_rows ? n_src : g->n_rows;
    p.n_chunks = (g->nnz + kSplitChunk - 1) / kSplitChunk;
    p.n_slabs = (F + kSplitCols - 1) / kSplitCols;
    p.n_parts = (int64_t)n_active + p.n_chunks * (kSplitGroups + 1);
    if (p.n_parts > INT32_MAX || !die_mapping_holds(&stream)) p.n_chunks = 0;
    return p;
}

// Lays the route's arrays out; with base == nullptr it only measures.
static SplitArgs carve_split(const SplitPlan& p, int32_t n_active, WsCarver& carve, size_t* decision = nullptr) {
    SplitArgs s = {};
    s.hist = carve.take<int32_t>((size_t)kSplitBlocks * kSplitBins);
    s.hits = carve.take<int32_t>(kSplitSampleBlocks);
    if (decision) *decision = carve.used + sizeof(int32_t);      // ctrl[1]
    s.ctrl = carve.take<int32_t>(2);
    s.first_row = carve.take<int32_t>(p.n_chunks + 1);
    s.slot = carve.take<uint2>(((size_t)p.n_nbr + 31) / 32);
    s.hot = carve.take<int32_t>(kSplitSlots + 1);
    s.table = carve.take<float>((size_t)p.n_slabs * (kSplitSlots + 1) * kSplitCols);
    s.stream = carve.take<uint16_t>((size_t)p.n_chunks * kSplitStage);
    s.ends = carve.take<uint64_t>((size_t)p.n_chunks * kSplitQuadWords);
    s.before = carve.take<uint16_t>((size_t)p.n_chunks * kSplitGroups);
    s.cold = carve.take<int32_t>((size_t)p.n_chunks * kSplitChunk);
    s.rows = carve.take<SplitRow>(n_active);
    s.chunks = carve.take<SplitChunk>(p.n_chunks);
    s.plane = carve.take<float>((size_t)p.n_slabs * p.n_parts * kSplitCols);
    return s;
}

static int32_t run_split(const SpmmArgs& a, const SplitPlan& p, void* ws, hipStream_t stream) {
    WsCarver carve(ws);
    SplitArgs s = carve_split(p, a.n_active, carve);
    s.row_ptr = a.row_ptr; s.col_idx = a.col_idx; s.n_active = a.n_active;
    s.n_nbr = p.n_nbr; s.limit = a.cut_id >= 0 ? a.cut_id : INT32_MAX;
    s.n_chunks = p.n_chunks; s.n_parts = p.n_parts; s.n_slabs = p.n_slabs;
    s.X = a.X; s.ldx = a.ldx; s.F = a.F; s.nbr_scale = a.nbr_scale;
    split_degrees_kernel<<<kSplitBlocks, 1024, 0, stream>>>(s);
    GNN_LAUNCH_CHECK("split_degrees_kernel");
    split_assign_kernel<<<kSplitBlocks, 1024, 0, stream>>>(s);
    GNN_LAUNCH_CHECK("split_assign_kernel");
    split_table_kernel<<<kSplitTableBlocks + kSplitSampleBlocks, 256, 0, stream>>>(s);
    GNN_LAUNCH_CHECK("split_table_kernel");
    if (a.cut_id >= 0) split_entries_kernel<true><<<(unsigned)p.n_chunks, 1024, 0, stream>>>(s);
    else split_entries_kernel<false><<<(unsigned)p.n_chunks, 1024, 0, stream>>>(s);
    GNN_LAUNCH_CHECK("split_entries_kernel");
    const int64_t per_die = (p.n_chunks * p.n_slabs + kDies - 1) / kDies;
    split_sum_kernel<<<(unsigned)(per_die * kDies), 256, 0, stream>>>(s);
    GNN_LAUNCH_CHECK("split_sum_kernel");
    SpmmArgs b = a;
    b.split_on = s.ctrl + 1; b.split_cold = s.cold; b.split_rows = s.rows; b.split_chunks = s.chunks;
    b.split_plane = s.plane; b.split_ld = (int64_t)p.n_slabs * kSplitCols;
    if (a.F <= 128) return launch_rows<GNN_F32, 4, 32, 1, false, true>(b, stream);
    if (a.F <= 256) return launch_rows<GNN_F32, 4, 64, 1, false, true>(b, stream);
    if (a.F <= 512) return launch_rows<GNN_F32, 4, 64, 2, false, true>(b, stream);
    return launch_rows<GNN_F32, 4, 64, 3, false, true>(b, stream);
}

template <int DT, bool FILTER>
static int32_t dispatch(const SpmmArgs& a, bool vec_ok, hipStream_t stream) {
    constexpr int VE = DT == GNN_F32 ? 4 : 8;
    const int F = a.F;
    // any alignment / leading dimension: element-wise lanes, 256 columns per workgroup
    if (!vec_ok) return launch_rows<DT, 1, 64, 4, FILTER>(a, stream);
    // Narrow outputs (class scores, a layer in the exchanged order).  A tile of the row kernel is as long as the lanes
    // that span a row, and a short tile pays the per-tile work (staging, ballots, row claims) for few neighbours: rows
    // narrower than 16 vectors of 16 bytes keep their 16 lanes and 16-neighbour tiles and take fewer bytes per lane
    // instead (measured on 64-byte rows: 8 lanes x 16 bytes 2.45 ms, 16 lanes x 4 bytes 1.81 ms).
    if (DT == GNN_BF16) {
        if (F <= 16) return launch_rows<GNN_BF16, 1, 16, 1, FILTER>(a, stream);
        if (F <= 32) return launch_rows<GNN_BF16, 2, 16, 1, FILTER>(a, stream);
        if (F <= 64) return launch_rows<GNN_BF16, 4, 16, 1, FILTER>(a, stream);
    } else {
        if (F <= 16) return launch_rows<GNN_F32, 1, 16, 1, FILTER>(a, stream);
        if (F <= 32) return launch_rows<GNN_F32, 2, 16, 1, FILTER>(a, stream);
    }
    if (F <= 16 * VE) return launch_rows<DT, VE, 16, 1, FILTER>(a, stream);
    if (F <= 32 * VE) return launch_rows<DT, VE, 32, 1, FILTER>(a, stream);
    if (F <= 64 * VE) return launch_rows<DT, VE, 64, 1, FILTER>(a, stream);
    if (F <= 128 * VE) return launch_rows<DT, VE, 64, 2, FILTER>(a, stream);
    return launch_rows<DT, VE, 64, 3, FILTER>(a, stream);
}

static int32_t spmm_common(const gnn_csr* g, const char* gname, const int32_t* rows, int32_t n_active, const int32_t* dist,
                           int32_t max_dist, int32_t src_prefix, const void* X, int64_t ldx, void* Y, int64_t ldy, int32_t F, int32_t dtype,
                           const float* out_scale, const float* nbr_scale, int32_t accumulate, const void* relu_h, int64_t ldh,
                           void* ws, size_t* ws_bytes, hipStream_t stream, const float* start_bias = nullptr) {
    GNN_CHECK(check_csr(g, gname));
    GNN_REQUIRE(n_active >= 0, GNN_ERR_INVALID_ARG, "negative row count");
    GNN_REQUIRE(rows != nullptr || n_active <= g->n_rows, GNN_ERR_SHAPE, "n_active %d exceeds n_rows %d", n_active, g->n_rows);
    GNN_REQUIRE(dtype == GNN_F32 || dtype == GNN_BF16, GNN_ERR_UNSUPPORTED, "unknown dtype %d", dtype);
    GNN_REQUIRE(F >= 0, GNN_ERR_INVALID_ARG, "F < 0");
    GNN_REQUIRE(ldx >= F && ldy >= F, GNN_ERR_SHAPE, "leading dimension smaller than F = %d", F);
    const int ve = dtype == GNN_F32 ? 4 : 8;
    GNN_REQUIRE(relu_h == nullptr || ldh >= F, GNN_ERR_SHAPE, "ld_relu smaller than F = %d", F);
    const bool vec_ok = ((uintptr_t)X % 16 == 0) && ((uintptr_t)Y % 16 == 0) && ldx % ve == 0 && ldy % ve == 0 &&
                        (relu_h == nullptr || ((uintptr_t)relu_h % 16 == 0 && ldh % ve == 0));
    GNN_REQUIRE(src_prefix >= -1, GNN_ERR_INVALID_ARG, "src_prefix %d: -1 or a vertex count", src_prefix);
    // A source prefix that leaves something out: rows sorted by column are cut at that id (no test per entry), rows in
    // any order get the test in the filter.
    const bool use_prefix = src_prefix >= 0 && src_prefix < g->n_cols;
    const bool sorted = (g->flags & GNN_CSR_SORTED_COLUMNS) != 0;
    const int32_t cut_id = (use_prefix && sorted) ? src_prefix : -1, id_limit = (use_prefix && !sorted) ? src_prefix : -1;
    const bool filter = dist != nullptr || g->edge_keep != nullptr || id_limit >= 0;
    BlockedPlan plan;
    SplitPlan split;
    if (ws_bytes != nullptr) {
        auto blocked = [&](bool copies) {
            return plan_blocked(g, rows != nullptr, copies, n_active, F, ldx * (dtype == GNN_F32 ? 4 : 2), vec_ok, filter, nbr_scale != nullptr,
                                dtype == GNN_F32, cut_id);
        };
        if (n_active > 0 && F > 0) plan = blocked(true);
        size_t need = blocked_bytes(plan);
        if (plan.fours && ws != nullptr && *ws_bytes < need) {
            // no room for the copy of the rows and the streams: the stream kernel makes none
            plan = blocked(false);
            need = blocked_bytes(plan);
        }
        if (plan.passes == 0 && n_active > 0 && F > 0) {
            split = plan_split(g, rows, n_active, F, dtype, ldx * (dtype == GNN_F32 ? 4 : 2), vec_ok, filter, cut_id, stream);
            if (split.n_chunks > 0) {
                WsCarver wanted(nullptr);
                carve_split(split, n_active, wanted);
                if (ws == nullptr) need = wanted.used;                      // asked for
                else if (*ws_bytes < wanted.used) split.n_chunks = 0;       // the row kernel needs none
            }
        }
        bool query_only = false;
        GNN_CHECK(ws_protocol(ws, ws_bytes, need, &query_only));
        if (query_only) return GNN_OK;
    }
    if (n_active == 0 || F == 0) return GNN_OK;
    GNN_REQUIRE(X != nullptr && Y != nullptr, GNN_ERR_INVALID_ARG, "X or Y is NULL");
    if (start_bias != nullptr) {
        // no self term under the sum (GCN in the exchanged order): the listed rows start from the bias
        const int grid = grid_for((int64_t)n_active * F, 256, 1 << 14);
        if (dtype == GNN_F32) spmm_bias_rows_kernel<GNN_F32><<<grid, 256, 0, stream>>>(rows, n_active, start_bias, Y, ldy, F);
        else spmm_bias_rows_kernel<GNN_BF16><<<grid, 256, 0, stream>>>(rows, n_active, start_bias, Y, ldy, F);
        GNN_LAUNCH_CHECK("spmm_bias_rows_kernel");
    }

    SpmmArgs a;
    a.row_ptr = g->row_ptr; a.col_idx = g->col_idx; a.rows = rows; a.n_active = n_active;
    a.X = X; a.ldx = ldx; a.Y = Y; a.ldy = ldy; a.F = F;
    a.out_scale = out_scale; a.nbr_scale = nbr_scale; a.dist = dist; a.max_dist = dist ? max_dist : INT32_MAX;
    a.edge_keep = g->edge_keep;
    a.cut_id = cut_id; a.id_limit = id_limit;
    a.accumulate = accumulate;
    a.relu_h = relu_h; a.ldh = ldh;
    a.rows_per_group = 1;
    {
        const int64_t row_bytes = ldx * (dtype == GNN_F32 ? 4 : 2);
        const bool small = g->n_cols < (1 << 24) && row_bytes < (1 << 24) && (int64_t)g->n_cols * row_bytes < ((int64_t)1 << 32);
        a.x_row_bytes = small ? (uint32_t)row_bytes : 0u;
    }
    a.seg = nullptr; a.seg_end = nullptr; a.edge_w = nullptr; a.n_blocks = 0; a.block0 = 0;
    a.split_on = nullptr; a.split_cold = nullptr; a.split_rows = nullptr; a.split_chunks = nullptr; a.split_plane = nullptr; a.split_ld = 0;

    if (plan.passes > 0) {
        if (dtype == GNN_F32) return filter ? run_blocked<GNN_F32, true>(a, plan, ws, stream) : run_blocked<GNN_F32, false>(a, plan, ws, stream);
        return filter ? run_blocked<GNN_BF16, true>(a, plan, ws, stream) : run_blocked<GNN_BF16, false>(a, plan, ws, stream);
    }
    if (split.n_chunks > 0) return run_split(a, split, ws, stream);
    if (dtype == GNN_F32) return filter ? dispatch<GNN_F32, true>(a, vec_ok, stream) : dispatch<GNN_F32, false>(a, vec_ok, stream);
    return filter ? dispatch<GNN_BF16, true>(a, vec_ok, stream) : dispatch<GNN_BF16, false>(a, vec_ok, stream);
}

}  // namespace gnnhot

using namespace gnnhot;

extern "C" int32_t gnn_spmm_route(const gnn_csr* g, const int32_t* rows, int32_t n_active, const void* X, int64_t ldx, const void* Y, int64_t ldy,
                                  int32_t F, int32_t dtype, int32_t scaled, int32_t* route_host, int64_t* decision_host, void* stream) {
    GNN_CHECK(check_csr(g, "g"));
    GNN_REQUIRE(route_host != nullptr, GNN_ERR_INVALID_ARG, "route_host is NULL");
    GNN_REQUIRE(n_active >= 0 && F >= 0 && (rows != nullptr || n_active <= g->n_rows), GNN_ERR_INVALID_ARG, "negative or too many rows, or F < 0");
    GNN_REQUIRE(dtype == GNN_F32 || dtype == GNN_BF16, GNN_ERR_UNSUPPORTED, "unknown dtype %d", dtype);
    const int ve = dtype == GNN_F32 ? 4 : 8;
    const bool vec_ok = (uintptr_t)X % 16 == 0 && (uintptr_t)Y % 16 == 0 && ldx % ve == 0 && ldy % ve == 0, filter = g->edge_keep != nullptr;
    const int64_t row_bytes = ldx * (16 / ve);
    *route_host = 0;
    if (n_active == 0 || F == 0) return GNN_OK;
    if (plan_blocked(g, rows != nullptr, true, n_active, F, row_bytes, vec_ok, filter, scaled != 0, dtype == GNN_F32, -1).passes > 0) {
        *route_host = 1;
        return GNN_OK;
    }
    const SplitPlan p = plan_split(g, rows, n_active, F, dtype, row_bytes, vec_ok, filter, -1, (hipStream_t)stream);
    if (p.n_chunks > 0) {
        WsCarver carve(nullptr);
        size_t decision = 0;
        carve_split(p, n_active, carve, &decision);
        *route_host = 2;
        if (decision_host) *decision_host = (int64_t)decision;
    }
    return GNN_OK;
}

extern "C" int32_t gnn_die_mapping(int32_t* xcc_ids_host, int32_t n_ids, int32_t* holds_host) {
    GNN_REQUIRE(n_ids >= 0 && (xcc_ids_host != nullptr || n_ids == 0), GNN_ERR_INVALID_ARG, "xcc_ids_host is NULL");
    int32_t ids[kProbeX * kProbeY];
    GNN_CHECK(probe_die_ids(ids));
    for (int i = 0; i < n_ids && i < kProbeX * kProbeY; ++i) xcc_ids_host[i] = ids[i];
    if (holds_host != nullptr) *holds_host = die_ids_round_robin(ids) ? 1 : 0;
    return GNN_OK;
}

extern "C" int32_t gnn_masked_spmm_fwd(const gnn_csr* g, const int32_t* rows, int32_t n_active, const void* X, int64_t ldx,
                                       void* Y, int64_t ldy, int32_t F, int32_t dtype, const float* row_scale,
                                       const float* col_scale, void* ws, size_t* ws_bytes, void* stream) {
    return spmm_common(g, "g", rows, n_active, nullptr, 0, -1, X, ldx, Y, ldy, F, dtype, row_scale, col_scale, 0, nullptr, 0, ws,
                       ws_bytes, (hipStream_t)stream);
}

extern "C" int32_t gnn_masked_spmm_fwd_add(const gnn_csr* g, const int32_t* rows, int32_t n_active, const void* X, int64_t ldx,
                                           void* Y, int64_t ldy, int32_t F, int32_t dtype, const float* row_scale,
                                           const float* col_scale, const float* bias, int32_t relu, void* ws, size_t* ws_bytes,
                                           void* stream) {
    GNN_REQUIRE(relu == 0 || relu == 1, GNN_ERR_INVALID_ARG, "relu must be 0 or 1");
    // the output matrix as its own mask stands for a ReLU of what is stored
    return spmm_common(g, "g", rows, n_active, nullptr, 0, -1, X, ldx, Y, ldy, F, dtype, row_scale, col_scale, 1, relu ? Y : nullptr, ldy, ws,
                       ws_bytes, (hipStream_t)stream, bias);
}

extern "C" int32_t gnn_masked_spmm_bwd(const gnn_csr* gT, const int32_t* out_rows, int32_t n_out, const int32_t* dist,
                                       int32_t max_active_dist, int32_t src_prefix, const void* dY, int64_t lddy, void* dX, int64_t lddx, int32_t F,
                                       int32_t dtype, const float* row_scale, const float* col_scale, int32_t accumulate,
                                       const void* relu_H, int64_t ld_relu, void* ws, size_t* ws_bytes, void* stream) {
    GNN_REQUIRE(accumulate == 0 || accumulate == 1, GNN_ERR_INVALID_ARG, "accumulate must be 0 or 1");
    return spmm_common(gT, "gT", out_rows, n_out, dist, max_active_dist, src_prefix, dY, lddy, dX, lddx, F, dtype, col_scale, row_scale,
                       accumulate, relu_H, ld_relu, ws, ws_bytes, (hipStream_t)stream);
}
