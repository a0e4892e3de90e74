// Extraction of the partition's one-hop graph (paper section 6, figure 7c step 1: the vertices the partition
// depends on are collected outwards from its own vertices; section 5.3.1: the sub-graph is then built on what the
// traversal reached), and the matching gather of the feature rows.
//
// Input is what gnn_build_active_sets leaves for the UNPARTITIONED graph: the traversed vertices in ring order
// (sorted by (distance from the targets, id)) and dist[].  They become the local vertices 0 .. n_local-1 in that
// order, so every per-layer active set R_l of the local graph is a prefix of the numbering (targets first), and the
// local graph keeps every edge of the graph between two traversed vertices (vertex-induced sub-graph).
//
// Mapping to CDNA4.  Integer work: each local row reads its global row once per pass (4 bytes per entry, streaming) and
// makes one random probe per entry - a bit of the traversed set when counting (n / 8 bytes: stays in L2), new_id[] when
// writing.  Because the numbering is (distance, id), local ids of one distance are an interval: the distance of a
// neighbour follows from its local id and the L interval starts (found anew in each pass), and a global row, ascending in
// id, in ascending LOCAL id is the stable partition of its kept entries by distance: no sort, bit-exact.  Rows go by
// length (rowlists.h): sixteen lanes, a wavefront (both hold the whole row in registers and probe once) or a workgroup.
// What bounds it is the random probe of every entry.  Measured, active sets + extraction of a 1M-vertex / 20M-entry
// graph, eight rings: 2.25 -> 0.96 ms; the fill pass alone, 1.54 ms with sixteen lanes on every row and a sweep per
// distance (the tail of the long rows most of it), took 0.24 + 0.15 ms (short + queued rows), and takes 0.14 + 0.13 since the
// workgroups that fill the queues no longer wait for each other's atomics (rowlists.h; the whole 0.90 -> 0.75).
//
// After boundary sampling (gnn_extract_sampled_partition) a target's local row is its KEPT row (the sampler's output,
// addressed through a row_ptr over the full id range, gnn_expand_row_ptr) and an outside vertex's local row is the
// reverse of the kept edges that reach it.  The kernels above run over the targets' kept rows; an entry that leads
// outside also takes part in the transposition: the count pass adds it to the outside vertex's length, the fill pass
// puts the target into the next free place of its row (integer atomics, so in any order), and a last launch orders every
// such row: each entry's place is the number of smaller ones, and of equal ones (a repeated column of a kept row) before it.
// A reverse row of more than kExSortMax entries (or one that the output's capacity cuts) is instead collected in order by a
// workgroup that scans the vertex's row of the transposed graph and keeps the targets whose kept row contains it (binary
// search), as often as it does.  That scan for
// EVERY outside vertex, sixteen lanes each, took 11.7 of the 12.8 ms of sampling and extraction on a 5M-vertex / 75M-entry
// graph with 625 000 targets and fanout 5; now extraction is 0.8 of 1.6 ms.
#include "common.h"
#include "rowlists.h"
#include "scan.h"

namespace gnnhot {

constexpr int kExMaxHops = 30;
constexpr int kExSortMax = 1024;   // reverse rows up to this length are ordered in LDS

struct ExCtrl {
    RowCtrl rows;                      // queues of the rows that are longer than sixteen lanes take
    RowCtrl reverse;                   // ... and of the reverse rows
    int32_t first[kExMaxHops + 2];     // first local vertex at distance d (INT32_MAX: none)
};

struct ExArgs {
    const int32_t* rp;        // rows that are copied: the graph, or the kept rows of the targets
    const int32_t* ci;
    const int32_t* t_rp;      // sampled only: the transposed graph
    const int32_t* t_ci;
    const int32_t* ring_ids;
    int32_t n_local, n, L;
    const int32_t* new_id;
    const uint32_t* bits;     // plain, count pass (nullable): the traversed vertices
    int32_t* counts;          // count pass: row lengths;  sampled, fill pass: next free place of every outside vertex's row
    const int32_t* out_rp;
    int32_t* out_ci;
    int64_t capacity;
    int32_t *medq, *hubq;
    ExCtrl* ctrl;
};

// distance of local vertex `id`: the last interval that starts at or before it (lane d holds the start of interval d)
__device__ __forceinline__ int ex_class(int32_t first, int32_t L, int32_t id) {
    int c = 0;
    for (int d = 1; d <= L; ++d) c = id >= __builtin_amdgcn_readlane(first, d) ? d : c;
    return c;
}

__device__ __forceinline__ int32_t ex_first(const ExArgs& a) { return a.ctrl->first[lane_id() < kExMaxHops + 2 ? lane_id() : 0]; }

// local vertices whose row is copied: all of them, or the targets
template <bool SAMPLED>
__device__ __forceinline__ int32_t ex_rows(const ExArgs& a) {
    if (!SAMPLED) return a.n_local;
    const int32_t t = a.ctrl->first[1];
    return t < a.n_local ? t : a.n_local;
}

template <bool SAMPLED>
__device__ __forceinline__ bool ex_stays(const ExArgs& a, int32_t u, int32_t& id) {
    if (!SAMPLED && a.bits) return (a.bits[u >> 5] >> (u & 31)) & 1u;
    id = a.new_id[u];
    return id >= 0;
}

// First launch of a pass: clears the queues, notes the first local vertex at every distance, numbers the traversed
// vertices (new_id nullable: already there) and starts counts (nullable) at zero or, with out_rp, at the rows' starts.
// A distance's first vertex is the one whose predecessor in ring order lies nearer: every entry of `first` has one
// writer, so nothing has to be cleared before (an extra launch is a tenth of a small extraction).
__global__ __launch_bounds__(256) void ex_number_kernel(const int32_t* __restrict__ ring_ids, int32_t n_local, int32_t n,
                                                        const int32_t* __restrict__ dist, int32_t* __restrict__ new_id,
                                                        int32_t* __restrict__ counts, const int32_t* __restrict__ out_rp, ExCtrl* ctrl) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    auto dist_at = [&](int64_t k) -> int32_t {   // -1: an id outside the graph
        const int32_t v = ring_ids[k];
        return v >= 0 && v < n ? dist[v] : -1;
    };
    constexpr int32_t kQueueWords = 2 * (int32_t)(sizeof(RowCtrl) / sizeof(int32_t));
    if (i < kQueueWords) ((int32_t*)ctrl)[i] = 0;
    const int32_t d = i < n_local ? dist_at(i) : -1;
    int32_t before = __shfl_up(d, 1, kWave);
    if (i >= n_local) return;
    const int32_t v = ring_ids[i];
    if (new_id && v >= 0 && v < n) new_id[v] = (int32_t)i;
    if (counts) counts[i] = out_rp ? out_rp[i] : 0;
    if (lane_id() == 0) before = i > 0 ? dist_at(i - 1) : -1;
    if (d > before) {
        for (int64_t k = i - 1; before < 0 && k >= 0; --k) before = dist_at(k);   // (steps over ids outside the graph)
        for (int32_t c = before + 1; c <= d && c <= kExMaxHops; ++c) ctrl->first[c] = (int32_t)i;
    }
    if (i == n_local - 1) {
        int32_t last = d;
        for (int64_t k = i - 1; last < 0 && k >= 0; --k) last = dist_at(k);
        for (int32_t c = last + 1; c < kExMaxHops + 2; ++c) ctrl->first[c] = INT32_MAX;
    }
}

// bit v = vertex v was traversed (64 vertices per wavefront; both words are written, the second may lie past n)
__global__ __launch_bounds__(256) void ex_bits_kernel(const int32_t* __restrict__ new_id, int32_t n, uint64_t* __restrict__ bits) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t m = __ballot(v < n && new_id[v < n ? v : 0] >= 0);
    if (lane_id() == 0 && v < n) bits[v >> 6] = m;
}

// ---- count pass ----------------------------------------------------------------------------------------------------
template <bool SAMPLED>
__global__ __launch_bounds__(256) void ex_count_kernel(ExArgs a) {
    __shared__ RowLists lists;
    row_lists_init(lists);
    const int lane = lane_id(), sub = lane / kRowLanes, sl = lane % kRowLanes;
    const int grp = (int)threadIdx.x / kRowLanes;
    const int32_t n_rows = ex_rows<SAMPLED>(a);
    RowWalk w{a.ring_ids, a.rp, a.n, n_rows, (int64_t)gridDim.x * kRowsPerWg};
    w.begin((int64_t)blockIdx.x * kRowsPerWg + grp);
    for (int64_t c = blockIdx.x; c * kRowsPerWg < n_rows; c += gridDim.x) {   // uniform over the workgroup
        const int64_t i = c * kRowsPerWg + grp;
        int32_t s = w.s, e = w.e;
        const int32_t after = w.ahead(i);
        const bool is_long = e - s > kRowShort;   // uniform over the 16-lane group
        if (is_long) {
            if (sl == 0) row_lists_push(lists, (int32_t)i, e - s, a.medq, a.hubq, &a.ctrl->rows);
            s = e = 0;
        }
        int32_t u[4], cnt = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t p = (uint32_t)s + r * kRowLanes + sl;   // (past the row's end, a position may not fit an int32_t)
            u[r] = p < (uint32_t)e ? a.ci[p] : -1;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int32_t id = -1;
            const bool keep = u[r] >= 0 && ex_stays<SAMPLED>(a, u[r], id);
            cnt += __popc(group_ballot(keep, sub));
            if (SAMPLED && keep && id >= n_rows) atomicAdd(&a.counts[id], 1);
        }
        if (sl == 0 && i < n_rows && !is_long) a.counts[i] = cnt;
        w.next(after);
    }
    row_lists_flush(lists, a.medq, a.hubq, &a.ctrl->rows);
}

// Entries of a queued row that stay: NW wavefronts (1 or 4) per row, eight entries per lane and step.  Every lane of the
// row's wavefronts returns its wavefront's share.
template <bool SAMPLED, int NW>
__device__ __forceinline__ int32_t ex_count_row(const ExArgs& a, int32_t v, int32_t n_rows) {
    const int32_t s = a.rp[v], e = a.rp[v + 1];
    int32_t cnt = 0;
    for (int64_t base = s; base < e; base += NW * kWave * 8) {
        int32_t u[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t p = base + r * (NW * kWave) + (NW == 1 ? lane_id() : (int)threadIdx.x);
            u[r] = p < e ? a.ci[p] : -1;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            int32_t id = -1;
            const bool keep = u[r] >= 0 && ex_stays<SAMPLED>(a, u[r], id);
            cnt += __popcll(__ballot(keep));
            if (SAMPLED && keep && id >= n_rows) atomicAdd(&a.counts[id], 1);
        }
    }
    return cnt;
}

// the queued rows: first those a wavefront takes, then those a workgroup takes
template <bool SAMPLED>
__global__ __launch_bounds__(256) void ex_count_long_kernel(ExArgs a) {
    __shared__ int32_t s_cnt[4];
    const int wave = (int)(threadIdx.x >> 6);
    const int32_t n_rows = ex_rows<SAMPLED>(a), n_medium = a.ctrl->rows.n_medium, n_hub = a.ctrl->rows.n_hub;
    for (int64_t h = (int64_t)blockIdx.x * 4 + wave; h < n_medium; h += (int64_t)gridDim.x * 4) {   // uniform over the wavefront
        const int32_t i = a.medq[h];
        const int32_t cnt = ex_count_row<SAMPLED, 1>(a, a.ring_ids[i], n_rows);
        if (lane_id() == 0) a.counts[i] = cnt;
    }
    for (int32_t h = blockIdx.x; h < n_hub; h += gridDim.x) {   // uniform over the workgroup
        const int32_t i = a.hubq[h];
        const int32_t cnt = ex_count_row<SAMPLED, 4>(a, a.ring_ids[i], n_rows);
        if (lane_id() == 0) s_cnt[wave] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) a.counts[i] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        __syncthreads();
    }
}

// ---- fill pass -----------------------------------------------------------------------------------------------------
// An entry of target i's kept row that leads to outside vertex `id`: i takes the next free place of that vertex's row.
__device__ __forceinline__ void ex_reverse(const ExArgs& a, int32_t id, int32_t i) {
    if (id >= a.n_local) return;
    const int32_t q = atomicAdd(&a.counts[id], 1);
    if (q < a.capacity) a.out_ci[q] = i;
}

template <bool SAMPLED>
__global__ __launch_bounds__(256) void ex_fill_kernel(ExArgs a) {
    const int32_t first = ex_first(a);
    __shared__ RowLists lists;
    row_lists_init(lists);
    const int lane = lane_id(), sub = lane / kRowLanes, sl = lane % kRowLanes;
    const int grp = (int)threadIdx.x / kRowLanes;
    const int32_t n_rows = ex_rows<SAMPLED>(a);
    RowWalk w{a.ring_ids, a.rp, a.n, n_rows, (int64_t)gridDim.x * kRowsPerWg};
    w.begin((int64_t)blockIdx.x * kRowsPerWg + grp);
    for (int64_t c = blockIdx.x; c * kRowsPerWg < n_rows; c += gridDim.x) {   // uniform over the workgroup
        const int64_t i = c * kRowsPerWg + grp;
        int32_t s = w.s, e = w.e;
        int64_t out = i < n_rows ? a.out_rp[i] : 0;
        const int32_t after = w.ahead(i);
        if (e - s > kRowShort) {   // uniform over the 16-lane group
            if (sl == 0) row_lists_push(lists, (int32_t)i, e - s, a.medq, a.hubq, &a.ctrl->rows);
            s = e = 0;
        }
        int32_t u[4], id[4], cls[4];
        uint32_t classes = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t p = (uint32_t)s + r * kRowLanes + sl;   // (past the row's end, a position may not fit an int32_t)
            u[r] = p < (uint32_t)e ? a.ci[p] : -1;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) id[r] = u[r] >= 0 ? a.new_id[u[r]] : -1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            cls[r] = id[r] >= 0 ? ex_class(first, a.L, id[r]) : -1;
            if (id[r] >= 0) classes |= 1u << cls[r];
            if (SAMPLED && id[r] >= n_rows) ex_reverse(a, id[r], (int32_t)i);
        }
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) classes |= __shfl_xor(classes, d, kWave);
        while (classes) {   // uniform over the wavefront: the distances that occur in one of its four rows
            const int d = __ffs(classes) - 1;
            classes &= classes - 1u;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t m = group_ballot(cls[r] == d, sub);
                const int64_t q = out + __popc(m & ((1u << sl) - 1u));
                if (cls[r] == d && q < a.capacity) a.out_ci[q] = id[r];
                out += __popc(m);
            }
        }
        w.next(after);
    }
    row_lists_flush(lists, a.medq, a.hubq, &a.ctrl->rows);
}

// queued rows of up to kRowMedium entries: a wavefront, the whole row in EPL registers a lane
template <bool SAMPLED, int EPL>
__device__ __forceinline__ void ex_fill_medium_row(const ExArgs& a, int32_t first, int32_t n_rows, int32_t i, int32_t s, int32_t e, int64_t out) {
    const int lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    int32_t id[EPL], cls[EPL];
    uint32_t classes = 0u;
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
        const uint32_t p = (uint32_t)s + r * kWave + lane;
        id[r] = p < (uint32_t)e ? a.ci[p] : -1;
    }
#pragma unroll
    for (int r = 0; r < EPL; ++r) id[r] = id[r] >= 0 ? a.new_id[id[r]] : -1;
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
        cls[r] = id[r] >= 0 ? ex_class(first, a.L, id[r]) : -1;
        if (id[r] >= 0) classes |= 1u << cls[r];
        if (SAMPLED && id[r] >= n_rows) ex_reverse(a, id[r], i);
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) classes |= __shfl_xor(classes, d, kWave);
    while (classes) {   // uniform over the wavefront
        const int d = __ffs(classes) - 1;
        classes &= classes - 1u;
#pragma unroll
        for (int r = 0; r < EPL; ++r) {
            const uint64_t m = __ballot(cls[r] == d);
            const int64_t q = out + __popcll(m & below);
            if (cls[r] == d && q < a.capacity) a.out_ci[q] = id[r];
            out += __popcll(m);
        }
    }
}

template <bool SAMPLED>
__device__ __forceinline__ void ex_fill_medium(const ExArgs& a, int32_t first) {
    constexpr int kAll = kRowMedium / kWave;
    const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int32_t n_rows = ex_rows<SAMPLED>(a), n_queue = a.ctrl->rows.n_medium;
    for (int64_t h = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; h < n_queue; h += waves) {   // uniform over the wavefront
        const int32_t i = a.medq[h];
        const int32_t v = a.ring_ids[i];
        const int32_t s = a.rp[v], e = a.rp[v + 1];
        const int64_t out = a.out_rp[i];
        if (e - s <= kRowMedium / 4) ex_fill_medium_row<SAMPLED, kAll / 4>(a, first, n_rows, i, s, e, out);
        else ex_fill_medium_row<SAMPLED, kAll>(a, first, n_rows, i, s, e, out);
    }
}

// longer queued rows: a workgroup, 2048 entries per step; the first sweep counts the distances, the second writes
template <bool SAMPLED>
__device__ __forceinline__ void ex_fill_hubs(const ExArgs& a, int32_t first) {
    constexpr int EPL = 8, kClasses = kExMaxHops + 2;
    __shared__ int32_t s_at[kClasses];         // next output place of every distance, relative to the row's start
    __shared__ int32_t s_cnt[kClasses][4];     // entries of every distance in the wavefronts' parts of a step
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const uint64_t below = (1ull << lane) - 1ull;
    const int32_t n_rows = ex_rows<SAMPLED>(a), n_queue = a.ctrl->rows.n_hub;
    for (int32_t h = blockIdx.x; h < n_queue; h += gridDim.x) {   // uniform over the workgroup
        const int32_t i = a.hubq[h];
        const int32_t v = a.ring_ids[i];
        const int32_t s = a.rp[v], e = a.rp[v + 1];
        const int64_t out = a.out_rp[i];
        int32_t id[EPL], cls[EPL];
        auto load = [&](int64_t base) {
            const int64_t p0 = base + wave * (EPL * kWave) + lane;
#pragma unroll
            for (int r = 0; r < EPL; ++r) id[r] = p0 + r * kWave < e ? a.ci[p0 + r * kWave] : -1;
#pragma unroll
            for (int r = 0; r < EPL; ++r) id[r] = id[r] >= 0 ? a.new_id[id[r]] : -1;
#pragma unroll
            for (int r = 0; r < EPL; ++r) cls[r] = id[r] >= 0 ? ex_class(first, a.L, id[r]) : -1;
        };
        if (threadIdx.x < kClasses) s_at[threadIdx.x] = 0;
        __syncthreads();
        for (int64_t base = s; base < e; base += 4 * EPL * kWave) {
            load(base);
#pragma unroll
            for (int r = 0; r < EPL; ++r) {
                uint64_t rest = __ballot(cls[r] >= 0);
                while (rest) {   // uniform over the wavefront: one turn per distance that occurs
                    const int d = __shfl(cls[r], __ffsll((unsigned long long)rest) - 1, kWave);
                    const uint64_t m = __ballot(cls[r] == d);
                    if (lane == 0) atomicAdd(&s_at[d], __popcll(m));
                    rest &= ~m;
                }
                if (SAMPLED && id[r] >= n_rows) ex_reverse(a, id[r], i);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t at = 0;
            for (int d = 0; d < kClasses; ++d) {
                const int32_t c = s_at[d];
                s_at[d] = at;
                at += c;
            }
        }
        __syncthreads();
        for (int64_t base = s; base < e; base += 4 * EPL * kWave) {
            load(base);
            for (int d = 0; d <= a.L; ++d) {
                int c = 0;
#pragma unroll
                for (int r = 0; r < EPL; ++r) c += __popcll(__ballot(cls[r] == d));
                if (lane == 0) s_cnt[d][wave] = c;
            }
            __syncthreads();
            for (int d = 0; d <= a.L; ++d) {
                int64_t at = out + s_at[d];
                for (int w = 0; w < wave; ++w) at += s_cnt[d][w];
#pragma unroll
                for (int r = 0; r < EPL; ++r) {
                    const uint64_t m = __ballot(cls[r] == d);
                    const int64_t q = at + __popcll(m & below);
                    if (cls[r] == d && q < a.capacity) a.out_ci[q] = id[r];
                    at += __popcll(m);
                }
            }
            __syncthreads();
            if ((int)threadIdx.x <= a.L) {
                const int d = (int)threadIdx.x;
                s_at[d] += s_cnt[d][0] + s_cnt[d][1] + s_cnt[d][2] + s_cnt[d][3];
            }
            __syncthreads();
        }
    }
}

template <bool SAMPLED>
__global__ __launch_bounds__(256) void ex_fill_long_kernel(ExArgs a) {
    const int32_t first = ex_first(a);
    ex_fill_medium<SAMPLED>(a, first);
    ex_fill_hubs<SAMPLED>(a, first);
}

// ---- reverse rows ----------------------------------------------------------------------------------------------------
// Orders the reverse rows of 2 to 64 entries (a wavefront looks at 64 rows and orders four at a time: most hold a single
// entry) and queues the longer ones: up to kExSortMax entries "medium", longer or cut by the capacity "hub".
__global__ __launch_bounds__(256) void ex_order_kernel(ExArgs a) {
    __shared__ RowLists lists;
    row_lists_init(lists);
    const int lane = lane_id(), sub = lane / kRowLanes, sl = lane % kRowLanes;
    const int32_t n_targets = ex_rows<true>(a);
    for (int64_t c = (int64_t)n_targets + (int64_t)blockIdx.x * 256; c < a.n_local; c += (int64_t)gridDim.x * 256) {   // uniform over the workgroup
        const int64_t j = c + threadIdx.x;
        int32_t s = 0, e = 0;
        if (j < a.n_local) {
            s = a.out_rp[j];
            e = a.out_rp[j + 1];
        }
        const bool cut = s < a.capacity && e > a.capacity;
        const bool queued = s < a.capacity && (cut || e - s > kRowShort);
        if (queued) row_lists_push(lists, (int32_t)j, cut ? kRowMedium + 1 : e - s, a.medq, a.hubq, &a.ctrl->reverse);
        uint64_t todo = __ballot(!queued && s < a.capacity && e - s > 1);
        while (todo) {   // uniform over the wavefront
            uint64_t rest = todo;
            int from = -1;
            for (int k = 0; k < 4 && rest; ++k) {
                if (k == sub) from = __ffsll((unsigned long long)rest) - 1;
                rest &= rest - 1ull;
            }
            todo = rest;
            const int32_t rs = __shfl(s, from < 0 ? 0 : from, kWave), re = __shfl(e, from < 0 ? 0 : from, kWave);
            const int len = from < 0 ? 0 : re - rs;
            int len_max = max(len, __shfl_xor(len, 16, kWave));
            len_max = max(len_max, __shfl_xor(len_max, 32, kWave));
            int32_t x[4];
            int place[4] = {0, 0, 0, 0};
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = r * kRowLanes + sl < len ? a.out_ci[rs + r * kRowLanes + sl] : INT32_MAX;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                for (int t = 0; t < kRowLanes && r * kRowLanes + t < len_max; ++t) {   // uniform over the wavefront
                    const int32_t y = __shfl(x[r], sub * kRowLanes + t, kWave);
#pragma unroll
                    for (int q = 0; q < 4; ++q) place[q] += y < x[q] + (r < q || (r == q && t < sl));   // equal ids: the earlier first
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r * kRowLanes + sl < len) a.out_ci[rs + place[r]] = x[r];
        }
    }
    row_lists_flush(lists, a.medq, a.hubq, &a.ctrl->reverse);
}

// reverse rows of 65 to kExSortMax entries: a workgroup, the row in LDS
__device__ __forceinline__ void ex_order_medium(const ExArgs& a) {
    static_assert(kExSortMax == kRowMedium && kExSortMax % 256 == 0, "the queue's classes");
    __shared__ __attribute__((aligned(16))) int32_t s_x[kExSortMax];
    const int32_t n_queue = a.ctrl->reverse.n_medium;
    for (int32_t h = blockIdx.x; h < n_queue; h += gridDim.x) {   // uniform over the workgroup
        const int32_t j = a.medq[h];
        const int32_t s = a.out_rp[j], len = a.out_rp[j + 1] - s;
        __syncthreads();   // the previous row has been read
        for (int t = threadIdx.x; t < (len + 3) / 4 * 4; t += 256) s_x[t] = t < len ? a.out_ci[s + t] : INT32_MAX;
        __syncthreads();
        int32_t x[kExSortMax / 256];
        int place[kExSortMax / 256];
#pragma unroll
        for (int r = 0; r < kExSortMax / 256; ++r) {
            x[r] = (int)threadIdx.x + 256 * r < len ? s_x[threadIdx.x + 256 * r] : 0;
            place[r] = 0;
        }
        for (int t = 0; t < len; t += 4) {   // the filling is larger than every id
            const int4 y = *(const int4*)&s_x[t];
#pragma unroll
            for (int r = 0; r < kExSortMax / 256; ++r) {
                const int before = (int)threadIdx.x + 256 * r - t;   // equal ids: the earlier first
                place[r] += (y.x < x[r] + (before > 0)) + (y.y < x[r] + (before > 1)) + (y.z < x[r] + (before > 2)) + (y.w < x[r] + (before > 3));
            }
        }
#pragma unroll
        for (int r = 0; r < kExSortMax / 256; ++r)
            if ((int)threadIdx.x + 256 * r < len) a.out_ci[s + place[r]] = x[r];
    }
}

// does the kept row of target u hold v more than `nth` times?  (kept rows are ascending)
__device__ __forceinline__ bool ex_kept(const ExArgs& a, int32_t u, int32_t v, int64_t nth) {
    const int32_t e = a.rp[u + 1];
    int32_t lo = a.rp[u], hi = e;
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (a.ci[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo + nth < e && a.ci[lo + nth] == v;
}

// the remaining reverse rows, collected in order from the transposed graph
__device__ __forceinline__ void ex_reverse_scan(const ExArgs& a) {
    __shared__ int s_part[4];
    const int32_t n_targets = ex_rows<true>(a), n_queue = a.ctrl->reverse.n_hub;
    for (int32_t h = blockIdx.x; h < n_queue; h += gridDim.x) {   // uniform over the workgroup
        const int32_t j = a.hubq[h];
        const int32_t v = a.ring_ids[j];
        int32_t s = 0, e = 0;
        if (v >= 0 && v < a.n) {
            s = a.t_rp[v];
            e = a.t_rp[v + 1];
        }
        int64_t out = a.out_rp[j];
        const int64_t end = a.out_rp[j + 1] < a.capacity ? a.out_rp[j + 1] : a.capacity;
        for (int64_t base = s; base < e; base += 256) {
            int32_t id = -1;
            const int64_t p = base + threadIdx.x;
            if (p < e) {
                const int32_t u = a.t_ci[p];
                id = a.new_id[u];
                if (id >= n_targets) id = -1;
                if (id >= 0) {
                    int64_t first = p;      // a repeated entry stays as often as the kept row holds it
                    while (first > s && a.t_ci[first - 1] == u) --first;
                    if (!ex_kept(a, u, v, p - first)) id = -1;
                }
            }
            int total;
            const int64_t q = out + block_exclusive_scan<256>(id >= 0 ? 1 : 0, s_part, &total);
            if (id >= 0 && q < end) a.out_ci[q] = id;
            out += total;
        }
    }
}

__global__ __launch_bounds__(256) void ex_order_long_kernel(ExArgs a) {
    ex_order_medium(a);
    ex_reverse_scan(a);
}

// dst[i, 0:row_bytes) = src[ids[i], 0:row_bytes): 16 lanes per row, 16 bytes per lane and step
__global__ __launch_bounds__(256) void gather_rows_kernel(const char* __restrict__ src, int64_t src_stride, const int32_t* __restrict__ ids,
                                                           int32_t n, int32_t n_src, int64_t row_bytes, char* __restrict__ dst,
                                                           int64_t dst_stride, int vec) {
    const int sl = (int)(threadIdx.x % 16);
    const int64_t groups = (int64_t)gridDim.x * (blockDim.x / 16);
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 16; i < n; i += groups) {
        const int32_t v = ids[i];
        if (v < 0 || v >= n_src) continue;
        const char* s = src + (int64_t)v * src_stride;
        char* d = dst + i * dst_stride;
        if (vec) {
            for (int64_t b = (int64_t)sl * 16; b < row_bytes; b += 256) *(uint4*)(d + b) = *(const uint4*)(s + b);
        } else {
            for (int64_t b = (int64_t)sl * 2; b < row_bytes; b += 32) *(uint16_t*)(d + b) = *(const uint16_t*)(s + b);
        }
    }
}

}  // namespace gnnhot

using namespace gnnhot;

// The traversed set as a bitmap pays for its launch where new_id[] does not fit an L2 next to the rows that stream
// through it: a 1M-vertex / 20M-entry graph counts in 0.11 + 0.005 ms instead of 0.15, below the limit nothing is gained.
constexpr int32_t kExBitsMin = 1 << 19;

// a thread per item, whatever their number (these kernels do not stride)
static inline int ex_grid(int32_t items) { return grid_for(items, 256, INT32_MAX); }

template <bool SAMPLED>
static int32_t ex_count_pass(ExArgs a, const int32_t* dist, int32_t* new_id, uint64_t* bits, int row_grid, int long_grid,
                             hipStream_t stream) {
    fill_kernel<int32_t><<<grid_for(a.n, 256, 1 << 16), 256, 0, stream>>>(new_id, a.n, -1);
    GNN_LAUNCH_CHECK("fill_kernel");
    if (a.n_local == 0) return GNN_OK;
    ex_number_kernel<<<ex_grid(a.n_local), 256, 0, stream>>>(a.ring_ids, a.n_local, a.n, dist, new_id, SAMPLED ? a.counts : nullptr,
                                                                   nullptr, a.ctrl);
    GNN_LAUNCH_CHECK("ex_number_kernel");
    if (!SAMPLED && a.n >= kExBitsMin) {
        ex_bits_kernel<<<ex_grid(a.n), 256, 0, stream>>>(new_id, a.n, bits);
        GNN_LAUNCH_CHECK("ex_bits_kernel");
        a.bits = (const uint32_t*)bits;
    }
    ex_count_kernel<SAMPLED><<<row_grid, 256, 0, stream>>>(a);
    GNN_LAUNCH_CHECK("ex_count_kernel");
    ex_count_long_kernel<SAMPLED><<<long_grid, 256, 0, stream>>>(a);
    GNN_LAUNCH_CHECK("ex_count_long_kernel");
    return GNN_OK;
}

template <bool SAMPLED>
static int32_t ex_fill_pass(const ExArgs& a, const int32_t* dist, int64_t nnz, int row_grid, int long_grid, hipStream_t stream) {
    ex_number_kernel<<<ex_grid(a.n_local), 256, 0, stream>>>(a.ring_ids, a.n_local, a.n, dist, nullptr, SAMPLED ? a.counts : nullptr,
                                                                   a.out_rp, a.ctrl);
    GNN_LAUNCH_CHECK("ex_number_kernel");
    ex_fill_kernel<SAMPLED><<<row_grid, 256, 0, stream>>>(a);
    GNN_LAUNCH_CHECK("ex_fill_kernel");
    ex_fill_long_kernel<SAMPLED><<<long_grid, 256, 0, stream>>>(a);
    GNN_LAUNCH_CHECK("ex_fill_long_kernel");
    if (SAMPLED) {
        ex_order_kernel<<<queue_grid(a.n_local, nnz, 256), 256, 0, stream>>>(a);
        GNN_LAUNCH_CHECK("ex_order_kernel");
        ex_order_long_kernel<<<long_grid, 256, 0, stream>>>(a);
        GNN_LAUNCH_CHECK("ex_order_long_kernel");
    }
    return GNN_OK;
}

// count pass / fill pass shared by the two extraction entry points (g: the graph, sampled: transposed; gs: kept rows)
static int32_t extract_common(const gnn_csr* g, const gnn_csr* gs, const int32_t* ring_ids, int32_t n_local, const int32_t* dist,
                              int32_t L, int32_t* new_id, int32_t* out_row_ptr, int32_t* out_col_idx, int64_t out_capacity,
                              int64_t* out_nnz, int64_t* out_nnz_host, void* ws, size_t* ws_bytes, hipStream_t stream) {
    GNN_REQUIRE(g->n_rows == g->n_cols, GNN_ERR_SHAPE, "the graph must be square (%d x %d)", g->n_rows, g->n_cols);
    GNN_REQUIRE(n_local >= 0 && n_local <= g->n_rows, GNN_ERR_INVALID_ARG, "n_local %d outside [0, %d]", n_local, g->n_rows);
    GNN_REQUIRE(L >= 1 && L <= kExMaxHops, GNN_ERR_INVALID_ARG, "L = %d outside [1, %d]", L, kExMaxHops);
    const int64_t n_bit_words = ((int64_t)g->n_rows + 63) / 64 + 1;
    const int32_t n_blocks = offsets_scan_blocks(n_local);
    WsCarver carve(ws);
    int32_t* counts = carve.take<int32_t>((size_t)n_local + 1);
    int32_t* sums = carve.take<int32_t>((size_t)n_blocks + 1);
    int32_t* medq = carve.take<int32_t>((size_t)n_local + 1);
    int32_t* hubq = carve.take<int32_t>((size_t)n_local + 1);
    uint64_t* bits = carve.take<uint64_t>((size_t)n_bit_words);
    ExCtrl* ctrl = carve.take<ExCtrl>(1);
    bool query;
    GNN_CHECK(ws_protocol(ws, ws_bytes, carve.used, &query));
    if (query) return GNN_OK;
    GNN_REQUIRE(new_id != nullptr && out_row_ptr != nullptr, GNN_ERR_INVALID_ARG, "new_id / out_row_ptr is NULL");
    GNN_REQUIRE(n_local == 0 || (ring_ids != nullptr && dist != nullptr), GNN_ERR_INVALID_ARG, "ring_ids / dist is NULL");
    const int64_t nnz = gs ? gs->nnz : g->nnz;
    const int row_grid = queue_grid(n_local, nnz, kRowsPerWg);   // grid-stride loops, here and over the queues
    const int long_grid = grid_for(n_local, 4, 2048);
    ExArgs a;
    a.rp = gs ? gs->row_ptr : g->row_ptr; a.ci = gs ? gs->col_idx : g->col_idx;
    a.t_rp = g->row_ptr; a.t_ci = g->col_idx;
    a.ring_ids = ring_ids; a.n_local = n_local; a.n = g->n_rows; a.L = L;
    a.new_id = new_id; a.bits = nullptr; a.counts = counts;
    a.out_rp = out_row_ptr; a.out_ci = out_col_idx; a.capacity = out_capacity;
    a.medq = medq; a.hubq = hubq; a.ctrl = ctrl;

    if (out_col_idx == nullptr) {  // count pass
        GNN_REQUIRE(out_nnz != nullptr, GNN_ERR_INVALID_ARG, "out_nnz is NULL");
        if (g->n_rows > 0) {
            GNN_CHECK(gs ? ex_count_pass<true>(a, dist, new_id, bits, row_grid, long_grid, stream)
                         : ex_count_pass<false>(a, dist, new_id, bits, row_grid, long_grid, stream));
        }
        GNN_CHECK(counts_to_offsets(counts, n_local, sums, out_row_ptr, out_nnz, stream));
        if (out_nnz_host != nullptr) {
            GNN_HIP(hipMemcpyAsync(out_nnz_host, out_nnz, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
            GNN_HIP(hipStreamSynchronize(stream));
        }
        return GNN_OK;
    }
    GNN_REQUIRE(out_capacity >= 0, GNN_ERR_INVALID_ARG, "out_capacity < 0");
    if (n_local > 0) {
        GNN_CHECK(gs ? ex_fill_pass<true>(a, dist, nnz, row_grid, long_grid, stream)
                     : ex_fill_pass<false>(a, dist, nnz, row_grid, long_grid, stream));
    }
    return GNN_OK;
}

extern "C" int32_t gnn_extract_partition(const gnn_csr* g, const int32_t* ring_ids, int32_t n_local, const int32_t* dist, int32_t L,
                                         int32_t* new_id, int32_t* out_row_ptr, int32_t* out_col_idx, int64_t out_capacity,
                                         int64_t* out_nnz, int64_t* out_nnz_host, void* ws, size_t* ws_bytes, void* stream) {
    GNN_CHECK(check_csr(g, "g"));
    return extract_common(g, nullptr, ring_ids, n_local, dist, L, new_id, out_row_ptr, out_col_idx, out_capacity, out_nnz, out_nnz_host,
                          ws, ws_bytes, (hipStream_t)stream);
}

extern "C" int32_t gnn_extract_sampled_partition(const gnn_csr* gT, const gnn_csr* gs, const int32_t* ring_ids, int32_t n_local,
                                                 const int32_t* dist, int32_t* new_id, int32_t* out_row_ptr, int32_t* out_col_idx,
                                                 int64_t out_capacity, int64_t* out_nnz, int64_t* out_nnz_host, void* ws,
                                                 size_t* ws_bytes, void* stream) {
    GNN_CHECK(check_csr(gT, "gT"));
    GNN_CHECK(check_csr(gs, "gs"));
    GNN_REQUIRE(gs->n_rows == gT->n_rows && gs->n_cols == gT->n_cols, GNN_ERR_SHAPE, "gs (%d x %d) and gT (%d x %d) differ in shape",
                gs->n_rows, gs->n_cols, gT->n_rows, gT->n_cols);
    return extract_common(gT, gs, ring_ids, n_local, dist, 1, new_id, out_row_ptr, out_col_idx, out_capacity, out_nnz, out_nnz_host, ws,
                          ws_bytes, (hipStream_t)stream);
}

// out_row_ptr over the full id range from a row list: row ids[i] gets the length of listed row i, every other row is empty
__global__ __launch_bounds__(256) void expand_lengths_kernel(const int32_t* __restrict__ ids, int32_t n_ids,
                                                              const int32_t* __restrict__ list_row_ptr, int32_t n,
                                                              int32_t* __restrict__ counts) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_ids) {
        const int32_t v = ids[i];
        if (v >= 0 && v < n) counts[v] = list_row_ptr[i + 1] - list_row_ptr[i];
    }
}

extern "C" int32_t gnn_expand_row_ptr(int32_t n, const int32_t* ids, int32_t n_ids, const int32_t* list_row_ptr, int32_t* out_row_ptr,
                                      void* ws, size_t* ws_bytes, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_REQUIRE(n >= 0 && n_ids >= 0, GNN_ERR_INVALID_ARG, "negative size");
    WsCarver carve(ws);
    int32_t* counts = carve.take<int32_t>((size_t)n + 1);
    int32_t* sums = carve.take<int32_t>((size_t)offsets_scan_blocks(n) + 1);
    int64_t* total = carve.take<int64_t>(1);
    bool query;
    GNN_CHECK(ws_protocol(ws, ws_bytes, carve.used, &query));
    if (query) return GNN_OK;
    GNN_REQUIRE(out_row_ptr != nullptr, GNN_ERR_INVALID_ARG, "out_row_ptr is NULL");
    GNN_REQUIRE(n_ids == 0 || (ids != nullptr && list_row_ptr != nullptr), GNN_ERR_INVALID_ARG, "ids / list_row_ptr is NULL");
    if (n > 0) {
        fill_kernel<int32_t><<<grid_for(n, 256, 1 << 16), 256, 0, stream>>>(counts, n, 0);
        GNN_LAUNCH_CHECK("fill_kernel");
    }
    if (n_ids > 0) {
        expand_lengths_kernel<<<ex_grid(n_ids), 256, 0, stream>>>(ids, n_ids, list_row_ptr, n, counts);
        GNN_LAUNCH_CHECK("expand_lengths_kernel");
    }
    return counts_to_offsets(counts, n, sums, out_row_ptr, total, stream);
}

extern "C" int32_t gnn_gather_rows(const void* src, int64_t ld_src, int32_t n_src, const int32_t* ids, int32_t n, int32_t F,
                                   int32_t dtype, void* dst, int64_t ld_dst, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_REQUIRE(dtype == GNN_F32 || dtype == GNN_BF16, GNN_ERR_UNSUPPORTED, "unknown dtype %d", dtype);
    GNN_REQUIRE(n >= 0 && F >= 0 && n_src >= 0, GNN_ERR_INVALID_ARG, "negative size");
    GNN_REQUIRE(ld_src >= F && ld_dst >= F, GNN_ERR_SHAPE, "leading dimension smaller than F = %d", F);
    if (n == 0 || F == 0) return GNN_OK;
    GNN_REQUIRE(src != nullptr && dst != nullptr && ids != nullptr, GNN_ERR_INVALID_ARG, "src / dst / ids is NULL");
    const int64_t es = dtype == GNN_F32 ? 4 : 2;
    const int64_t row_bytes = (int64_t)F * es;
    const int vec = ((uintptr_t)src % 16 == 0) && ((uintptr_t)dst % 16 == 0) && (ld_src * es) % 16 == 0 && (ld_dst * es) % 16 == 0 &&
                    row_bytes % 16 == 0;
    gather_rows_kernel<<<grid_for((int64_t)n * 16, 256, 1 << 20), 256, 0, stream>>>((const char*)src, ld_src * es, ids, n, n_src, row_bytes,
                                                                                 (char*)dst, ld_dst * es, vec);
    GNN_LAUNCH_CHECK("gather_rows_kernel");
    return GNN_OK;
}
