// Expansion-aware sampling, boundary only (paper section 5.3): dependencies between inner
// (target) vertices stay whole; of the neighbours that lie outside the target set each
// target keeps at most `fanout`.  The choice is a seeded counter-based hash of the edge
// (no generator state, no dependence on thread order): the `fanout` smallest (key, id) win.
//
// Rows are handled in three length classes (rowlists.h), so that every class keeps its whole row in registers or walks it
// with many independent loads in flight (a partition grown breadth-first holds the graph's hubs: on the 10M-vertex
// workload 15 % of the target rows are longer than 64 entries and hold 70 % of all candidates):
//   up to 64 entries    sixteen lanes per row, four entries per lane;
//   65 to 1024          one wavefront per row, four entries per lane up to 256, else sixteen (second launch of the pass);
//   longer              one workgroup per row, which strides the row four entries per thread and step (third launch).
// Count pass: ballots give |row in T| and the number of outside neighbours; a scan turns counts into row offsets.  Fill
// pass: a row with more than `fanout` outside neighbours finds the fanout-th smallest (key, id) - among its registers
// (group_kth), or, a long row, among the few keys below a guessed one - and emits the row in its original ascending
// order through a ballot-prefix compaction.
// Which lane group, wavefront or workgroup takes a row does not matter: every row's result depends on the row alone.
// Bound: HBM (streaming reads of the target rows) and the hash.  Kernel time of both passes on a 5M-vertex / 75M-entry graph,
// 625 000 targets, fanout 5: 0.80 -> 0.59 ms against `fanout` rounds over 64-bit pairs with the long rows re-read in every
// round (long rows 0.33 -> 0.16); 700 000 vertices of 100 entries, fanout 10, with the extraction: 2.26 -> 1.76 ms.  Since then
// 0.48 and 1.19: a long row's outside neighbours follow from its share of the output instead of a sweep, and its kept entries are
// placed 1024 at a time (fill 162 us -> 102), medium rows hold upper halves of keys (71 -> 62), one atomic a workgroup and half the
// workgroups (rowlists.h: count 119 -> 75).
#include "common.h"
#include "hashkey.h"
#include "rowlists.h"
#include "scan.h"

namespace gnnhot {

// Sixteen lanes per target row, four rows per wavefront (the paper's graphs have 15-50 neighbours per vertex): the
// length classes and the queues are those of rowlists.h.
__global__ __launch_bounds__(256) void sb_count_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                       int32_t n, const uint32_t* __restrict__ tbits,
                                                       const int32_t* __restrict__ targets, int32_t n_targets, int32_t fanout,
                                                       int32_t* __restrict__ counts, int32_t* __restrict__ medq,
                                                       int32_t* __restrict__ hubq, RowCtrl* ctrl) {
    __shared__ RowLists lists;
    row_lists_init(lists);
    const int lane = lane_id(), sub = lane / kRowLanes, sl = lane % kRowLanes;
    const int grp = (int)threadIdx.x / kRowLanes;
    RowWalk w{targets, row_ptr, n, n_targets, (int64_t)gridDim.x * kRowsPerWg};
    w.begin((int64_t)blockIdx.x * kRowsPerWg + grp);
    for (int64_t c = blockIdx.x; c * kRowsPerWg < n_targets; c += gridDim.x) {   // uniform over the workgroup
        const int64_t i = c * kRowsPerWg + grp;
        int32_t s = w.s, e = w.e;
        const int32_t after = w.ahead(i);
        const bool is_long = e - s > kRowShort;   // uniform over the 16-lane group
        if (is_long) {
            if (sl == 0) row_lists_push(lists, (int32_t)i, e - s, medq, hubq, ctrl);
            s = e = 0;
        }
        int32_t n_in = 0, n_ext = 0;
        int32_t ru[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {  // all four loads of a lane in flight together
            const uint32_t p = (uint32_t)s + r * kRowLanes + sl;   // (past the row's end, a position may not fit an int32_t)
            ru[r] = p < (uint32_t)e ? col_idx[p] : 0;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool valid = (uint32_t)s + r * kRowLanes + sl < (uint32_t)e;
            const bool inner = valid && in_set(tbits, ru[r]);
            n_in += __popc(group_ballot(inner, sub));
            n_ext += __popc(group_ballot(valid && !inner, sub));
        }
        if (sl == 0 && i < n_targets && !is_long) counts[i] = n_in + (n_ext < fanout ? n_ext : fanout);
        w.next(after);
    }
    row_lists_flush(lists, medq, hubq, ctrl);
}


__global__ __launch_bounds__(256) void sb_fill_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                      int32_t n, const uint32_t* __restrict__ tbits,
                                                      const int32_t* __restrict__ targets, int32_t n_targets, int32_t fanout,
                                                      uint64_t seed_hop_mixed, const int32_t* __restrict__ out_row_ptr,
                                                      int32_t* __restrict__ out_col_idx, int64_t capacity,
                                                      int32_t* __restrict__ medq, int32_t* __restrict__ hubq, RowCtrl* ctrl) {
    __shared__ RowLists lists;
    row_lists_init(lists);
    const int lane = lane_id(), sub = lane / kRowLanes, sl = lane % kRowLanes;
    const int grp = (int)threadIdx.x / kRowLanes;
    RowWalk w{targets, row_ptr, n, n_targets, (int64_t)gridDim.x * kRowsPerWg};
    w.begin((int64_t)blockIdx.x * kRowsPerWg + grp);
    for (int64_t c = blockIdx.x; c * kRowsPerWg < n_targets; c += gridDim.x) {   // uniform over the workgroup
    const int64_t i = c * kRowsPerWg + grp;
    const int32_t v = w.v;
    int32_t s = w.s, e = w.e;
    int64_t at = i < n_targets ? (int64_t)out_row_ptr[i] : 0;
    const int32_t after = w.ahead(i);
    if (e - s > kRowShort) {   // uniform over the 16-lane group: a wavefront or a workgroup of the later launches takes this row
        if (sl == 0) row_lists_push(lists, (int32_t)i, e - s, medq, hubq, ctrl);
        s = e = 0;
    }
    // each lane holds up to four entries of its row in registers, so the selection rounds need no further memory traffic
    int32_t ru[4];
    uint64_t rk[4];
    int rf[4];  // 0: no entry, 1: neighbour inside the target set, 2: outside
    int32_t n_out = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t p = (uint32_t)s + r * kRowLanes + sl;
        ru[r] = p < (uint32_t)e ? col_idx[p] : 0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t p = (uint32_t)s + r * kRowLanes + sl;
        rf[r] = p < (uint32_t)e ? (in_set(tbits, ru[r]) ? 1 : 2) : 0;
        rk[r] = rf[r] == 2 ? edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)ru[r]) : ~0ull;
        n_out += __popc(group_ballot(rf[r] == 2, sub));
    }
    // threshold pair: outside neighbours with (key, id) <= (tk, tu) are kept
    uint64_t tk = ~0ull;
    int32_t tu = 0x7fffffff;
    if (fanout == 0) {
        tk = 0ull;
        tu = -1;  // nothing is <= (0, -1): ids are non-negative
    }
    const bool want = fanout > 0 && n_out > fanout;   // uniform over the 16-lane group
    if (__ballot(want) != 0ull) {                      // uniform over the wavefront
        uint32_t cand = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) cand |= rf[r] == 2 ? 1u << r : 0u;
        group_kth<4, kRowLanes>(rk, ru, cand, fanout, want, tk, tu);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool keep = rf[r] == 1 || (rf[r] == 2 && !pair_less(tk, tu, rk[r], ru[r]));
        const uint32_t m = group_ballot(keep, sub);
        const int64_t my = at + __popc(m & ((1u << sl) - 1u));
        if (keep && my < capacity) out_col_idx[my] = ru[r];
        at += __popc(m);
    }
    w.next(after);
    }   // grid-stride loop
    row_lists_flush(lists, medq, hubq, ctrl);
}

// Targets from which twice the workgroups are worth their appends: the later half evens out the end of the launch.  us, 2048 / 4096: 1 M
// targets of 30 342 / 311, 2 M 940 / 870, 4 M 1666 / 1531; power-law 2.5 M of 15 976 / 913, 3 M of 40 1848 / 1748; but 625 000 of 100 1225 / 1243, 125 000
// 301 / 346.
constexpr int32_t kSbManyRows = 800000;

// ---- rows of 65 to 1024 entries: one wavefront per queued row, everything in registers -----------------------------------
// A row of up to EPL * 64 entries.  The selection compares the upper halves of the keys; where they do not decide (about
// n^2 / 2^33 of the rows) whole pairs do.
template <bool FILL, int EPL>
__device__ __forceinline__ void sb_medium_row(const int32_t* __restrict__ col_idx, const uint32_t* __restrict__ tbits, int32_t v, int32_t s, int32_t e,
                                              int32_t fanout, uint64_t seed_hop_mixed, int32_t* __restrict__ count, int64_t at,
                                              int32_t* __restrict__ out_col_idx, int64_t capacity) {
    const int lane = lane_id();
    int32_t ru[EPL];
    uint32_t inner = 0u, outer = 0u;     // bit r: the lane's r-th entry is a neighbour inside the target set, outside
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
        const uint32_t p = (uint32_t)s + r * kWave + lane;
        ru[r] = p < (uint32_t)e ? col_idx[p] : 0;
    }
    int32_t n_in = 0, n_ext = 0;
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
        const bool there = (uint32_t)s + r * kWave + lane < (uint32_t)e, in = there && in_set(tbits, ru[r]);
        inner |= in ? 1u << r : 0u;
        outer |= there && !in ? 1u << r : 0u;
        n_in += __popcll(__ballot(in));
        n_ext += __popcll(__ballot(there && !in));
    }
    if (!FILL) {
        if (lane == 0) *count = n_in + (n_ext < fanout ? n_ext : fanout);
        return;
    }
    uint32_t half[EPL];
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
        half[r] = ~0u;
        if ((uint32_t)s + r * kWave < (uint32_t)e)     // uniform over the wavefront
            half[r] = (outer >> r) & 1u ? (uint32_t)(edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)ru[r]) >> 32) : ~0u;
    }
    uint32_t top = fanout > 0 ? ~0u : 0u;
    bool whole = true;
    uint64_t tk = 0ull;
    int32_t tu = -1;
    if (fanout > 0 && n_ext > fanout) {   // uniform over the wavefront
        whole = wave_kth_half<EPL>(half, ru, outer, fanout, top, tu);
        uint32_t kth = 0u;
        const int32_t rank = whole ? 0 : wave_kth_rank<EPL>(half, outer, fanout, kth);
        for (int32_t round = 0; round < rank; ++round) {     // of the pairs with that half, the smallest above (tk, tu)
            uint64_t best_k = ~0ull;
            int32_t best_u = 0x7fffffff;
#pragma unroll
            for (int r = 0; r < EPL; ++r) {
                if (((outer >> r) & 1u) == 0u || half[r] != kth) continue;
                const uint64_t k = edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)ru[r]);
                if ((round == 0 || pair_less(tk, tu, k, ru[r])) && pair_less(k, ru[r], best_k, best_u)) {
                    best_k = k;
                    best_u = ru[r];
                }
            }
            wave_min_pair(best_k, best_u);
            tk = best_k;
            tu = best_u;
        }
    }
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
        bool keep = fanout > 0 && half[r] <= top;
        if (!whole) keep = !pair_less(tk, tu, edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)ru[r]), ru[r]);
        keep = ((inner >> r) & 1u) != 0u || (((outer >> r) & 1u) != 0u && keep);
        const uint64_t m = __ballot(keep);
        const int64_t my = at + __popcll(m & below);
        if (keep && my < capacity) out_col_idx[my] = ru[r];
        at += __popcll(m);
    }
}

template <bool FILL>
__global__ __launch_bounds__(256) void sb_medium_rows_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                             const uint32_t* __restrict__ tbits, const int32_t* __restrict__ targets,
                                                             const int32_t* __restrict__ medq, const RowCtrl* __restrict__ ctrl,
                                                             int32_t fanout, uint64_t seed_hop_mixed, int32_t* __restrict__ counts,
                                                             const int32_t* __restrict__ out_row_ptr, int32_t* __restrict__ out_col_idx,
                                                             int64_t capacity) {
    const int64_t wave_g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int32_t n_med = ctrl->n_medium;
    for (int64_t h = wave_g; h < n_med; h += n_waves) {   // uniform over the wavefront
        const int32_t i = medq[h];
        const int32_t v = targets[i];
        const int32_t s = row_ptr[v], e = row_ptr[v + 1];
        int32_t* const count = FILL ? nullptr : counts + i;
        const int64_t at = FILL ? (int64_t)out_row_ptr[i] : 0;
        constexpr int kAll = kRowMedium / kWave;
        if (e - s <= kRowMedium / 4) sb_medium_row<FILL, kAll / 4>(col_idx, tbits, v, s, e, fanout, seed_hop_mixed, count, at, out_col_idx, capacity);
        else sb_medium_row<FILL, kAll>(col_idx, tbits, v, s, e, fanout, seed_hop_mixed, count, at, out_col_idx, capacity);
    }
}


// ---- rows of more than 1024 entries: one workgroup per queued row -----------------------------------------------
// Sums of two ints over the workgroup (every thread gets them).  Two barriers.
__device__ __forceinline__ void block_sum2(int& a, int& b, int* s_a, int* s_b) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        a += __shfl_xor(a, d, kWave);
        b += __shfl_xor(b, d, kWave);
    }
    const int w = (int)(threadIdx.x >> 6);
    if (lane_id() == 0) {
        s_a[w] = a;
        s_b[w] = b;
    }
    __syncthreads();
    a = s_a[0] + s_a[1] + s_a[2] + s_a[3];
    b = s_b[0] + s_b[1] + s_b[2] + s_b[3];
    __syncthreads();
}

// Smallest (key, id) pair over the workgroup (every thread gets it).  Two barriers.
__device__ __forceinline__ void block_min_pair(uint64_t& k, int32_t& u, uint64_t* s_k, int32_t* s_u) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint64_t ok = __shfl_xor(k, d, kWave);
        const int32_t ou = __shfl_xor(u, d, kWave);
        if (pair_less(ok, ou, k, u)) {
            k = ok;
            u = ou;
        }
    }
    const int w = (int)(threadIdx.x >> 6);
    if (lane_id() == 0) {
        s_k[w] = k;
        s_u[w] = u;
    }
    __syncthreads();
    k = s_k[0];
    u = s_u[0];
#pragma unroll
    for (int q = 1; q < 4; ++q)
        if (pair_less(s_k[q], s_u[q], k, u)) {
            k = s_k[q];
            u = s_u[q];
        }
    __syncthreads();
}

constexpr int kSbListCap = 512;   // pairs below the guessed key that a workgroup lists

// The same selection for the queued rows: 256 threads stride the row, four entries per thread and step with all their
// loads (ids, then target bits) issued before the first use.  The keys are uniform, so the row's pair is among the few
// below a guessed key: one sweep lists those in LDS and the first wavefront selects from the list; where the guess fails
// or the fanout is too large for the list, `fanout` sweeps of "smallest pair above the previous one" find it.  FILL false: counts[i];
// FILL true: the kept ids in ascending position order.  Which workgroup takes which row does not matter: every row's
// result depends on the row alone.
template <bool FILL>
__global__ __launch_bounds__(256) void sb_long_rows_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                           const uint32_t* __restrict__ tbits, const int32_t* __restrict__ targets,
                                                           const int32_t* __restrict__ hubq, const RowCtrl* __restrict__ ctrl,
                                                           int32_t fanout, uint64_t seed_hop_mixed, int32_t* __restrict__ counts,
                                                           const int32_t* __restrict__ out_row_ptr, int32_t* __restrict__ out_col_idx,
                                                           int64_t capacity) {
    __shared__ int s_a[4], s_b[4], s_part[4];
    __shared__ uint64_t s_k[4], s_key[kSbListCap];
    __shared__ int32_t s_u[4], s_id[kSbListCap], s_n;
    const int tid = (int)threadIdx.x;
    const int32_t n_hub = ctrl->n_hub;
    for (int32_t h = blockIdx.x; h < n_hub; h += gridDim.x) {   // uniform over the workgroup
        const int32_t i = hubq[h];
        const int32_t v = targets[i];
        const int32_t s = row_ptr[v], e = row_ptr[v + 1];
        int n_in = 0, n_ext = 0;
        // the row's share of the output says how many lie outside: all entries, or the inner ones and `fanout`
        if (FILL) n_ext = e - s - (out_row_ptr[i + 1] - out_row_ptr[i]) + fanout;
        for (uint32_t base = s; base < (uint32_t)e && !FILL; base += 1024) {
            int32_t u[4];
            bool ok[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t p = base + r * 256 + tid;
                ok[r] = p < (uint32_t)e;
                u[r] = ok[r] ? col_idx[p] : 0;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool inner = in_set(tbits, u[r]);     // u = 0 where the thread has no entry: a valid probe
                n_in += ok[r] && inner;
                n_ext += ok[r] && !inner;
            }
        }
        if (!FILL) {
            block_sum2(n_in, n_ext, s_a, s_b);
            if (tid == 0) counts[i] = n_in + (n_ext < fanout ? n_ext : fanout);
            continue;
        }
        uint64_t thr_k = ~0ull;
        int32_t thr_u = 0x7fffffff;
        if (fanout == 0) {
            thr_k = 0ull;
            thr_u = -1;
        }
        const int32_t aim = fanout <= kSbListCap / 2 ? guess_count(fanout) : kSbListCap;
        bool found = false;
        if (fanout > 0 && n_ext > fanout && aim <= kSbListCap / 2) {   // uniform over the workgroup
            const uint64_t guess = key_guess(aim, n_ext);
            if (tid == 0) s_n = 0;
            __syncthreads();
            for (int64_t base = s; base < e; base += 1024) {
                int32_t u[4];
                bool ok[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t p = base + r * 256 + tid;
                    ok[r] = p < e;
                    u[r] = ok[r] ? col_idx[p] : 0;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) ok[r] = ok[r] && !in_set(tbits, u[r]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint64_t k = edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)u[r]);
                    if (ok[r] && k <= guess) {
                        const int pos = atomicAdd(&s_n, 1);   // the order of the list does not matter
                        if (pos < kSbListCap) {
                            s_key[pos] = k;
                            s_id[pos] = u[r];
                        }
                    }
                }
            }
            __syncthreads();
            const int32_t n_list = s_n;
            found = n_list >= fanout && n_list <= kSbListCap;
            if (found) {
                if (tid < kWave) {
                    constexpr int NP = kSbListCap / kWave;
                    uint64_t k[NP];
                    int32_t u[NP];
                    uint32_t cand = 0u;
#pragma unroll
                    for (int j = 0; j < NP; ++j) {
                        const bool in = j * kWave + tid < n_list;
                        k[j] = in ? s_key[j * kWave + tid] : ~0ull;
                        u[j] = in ? s_id[j * kWave + tid] : 0x7fffffff;
                        cand |= in ? 1u << j : 0u;
                    }
                    group_kth<NP, kWave>(k, u, cand, fanout, true, thr_k, thr_u);
                    if (tid == 0) {
                        s_k[0] = thr_k;
                        s_u[0] = thr_u;
                    }
                }
                __syncthreads();
                thr_k = s_k[0];
                thr_u = s_u[0];
                __syncthreads();
            }
        }
        if (fanout > 0 && n_ext > fanout && !found) {   // uniform over the workgroup
            uint64_t prev_k = 0ull;
            int32_t prev_u = -1;
            for (int32_t round = 0; round < fanout; ++round) {
                uint64_t best_k = ~0ull;
                int32_t best_u = 0x7fffffff;
                for (uint32_t base = s; base < (uint32_t)e; base += 1024) {
                    int32_t u[4];
                    bool ok[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const uint32_t p = base + r * 256 + tid;
                        ok[r] = p < (uint32_t)e;
                        u[r] = ok[r] ? col_idx[p] : 0;
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (ok[r] && !in_set(tbits, u[r])) {
                            const uint64_t k = edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)u[r]);
                            if (pair_less(prev_k, prev_u, k, u[r]) && pair_less(k, u[r], best_k, best_u)) {
                                best_k = k;
                                best_u = u[r];
                            }
                        }
                    }
                }
                block_min_pair(best_k, best_u, s_k, s_u);
                prev_k = best_k;
                prev_u = best_u;
            }
            thr_k = prev_k;
            thr_u = prev_u;
        }
        // a wavefront takes 256 entries in a row of a step's 1024
        int64_t pos = out_row_ptr[i];
        const int lane = tid & 63, wave = tid >> 6;
        for (uint32_t base = s; base < (uint32_t)e; base += 1024) {
            int32_t u[4];
            uint64_t m[4];
            bool keep[4];
            const uint32_t p0 = base + wave * 256 + lane;
#pragma unroll
            for (int r = 0; r < 4; ++r) u[r] = p0 + r * kWave < (uint32_t)e ? col_idx[p0 + r * kWave] : 0;
            int mine = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                keep[r] = in_set(tbits, u[r]) || !pair_less(thr_k, thr_u, edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)u[r]), u[r]);
                keep[r] = keep[r] && p0 + r * kWave < (uint32_t)e;
                m[r] = __ballot(keep[r]);
                mine += __popcll(m[r]);
            }
            if (lane == 0) s_part[wave] = mine;
            __syncthreads();
            int64_t my = pos;
            for (int w = 0; w < 4; ++w) {
                if (w < wave) my += s_part[w];
                pos += s_part[w];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t q = my + __popcll(m[r] & ((1ull << lane) - 1ull));
                if (keep[r] && q < capacity) out_col_idx[q] = u[r];
                my += __popcll(m[r]);
            }
            __syncthreads();     // s_part has been read
        }
    }
}

}  // namespace gnnhot

using namespace gnnhot;

extern "C" int32_t gnn_sample_boundary(const gnn_csr* g, const uint32_t* target_bitmap, const int32_t* targets, int32_t n_targets,
                                       int32_t fanout, int32_t hops, uint64_t seed, int32_t* out_row_ptr, int32_t* out_col_idx,
                                       int64_t out_capacity, int64_t* out_nnz, int64_t* out_nnz_host, void* ws, size_t* ws_bytes,
                                       void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_CHECK(check_csr(g, "g"));
    GNN_REQUIRE(fanout >= 0, GNN_ERR_INVALID_ARG, "fanout < 0");
    GNN_REQUIRE(hops == 1, GNN_ERR_UNSUPPORTED, "only hops = 1 is implemented (got %d)", hops);
    GNN_REQUIRE(n_targets >= 0, GNN_ERR_INVALID_ARG, "n_targets < 0");
    const int32_t n_blocks = offsets_scan_blocks(n_targets);
    WsCarver carve(ws);
    int32_t* counts = carve.take<int32_t>((size_t)n_targets + 1);
    int32_t* sums = carve.take<int32_t>((size_t)n_blocks + 1);
    int32_t* medq = carve.take<int32_t>((size_t)n_targets + 1);   // positions (in `targets`) of the rows of 65 to 1024 entries
    int32_t* hubq = carve.take<int32_t>((size_t)n_targets + 1);   // ... and of the longer ones
    RowCtrl* ctrl = carve.take<RowCtrl>(1);
    bool query;
    GNN_CHECK(ws_protocol(ws, ws_bytes, carve.used, &query));
    if (query) return GNN_OK;
    GNN_REQUIRE(out_row_ptr != nullptr, GNN_ERR_INVALID_ARG, "out_row_ptr is NULL");
    GNN_REQUIRE(n_targets == 0 || (targets != nullptr && target_bitmap != nullptr), GNN_ERR_INVALID_ARG, "targets / bitmap is NULL");
    // grid-stride: one queue append per workgroup
    const int wave_grid = queue_grid(n_targets, g->nnz, kRowsPerWg, n_targets < kSbManyRows ? kRowGrid : 2 * kRowGrid);
    if (n_targets > 0) {   // both passes queue their long rows afresh (workspace contents do not survive a call)
        fill_kernel<int32_t><<<1, 64, 0, stream>>>((int32_t*)ctrl, (int64_t)(sizeof(RowCtrl) / sizeof(int32_t)), 0);
        GNN_LAUNCH_CHECK("fill_kernel");
    }
    const int long_grid = 2048;   // grid-stride over the queues, whose lengths only the device knows

    if (out_col_idx == nullptr) {  // count pass
        GNN_REQUIRE(out_nnz != nullptr, GNN_ERR_INVALID_ARG, "out_nnz is NULL");
        if (n_targets > 0) {
            sb_count_kernel<<<wave_grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, g->n_rows, target_bitmap, targets, n_targets, fanout,
                                                           counts, medq, hubq, ctrl);
            GNN_LAUNCH_CHECK("sb_count_kernel");
            sb_medium_rows_kernel<false><<<long_grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, target_bitmap, targets, medq, ctrl, fanout,
                                                                        0ull, counts, nullptr, nullptr, 0);
            GNN_LAUNCH_CHECK("sb_medium_rows_kernel");
            sb_long_rows_kernel<false><<<long_grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, target_bitmap, targets, hubq, ctrl, fanout,
                                                                      0ull, counts, nullptr, nullptr, 0);
            GNN_LAUNCH_CHECK("sb_long_rows_kernel");
        }
        GNN_CHECK(counts_to_offsets(counts, n_targets, sums, out_row_ptr, out_nnz, stream));
        if (out_nnz_host != nullptr) {
            GNN_HIP(hipMemcpyAsync(out_nnz_host, out_nnz, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
            GNN_HIP(hipStreamSynchronize(stream));
        }
        return GNN_OK;
    }
    GNN_REQUIRE(out_capacity >= 0, GNN_ERR_INVALID_ARG, "out_capacity < 0");
    if (n_targets > 0) {
        // seed + hop is mixed once on the host side of the launch (same function as on the device)
        const uint64_t x = mix64(seed + (uint64_t)hops);
        sb_fill_kernel<<<wave_grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, g->n_rows, target_bitmap, targets, n_targets, fanout, x,
                                                      out_row_ptr, out_col_idx, out_capacity, medq, hubq, ctrl);
        GNN_LAUNCH_CHECK("sb_fill_kernel");
        sb_medium_rows_kernel<true><<<long_grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, target_bitmap, targets, medq, ctrl, fanout, x,
                                                                   nullptr, out_row_ptr, out_col_idx, out_capacity);
        GNN_LAUNCH_CHECK("sb_medium_rows_kernel");
        sb_long_rows_kernel<true><<<long_grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, target_bitmap, targets, hubq, ctrl, fanout, x,
                                                                 nullptr, out_row_ptr, out_col_idx, out_capacity);
        GNN_LAUNCH_CHECK("sb_long_rows_kernel");
    }
    return GNN_OK;
}
