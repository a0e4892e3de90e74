// Layer-wise sampling as a per-layer edge mask (paper section 5.2: for layer-wise sampling methods the maskings are
// generated per layer and the layer aggregates through them).  The one-hop graph is never rebuilt: a layer's mask is
// one bit per CSR entry, which the aggregation kernels test next to their dist filter.
//
//   lm_mask_kernel       sixteen lanes per listed row of up to 64 entries (four per lane): a row's keep decision is
//                        "(key, id) <= threshold pair".  A tile of sixteen consecutive entries becomes one 16-bit
//                        ballot that lane 0 ORs into the bitmap (at most two words), so the result does not depend
//                        on which group runs first.  The threshold rule has a fixed pair; the fanout rule selects its
//                        pair in registers (group_kth).
//   lm_mask_long_kernel  the longer rows, a wavefront each.  Up to 1024 entries the fanout rule holds the upper halves of the row's
//                        keys in registers (up to 256 entries in a quarter of them: the rounds look at every place); beyond,
//                        one sweep lists the entries between two guessed keys in LDS (the keys are uniform: the pair lies
//                        between them, and they hold some 12 * sqrt(fanout) entries) and counts those below; the pair is
//                        selected from that list.  If nothing lies below (fanouts up to 58), the bits are written from the
//                        list, else by a second sweep.  Where the guess fails, or
//                        the fanout is too large for the list (above 4624), `fanout` rounds over the row itself find the pair.
//   lm_transpose_kernel  the same mask in the positions of the transposed graph (backward aggregation): entry q =
//                        (row u, column v) of the transposed graph looks up u in row v of the graph by binary search.
//   lm_mask_t_kernel     the fast way to the same transposed mask: both rules are "(key, id) <= the row's threshold
//                        pair", so with the pairs of the forward rows kept (12 bytes per row) an entry of the
//                        transposed graph is decided by one hash and one random read of a key - the id is read where the
//                        keys are equal.  A workgroup takes 4096 consecutive entries whatever rows they belong to, so
//                        every word of the bitmap has one writer: no atomics, nothing to clear, no long rows.
// Bound: the random reads (transposed), the hash (two 64-bit multiplications a mix) and the selection.  Measured on a
// 1.2M-vertex / 60M-entry power-law graph, fanout 10: forward and transposed mask 2.61 -> 0.65 ms (forward 1.5 -> 0.33,
// transposed 1.09 -> 0.31, its random reads into a 2.4 MB table), against `fanout` rounds over 64-bit pairs and a lane group
// per row of the transposed graph.  Of the forward mask, long rows 335 us with whole keys in all registers whatever the length and two
// sweeps over rows above 1024, 288 by length and with upper halves, 177 with one sweep; short rows 196, 170 with half of the
// places where no row of the wavefront has more than 32.  300 000 vertices of degree 190, fanout 15, both masks: 797 -> 575.
#include "common.h"
#include "hashkey.h"
#include <algorithm>

namespace gnnhot {

constexpr int kLmLanes = 16;

__device__ __forceinline__ uint32_t lm_group_ballot(bool p, int sub) { return (uint32_t)((__ballot(p) >> (sub * kLmLanes)) & 0xffffu); }

// ORs the 16 bits `m` (bit i = entry p0 + i) into the bitmap; called by one lane of the group
__device__ __forceinline__ void lm_or_bits(uint32_t* __restrict__ bits, int64_t p0, uint32_t m) {
    if (m == 0u) return;
    const int sh = (int)(p0 & 31);
    atomicOr(&bits[p0 >> 5], m << sh);
    if (sh > 16 && (m >> (32 - sh)) != 0u) atomicOr(&bits[(p0 >> 5) + 1], m >> (32 - sh));
}

constexpr int kLmShortRow = 64;              // rows up to this length: sixteen lanes, longer ones: a wavefront
constexpr int kLmRegRow = 16 * kWave;        // fanout rule: rows up to this length stay in a wavefront's registers
constexpr int kLmListCap = 256;              // pairs a wavefront lists in LDS for fanouts up to 144
constexpr int kLmListCapWide = 1024;         // ... and above (48 KB a workgroup instead of 12)

// Entries a row's list holds, with room for six standard deviations.
static inline int32_t lm_list_need(int32_t fanout) {
    const int32_t aim = fanout < guess_spread(fanout) ? fanout + guess_spread(fanout) : 2 * guess_spread(fanout);
    return aim + 6 * (int32_t)ceilf(sqrtf((float)aim));
}

__global__ __launch_bounds__(256) void lm_mask_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                      const int32_t* __restrict__ rows, int32_t n_active, int32_t rule, int32_t fanout,
                                                      uint64_t threshold, uint64_t seed_layer_mixed, uint32_t* __restrict__ bits,
                                                      int32_t* __restrict__ kept_len, uint64_t* __restrict__ row_thr_key,
                                                      int32_t* __restrict__ row_thr_id) {
    constexpr int kPerLane = kLmShortRow / kLmLanes;
    const int lane = lane_id(), sub = lane / kLmLanes, sl = lane % kLmLanes;
    const int64_t groups = ((int64_t)gridDim.x * blockDim.x) / kLmLanes;
    // the loop bound is uniform over the wavefront: its four groups take consecutive rows
    for (int64_t base = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 4; base < n_active; base += groups) {
        const int64_t i = base + sub;
        int32_t v = 0, s = 0, e = 0;
        bool mine = i < n_active;
        if (mine) {
            v = rows ? rows[i] : (int32_t)i;
            s = row_ptr[v];
            e = row_ptr[v + 1];
        }
        if (e - s > kLmShortRow) {   // lm_mask_long_kernel takes this row
            mine = false;
            e = s;
        }
        int32_t u[kPerLane];
        uint64_t key[kPerLane];
        uint32_t cand = 0u;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const uint32_t p = (uint32_t)s + j * kLmLanes + sl;   // (past the row's end, a position may not fit an int32_t)
            u[j] = p < (uint32_t)e ? col_idx[p] : -1;
        }
        // most wavefronts have four rows of up to 32 entries: hash and select among half of the places then
        const bool half = __ballot(e - s > kLmShortRow / 2) == 0ull;   // uniform over the wavefront
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            key[j] = ~0ull;
            if (j < kPerLane / 2 || !half) key[j] = edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)(u[j] >= 0 ? u[j] : 0));
            cand |= u[j] >= 0 ? 1u << j : 0u;
        }
        // pairs (key, id) <= (thr_k, thr_u) are kept
        uint64_t thr_k = threshold;
        int32_t thr_u = 0x7fffffff;
        if (rule == GNN_LAYER_MASK_FANOUT) {   // uniform over the grid
            thr_k = ~0ull;
            if (fanout == 0) {
                thr_k = 0ull;
                thr_u = -1;  // nothing is <= (0, -1): ids are non-negative
            }
            const bool need = fanout > 0 && e - s > fanout;  // uniform over the 16-lane group
            if (__ballot(need) != 0ull) {
                if (half) {
                    const uint64_t k2[2] = {key[0], key[1]};
                    const int32_t u2[2] = {u[0], u[1]};
                    group_kth<2, kLmLanes>(k2, u2, cand, fanout, need, thr_k, thr_u);
                } else {
                    group_kth<kPerLane, kLmLanes>(key, u, cand, fanout, need, thr_k, thr_u);
                }
            }
        }
        int32_t kept = 0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            if (j >= kPerLane / 2 && half) break;   // uniform over the wavefront
            const bool keep = u[j] >= 0 && !pair_less(thr_k, thr_u, key[j], u[j]);
            const uint32_t m = lm_group_ballot(keep, sub);
            kept += __popc(m);
            if (sl == 0) lm_or_bits(bits, (int64_t)s + j * kLmLanes, m);
        }
        if (sl == 0 && mine) {
            kept_len[v] = kept;
            if (row_thr_key) {
                row_thr_key[v] = thr_k;
                row_thr_id[v] = thr_u;
            }
        }
    }
}

// ORs the 64 bits `m` (bit i = entry p0 + i) into the bitmap; called by a whole wavefront, three lanes write
__device__ __forceinline__ void lm_or_tile(uint32_t* __restrict__ bits, int64_t p0, uint64_t m) {
    const int lane = lane_id(), sh = (int)(p0 & 31);
    if (lane > 2) return;
    const uint64_t low = m << sh;
    const uint32_t w = lane == 0 ? (uint32_t)low : (lane == 1 ? (uint32_t)(low >> 32) : (sh ? (uint32_t)(m >> (64 - sh)) : 0u));
    if (w != 0u) atomicOr(&bits[(p0 >> 5) + lane], w);
}

// The `rank`-th smallest pair of a row, one round over the row for each; HALF: among those whose keys have this upper half.
template <bool HALF>
__device__ __forceinline__ void lm_pair_by_rounds(const int32_t* __restrict__ col_idx, int32_t v, int32_t s, int32_t e, int32_t rank,
                                                  uint64_t seed_layer_mixed, uint32_t half, uint64_t& thr_k, int32_t& thr_u) {
    const int lane = lane_id();
    uint64_t prev_k = 0ull;
    int32_t prev_u = -1;
    for (int32_t round = 0; round < rank; ++round) {
        uint64_t best_k = ~0ull;
        int32_t best_u = 0x7fffffff;
        for (uint32_t p = (uint32_t)s + lane; p < (uint32_t)e; p += kWave) {
            const int32_t u = col_idx[p];
            const uint64_t k = edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)u);
            if (HALF && (uint32_t)(k >> 32) != half) continue;
            if (pair_less(prev_k, prev_u, k, u) && pair_less(k, u, best_k, best_u)) {
                best_k = k;
                best_u = u;
            }
        }
        wave_min_pair(best_k, best_u);
        prev_k = best_k;
        prev_u = best_u;
    }
    thr_k = prev_k;
    thr_u = prev_u;
}

// A row of up to NP * 64 entries by the fanout rule: finds the pair, writes the bits, returns how many are kept.  A lane holds ids and
// the keys' upper halves; a whole key is made again where its half decides nothing: for the pair itself, and where two of the
// smallest halves are equal (about n^2 / 2^33 of the rows).
template <int NP>
__device__ __forceinline__ int32_t lm_row_in_registers(const int32_t* __restrict__ col_idx, uint32_t* __restrict__ bits, int32_t v, int32_t s,
                                                       int32_t e, int32_t fanout, uint64_t seed_layer_mixed, uint64_t& thr_k, int32_t& thr_u) {
    const int lane = lane_id();
    int32_t u[NP];
    uint32_t half[NP], cand = 0u;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const uint32_t p = (uint32_t)s + j * kWave + lane;
        u[j] = p < (uint32_t)e ? col_idx[p] : -1;
        cand |= u[j] >= 0 ? 1u << j : 0u;
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        half[j] = ~0u;
        if ((uint32_t)s + j * kWave < (uint32_t)e) {   // uniform over the wavefront
            const uint64_t k = edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)(u[j] >= 0 ? u[j] : 0));
            half[j] = u[j] >= 0 ? (uint32_t)(k >> 32) : ~0u;
        }
    }
    uint32_t top = fanout > 0 ? ~0u : 0u;      // entries up to this half stay
    bool whole = true;                         // the half decides
    if (fanout > 0 && e - s > fanout) {
        whole = wave_kth_half<NP>(half, u, cand, fanout, top, thr_u);
        if (whole) thr_k = edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)thr_u);
        else {
            uint32_t kth;
            const int32_t rank = wave_kth_rank<NP>(half, cand, fanout, kth);
            lm_pair_by_rounds<true>(col_idx, v, s, e, rank, seed_layer_mixed, kth, thr_k, thr_u);
        }
    }
    int32_t kept = 0;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        if ((uint32_t)s + j * kWave < (uint32_t)e) {   // uniform over the wavefront
            bool keep = u[j] >= 0 && fanout > 0 && half[j] <= top;
            if (!whole) keep = u[j] >= 0 && !pair_less(thr_k, thr_u, edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)(u[j] >= 0 ? u[j] : 0)), u[j]);
            const uint64_t m = __ballot(keep);
            kept += __popcll(m);
            lm_or_tile(bits, (int64_t)s + j * kWave, m);
        }
    }
    return kept;
}

// The fanout rule's pair of a row of more than kLmRegRow (> fanout) entries; see the head of the file.  Where the list holds every
// entry below the pair it writes the bits, too, and returns how many are kept, else -1.
template <int CAP>
__device__ __forceinline__ int32_t lm_pair_of_hub(const int32_t* __restrict__ col_idx, uint32_t* __restrict__ bits, int32_t v, int32_t s, int32_t e,
                                               int32_t fanout, uint64_t seed_layer_mixed, uint64_t* key, int32_t* at, uint64_t& thr_k,
                                               int32_t& thr_u) {
    constexpr int kU = 4;
    const int lane = lane_id();
    const uint64_t lanes_below = (1ull << lane) - 1ull;
    const int32_t spread = guess_spread(fanout);
    int32_t n_list = 0, n_below = 0;
    if (fanout <= CAP * 8) {   // (the list may hold it: see lm_list_need)
        const uint64_t low = fanout > spread ? key_guess(fanout - spread, e - s) : 0ull, high = key_guess(fanout + spread, e - s);
        for (int64_t p = s; p < e; p += kU * kWave) {
            int32_t u[kU];
#pragma unroll
            for (int j = 0; j < kU; ++j) u[j] = p + j * kWave + lane < e ? col_idx[p + j * kWave + lane] : -1;
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint64_t k = edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)(u[j] >= 0 ? u[j] : 0));
                const bool take = u[j] >= 0 && k >= low && k <= high;
                n_below += __popcll(__ballot(u[j] >= 0 && k < low));
                const uint64_t m = __ballot(take);
                const int32_t pos = n_list + __popcll(m & lanes_below);
                if (take && pos < CAP) {
                    key[pos] = k;
                    at[pos] = (int32_t)(p + j * kWave + lane);
                }
                n_list += __popcll(m);
            }
        }
        wave_lds_sync();
    }
    if (n_below < fanout && n_below + n_list >= fanout && n_list <= CAP) {   // uniform over the wavefront
        constexpr int NP = CAP / kWave;
        uint64_t k[NP];
        int32_t u[NP];
        uint32_t cand = 0u;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const bool in = j * kWave + lane < n_list;
            k[j] = in ? key[j * kWave + lane] : ~0ull;
            u[j] = in ? col_idx[at[j * kWave + lane]] : 0x7fffffff;
            cand |= in ? 1u << j : 0u;
        }
        group_kth<NP, kWave>(k, u, cand, fanout - n_below, true, thr_k, thr_u);
        int32_t kept = -1;
        if (n_below == 0) {     // uniform over the wavefront
            kept = 0;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const bool keep = ((cand >> j) & 1u) != 0u && !pair_less(thr_k, thr_u, k[j], u[j]);
                kept += __popcll(__ballot(keep));
                if (keep) {
                    const int32_t p = at[j * kWave + lane];
                    atomicOr(&bits[p >> 5], 1u << (p & 31));
                }
            }
        }
        wave_lds_sync();   // the list is read before the next row overwrites it
        return kept;
    }
    lm_pair_by_rounds<false>(col_idx, v, s, e, fanout, seed_layer_mixed, 0u, thr_k, thr_u);
    return -1;
}

// Rows longer than kLmShortRow: a wavefront looks at up to kLmLook rows of the list and takes the long ones one by one.
// 64 wavefronts share a stretch of the list and take its rows in turn, one row of every 64: long rows that follow each other
// (a graph numbered by degree, a list of hubs) go to different wavefronts, a list of fewer rows than the chip holds wavefronts
// gives each of its rows one, and what runs at a time still lies close together.  From one group of 64 rows to the next the
// wavefronts move by 37 places, so that long rows at regular distances do not meet in one of them.
// Measured (fanout 10): 64 rows of 100 000 entries at the head of a list 10.5 ms with sixteen consecutive rows for a wavefront,
// then 0.74; 2000 rows of 490 entries 121 us, then 39; 1.2M rows of 50 (with the short ones) 541 us, then 533 - 595 with
// rows as far apart as there are wavefronts, which then run all over the graph at a time.
constexpr int kLmLook = 32;
constexpr int kLmShare = 64;
constexpr int kLmWaves = 8192;    // fewer rows than this (twice what the chip holds at a time): one for a wavefront

template <int CAP>
__global__ __launch_bounds__(256) void lm_mask_long_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                           const int32_t* __restrict__ rows, int32_t n_active, int32_t rule, int32_t fanout,
                                                           uint64_t threshold, uint64_t seed_layer_mixed, uint32_t* __restrict__ bits,
                                                           int32_t* __restrict__ kept_len, uint64_t* __restrict__ row_thr_key,
                                                           int32_t* __restrict__ row_thr_id, int32_t look) {
    __shared__ uint64_t s_key[4][CAP];
    __shared__ int32_t s_at[4][CAP];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int64_t wave_g = (int64_t)blockIdx.x * 4 + wave;
    const int64_t group = wave_g / kLmShare * look + lane;       // of 64 rows; lanes 0 .. look - 1
    const int64_t i = group * kLmShare + ((wave_g + 37 * group) & (kLmShare - 1));
    int32_t v_l = 0, s_l = 0, e_l = 0;
    if (lane < look && i < n_active) {
        v_l = rows ? rows[i] : (int32_t)i;
        s_l = row_ptr[v_l];
        e_l = row_ptr[v_l + 1];
    }
    uint64_t todo = __ballot(e_l - s_l > kLmShortRow);
    while (todo) {   // uniform over the wavefront
        const int from = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1ull;
        const int32_t v = __builtin_amdgcn_readlane(v_l, from), s = __builtin_amdgcn_readlane(s_l, from),
                      e = __builtin_amdgcn_readlane(e_l, from);
        uint64_t thr_k = threshold;   // pairs above (thr_k, thr_u) are out
        int32_t thr_u = 0x7fffffff, kept = 0;
        const bool by_fanout = rule == GNN_LAYER_MASK_FANOUT;
        if (by_fanout) {
            thr_k = fanout == 0 ? 0ull : ~0ull;
            thr_u = fanout == 0 ? -1 : 0x7fffffff;
        }
        if (by_fanout && e - s <= kLmRegRow / 4) {
            kept = lm_row_in_registers<kLmRegRow / 4 / kWave>(col_idx, bits, v, s, e, fanout, seed_layer_mixed, thr_k, thr_u);
        } else if (by_fanout && e - s <= kLmRegRow) {
            kept = lm_row_in_registers<kLmRegRow / kWave>(col_idx, bits, v, s, e, fanout, seed_layer_mixed, thr_k, thr_u);
        } else {
            int32_t written = -1;
            if (by_fanout && fanout > 0 && e - s > fanout)
                written = lm_pair_of_hub<CAP>(col_idx, bits, v, s, e, fanout, seed_layer_mixed, s_key[wave], s_at[wave], thr_k, thr_u);
            if (written >= 0) kept = written;
            constexpr int kU = 4;
            for (int64_t p = s; p < e && written < 0; p += kU * kWave) {
                int32_t u[kU];
#pragma unroll
                for (int j = 0; j < kU; ++j) u[j] = p + j * kWave + lane < e ? col_idx[p + j * kWave + lane] : -1;
#pragma unroll
                for (int j = 0; j < kU; ++j) {
                    const uint64_t k = edge_key(seed_layer_mixed, (uint64_t)v, (uint64_t)(u[j] >= 0 ? u[j] : 0));
                    const uint64_t m = __ballot(u[j] >= 0 && !pair_less(thr_k, thr_u, k, u[j]));
                    kept += __popcll(m);
                    if (m != 0ull) lm_or_tile(bits, p + j * kWave, m);   // uniform over the wavefront
                }
            }
        }
        if (lane == 0) {
            kept_len[v] = kept;
            if (row_thr_key) {
                row_thr_key[v] = thr_k;
                row_thr_id[v] = thr_u;
            }
        }
    }
}

// The mask of a layer in the positions of the transposed graph, from the per-row threshold pairs the forward pass
// left: entry q = (row u, column v) of the transposed graph is the forward entry (v <- u), kept iff
// (key(v, u), u) <= (row_thr_key[v], row_thr_id[v]).
constexpr int kLmChunk = 4096;   // entries per workgroup
// A chunk whose rows (the empty ones between its first and its last entry among them) are more than this searches the row of
// every entry, four entries of a thread side by side, instead of walking the rows one for each thread: 128 dependent loads
// against four times the depth of the search.  The call with 1M / 8M empty rows in one place of the graph: walked 1.16 /
// 8.9 ms, searched 31 / 38 us (without any 23 us).
constexpr int kLmWalk = 8 * kLmChunk;

// TOPS: an entry reads the upper 16 bits of its row's key out of a table of their own; the pair itself is read where those of both
// keys are equal, one entry in 65 536.  What bounds the entries is a line out of an L2 each (200 G/s, 25 TB/s) where the table fits, else the
// misses: 1.2 M rows of 50, power-law 428 -> 313 us, uniform 660 -> 321, the copy (10 us) included; 2 M of 30 599 -> 373, 831 -> 415.
template <bool TOPS>
__global__ __launch_bounds__(256) void lm_mask_t_kernel(int32_t n_t, int64_t nnz, const int32_t* __restrict__ rpT,
                                                        const int32_t* __restrict__ ciT, const uint64_t* __restrict__ row_thr_key,
                                                        const int32_t* __restrict__ row_thr_id, const uint16_t* __restrict__ tops,
                                                        uint64_t seed_layer_mixed, uint32_t* __restrict__ keep_t) {
    constexpr int kTiles = kLmChunk / 256;          // 64-entry tiles per wavefront
    __shared__ int32_t s_start[kLmChunk];           // at the first entry of a row: its number relative to the chunk's first row
    __shared__ int32_t s_last[4], s_row[2];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int64_t q0 = (int64_t)blockIdx.x * kLmChunk;
    const int64_t q1 = q0 + kLmChunk < nnz ? q0 + kLmChunk : nnz;
    for (int t = threadIdx.x; t < kLmChunk; t += 256) s_start[t] = 0;
    if (wave < 2) {   // the rows that hold the first and the last entry: a search with 64 probes a step; rpT[lo] <= q < rpT[hi]
        const int64_t q = wave == 0 ? q0 : q1 - 1;
        int64_t lo = 0, hi = n_t;
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + 63) / 64;
            const int64_t at = lo + step * (lane + 1);
            const int n_below = __popcll(__ballot(at < hi && (int64_t)rpT[at < hi ? at : lo] <= q));
            lo += step * n_below;
            hi = lo + step < hi ? lo + step : hi;
        }
        if (lane == 0) s_row[wave] = (int32_t)lo;
    }
    __syncthreads();
    const int32_t row0 = s_row[0], row1 = s_row[1];
    if (row1 - row0 <= kLmWalk) {   // uniform over the workgroup
        for (int64_t r = (int64_t)row0 + 1 + threadIdx.x; r <= row1; r += 256)
            atomicMax(&s_start[rpT[r] - q0], (int32_t)(r - row0));   // of several rows that start here all but the last are empty
    } else {
        constexpr int kQ = 4;   // searches side by side
        for (int t0 = (int)threadIdx.x; t0 < kLmChunk; t0 += 256 * kQ) {
            int32_t lo[kQ], hi[kQ];
#pragma unroll
            for (int j = 0; j < kQ; ++j) {
                lo[j] = row0;
                hi[j] = row1 + 1;
            }
            for (int64_t width = (int64_t)row1 + 1 - row0; width > 1; width = (width + 1) / 2) {   // uniform over the workgroup
#pragma unroll
                for (int j = 0; j < kQ; ++j) {
                    const int32_t mid = lo[j] + (hi[j] - lo[j]) / 2;   // (lo itself once the search has ended)
                    if (rpT[mid] <= q0 + t0 + j * 256) lo[j] = mid;
                    else hi[j] = mid;
                }
            }
#pragma unroll
            for (int j = 0; j < kQ; ++j) {
                const int t = t0 + j * 256;
                if (q0 + t < q1 && lo[j] > row0 && rpT[lo[j]] == q0 + t) s_start[t] = lo[j] - row0;
            }
        }
    }
    __syncthreads();
    // the last row that starts in each wavefront's part
    int32_t last = 0;
    for (int t = 0; t < kTiles; ++t) last = max(last, s_start[(wave * kTiles + t) * kWave + lane]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) last = max(last, __shfl_xor(last, d, kWave));
    if (lane == 0) s_last[wave] = last;
    __syncthreads();
    int32_t row = 0;   // of the entry before the tile, relative to row0
    for (int w = 0; w < wave; ++w) row = max(row, s_last[w]);
    constexpr int kU = 4;
    for (int t = 0; t < kTiles; t += kU) {
        const int64_t p0 = q0 + (wave * kTiles + t) * kWave;
        if (p0 >= q1) break;   // uniform over the wavefront
        int32_t u[kU], v[kU];
        uint64_t thr[TOPS ? 1 : kU];
        uint32_t top[TOPS ? kU : 1];
#pragma unroll
        for (int j = 0; j < kU; ++j) v[j] = p0 + j * kWave + lane < q1 ? ciT[p0 + j * kWave + lane] : -1;
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int32_t st = s_start[(wave * kTiles + t + j) * kWave + lane];
            const uint64_t starts = __ballot(st != 0);
            const uint64_t upto = starts & (~0ull >> (63 - lane));
            const int32_t mine = __shfl(st, upto ? 63 - __clzll((long long)upto) : 0, kWave);
            u[j] = row0 + (upto ? mine : row);
            if (starts) row = __shfl(st, 63 - __clzll((long long)starts), kWave);   // uniform over the wavefront
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            if (TOPS) top[TOPS ? j : 0] = tops[v[j] >= 0 ? v[j] : 0];
            else thr[TOPS ? 0 : j] = row_thr_key[v[j] >= 0 ? v[j] : 0];
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const uint64_t k = edge_key(seed_layer_mixed, (uint64_t)(v[j] >= 0 ? v[j] : 0), (uint64_t)u[j]);
            bool bit;
            if (TOPS) {
                const uint32_t t = (uint32_t)(k >> 48);
                bit = v[j] >= 0 && t < top[TOPS ? j : 0];
                if (v[j] >= 0 && t == top[TOPS ? j : 0]) bit = !pair_less(row_thr_key[v[j]], row_thr_id[v[j]], k, u[j]);
            } else {
                bit = v[j] >= 0 && k <= thr[TOPS ? 0 : j];
                if (bit && k == thr[TOPS ? 0 : j]) bit = u[j] <= row_thr_id[v[j]];
            }
            const uint64_t m = __ballot(bit);
            const int64_t p = p0 + j * kWave + lane * 32;
            if (lane < 2 && p < q1) keep_t[p >> 5] = (uint32_t)(m >> (32 * lane));
        }
    }
}

__global__ __launch_bounds__(256) void lm_tops_kernel(const uint64_t* __restrict__ row_thr_key, uint16_t* __restrict__ tops, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        tops[i] = (uint16_t)(row_thr_key[i] >> 48);
}

// The line: a table of keys that an L2 (4 MB) holds anyway gains nothing, and fewer entries a row would not pay for the copy (measured down to
// 5).  us, keys / tops, power-law and uniform graphs: 300 000 rows of 5 14.5 / 14.5, 13.4 / 15.3, of 10 22.5 / 22.9, 23.0 / 25.8, of 190 245 / 226,
// 254 / 251; 500 000 of 20 62.2 / 58.5, 68.7 / 63.4, of 100 253 / 214, 268 / 233; 1.2 M of 5 45.5 / 42.2, 64.6 / 40.5, of 10 88 / 71, 142 / 79.
static bool lm_takes_tops(const gnn_csr* gT) { return gT->n_cols >= 400000 && gT->nnz >= 4 * (int64_t)gT->n_cols; }

// Clears the bitmap and gives the rows from `first` on the threshold of a row that is not listed (k nullable): nothing is <= (0, -1).
// One launch and only the rows that no other launch writes, against two over everything, the whole forward mask, us: 50 000 rows of 20 24.4 ->
// 21.3, 300 000 of 5 26.2 -> 24.0, 1.2 M of 50 341 -> 334.  (Bits put together per row, one atomic a word, plain stores inside a row: 241 -> 295.)
__global__ __launch_bounds__(256) void lm_init_kernel(uint32_t* __restrict__ bits, int64_t n_words, uint64_t* __restrict__ k, int32_t* __restrict__ u,
                                                      int64_t first, int64_t n) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < n_words; i += stride) bits[i] = 0u;
    if (k == nullptr) return;
    for (int64_t i = first + tid; i < n; i += stride) {
        k[i] = 0ull;
        u[i] = -1;
    }
}

__global__ __launch_bounds__(256) void lm_transpose_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                           const uint32_t* __restrict__ keep, int32_t n_t,
                                                           const int32_t* __restrict__ rpT, const int32_t* __restrict__ ciT,
                                                           uint32_t* __restrict__ keep_t) {
    const int lane = lane_id(), sub = lane / kLmLanes, sl = lane % kLmLanes;
    const int64_t groups = ((int64_t)gridDim.x * blockDim.x) / kLmLanes;
    for (int64_t base = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 4; base < n_t; base += groups) {
        const int64_t u = base + sub;
        int32_t s = 0, e = 0;
        if (u < n_t) {
            s = rpT[u];
            e = rpT[u + 1];
        }
        int len_max = e - s;
        len_max = max(len_max, __shfl_xor(len_max, 16, kWave));
        len_max = max(len_max, __shfl_xor(len_max, 32, kWave));
        for (int32_t off = 0; off < len_max; off += kLmLanes) {
            const uint32_t q = (uint32_t)s + off + sl;
            bool bit = false;
            if (q < (uint32_t)e) {
                const int32_t v = ciT[q];
                int32_t lo = row_ptr[v], hi = row_ptr[v + 1];  // first position of row v whose column is >= u
                while (lo < hi) {
                    const int32_t mid = lo + ((hi - lo) >> 1);
                    if (col_idx[mid] < (int32_t)u) lo = mid + 1;
                    else hi = mid;
                }
                if (lo < row_ptr[v + 1] && col_idx[lo] == (int32_t)u) bit = (keep[lo >> 5] >> (lo & 31)) & 1u;
            }
            const uint32_t m = lm_group_ballot(bit, sub);
            if (sl == 0) lm_or_bits(keep_t, (int64_t)s + off, m);
        }
    }
}

}  // namespace gnnhot

using namespace gnnhot;

extern "C" int32_t gnn_layer_edge_mask(const gnn_csr* g, const int32_t* rows, int32_t n_active, int32_t rule, int32_t fanout,
                                       uint64_t threshold, uint64_t seed, int32_t layer, uint32_t* edge_keep, int32_t* kept_len,
                                       uint64_t* row_thr_key, int32_t* row_thr_id, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_CHECK(check_csr(g, "g"));
    GNN_REQUIRE(n_active >= 0, GNN_ERR_INVALID_ARG, "negative row count");
    GNN_REQUIRE(rows != nullptr || n_active <= g->n_rows, GNN_ERR_SHAPE, "n_active %d exceeds n_rows %d", n_active, g->n_rows);
    GNN_REQUIRE(rule == GNN_LAYER_MASK_THRESHOLD || rule == GNN_LAYER_MASK_FANOUT, GNN_ERR_INVALID_ARG, "unknown mask rule %d", rule);
    GNN_REQUIRE(fanout >= 0, GNN_ERR_INVALID_ARG, "fanout < 0");
    GNN_REQUIRE(layer >= 0, GNN_ERR_INVALID_ARG, "layer < 0");
    const int64_t n_words = (g->nnz + 31) / 32;
    GNN_REQUIRE(n_words == 0 || edge_keep != nullptr, GNN_ERR_INVALID_ARG, "edge_keep is NULL");
    GNN_REQUIRE(n_active == 0 || kept_len != nullptr, GNN_ERR_INVALID_ARG, "kept_len is NULL");
    GNN_REQUIRE((row_thr_key == nullptr) == (row_thr_id == nullptr), GNN_ERR_INVALID_ARG, "row_thr_key and row_thr_id go together");
    const int64_t first = rows == nullptr ? n_active : 0, n_clear = std::max(n_words, row_thr_key ? g->n_rows - first : 0);
    if (n_clear > 0) {
        lm_init_kernel<<<grid_for(n_clear, 256, 4096), 256, 0, stream>>>(edge_keep, n_words, row_thr_key, row_thr_id, first, g->n_rows);
        GNN_LAUNCH_CHECK("lm_init_kernel");
    }
    if (n_active > 0) {
        lm_mask_kernel<<<grid_for((int64_t)n_active * kLmLanes, 256, 1 << 15), 256, 0, stream>>>(
            g->row_ptr, g->col_idx, rows, n_active, rule, fanout, threshold, mix64(seed + (uint64_t)layer), edge_keep, kept_len, row_thr_key,
            row_thr_id);
        GNN_LAUNCH_CHECK("lm_mask_kernel");
        if (g->nnz > kLmShortRow) {   // else no row is longer
            const bool wide = rule == GNN_LAYER_MASK_FANOUT && lm_list_need(fanout) > kLmListCap && lm_list_need(fanout) <= kLmListCapWide;
            const int32_t look = n_active > kLmLook * kLmWaves ? kLmLook : (n_active + kLmWaves - 1) / kLmWaves;
            const int64_t groups = ((int64_t)n_active + kLmShare - 1) / kLmShare, stretches = (groups + look - 1) / look;
            const uint32_t grid = (uint32_t)(stretches * (kLmShare / 4));
            const uint64_t mixed = mix64(seed + (uint64_t)layer);
            if (wide)
                lm_mask_long_kernel<kLmListCapWide><<<grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, rows, n_active, rule, fanout,
                                                                                           threshold, mixed, edge_keep, kept_len, row_thr_key,
                                                                                           row_thr_id, look);
            else
                lm_mask_long_kernel<kLmListCap><<<grid, 256, 0, stream>>>(g->row_ptr, g->col_idx, rows, n_active, rule, fanout,
                                                                                       threshold, mixed, edge_keep, kept_len, row_thr_key,
                                                                                       row_thr_id, look);
            GNN_LAUNCH_CHECK("lm_mask_long_kernel");
        }
    }
    return GNN_OK;
}

extern "C" int32_t gnn_transpose_edge_mask(const gnn_csr* g, const gnn_csr* gT, const uint32_t* keep, uint32_t* keep_t, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_CHECK(check_csr(g, "g"));
    GNN_CHECK(check_csr(gT, "gT"));
    GNN_REQUIRE((g->flags & GNN_CSR_SORTED_COLUMNS) != 0, GNN_ERR_UNSUPPORTED, "g must promise sorted columns");
    GNN_REQUIRE(gT->n_rows == g->n_cols && gT->n_cols == g->n_rows, GNN_ERR_SHAPE, "gT is not shaped like the transpose of g");
    const int64_t n_words = (gT->nnz + 31) / 32;
    GNN_REQUIRE(n_words == 0 || (keep != nullptr && keep_t != nullptr), GNN_ERR_INVALID_ARG, "keep or keep_t is NULL");
    if (n_words > 0) {
        fill_kernel<uint32_t><<<grid_for(n_words, 256, 4096), 256, 0, stream>>>(keep_t, n_words, 0u);
        GNN_LAUNCH_CHECK("fill_kernel");
        lm_transpose_kernel<<<grid_for((int64_t)gT->n_rows * kLmLanes, 256, 1 << 15), 256, 0, stream>>>(
            g->row_ptr, g->col_idx, keep, gT->n_rows, gT->row_ptr, gT->col_idx, keep_t);
        GNN_LAUNCH_CHECK("lm_transpose_kernel");
    }
    return GNN_OK;
}

static int32_t mask_transposed(const gnn_csr* gT, const uint64_t* row_thr_key, const int32_t* row_thr_id, uint64_t seed, int32_t layer,
                               uint32_t* keep_t, void* ws, size_t* ws_bytes, hipStream_t stream) {
    GNN_CHECK(check_csr(gT, "gT"));
    GNN_REQUIRE(layer >= 0, GNN_ERR_INVALID_ARG, "layer < 0");
    WsCarver carve(ws);
    uint16_t* const tops = ws_bytes != nullptr && lm_takes_tops(gT) ? carve.take<uint16_t>((size_t)gT->n_cols) : nullptr;
    if (ws_bytes != nullptr) {
        bool query;
        GNN_CHECK(ws_protocol(ws, ws_bytes, carve.used, &query));
        if (query) return GNN_OK;
    }
    const int64_t n_words = (gT->nnz + 31) / 32;
    GNN_REQUIRE(n_words == 0 || (row_thr_key && row_thr_id && keep_t), GNN_ERR_INVALID_ARG, "row_thr_key, row_thr_id or keep_t is NULL");
    if (n_words == 0) return GNN_OK;
    const int grid = (int)((gT->nnz + kLmChunk - 1) / kLmChunk);
    const uint64_t mixed = mix64(seed + (uint64_t)layer);
    if (tops != nullptr) {
        lm_tops_kernel<<<grid_for(gT->n_cols, 256, 4096), 256, 0, stream>>>(row_thr_key, tops, gT->n_cols);
        GNN_LAUNCH_CHECK("lm_tops_kernel");
        lm_mask_t_kernel<true><<<grid, 256, 0, stream>>>(gT->n_rows, gT->nnz, gT->row_ptr, gT->col_idx, row_thr_key, row_thr_id, tops, mixed, keep_t);
    } else {
        lm_mask_t_kernel<false><<<grid, 256, 0, stream>>>(gT->n_rows, gT->nnz, gT->row_ptr, gT->col_idx, row_thr_key, row_thr_id, nullptr, mixed,
                                                          keep_t);
    }
    GNN_LAUNCH_CHECK("lm_mask_t_kernel");
    return GNN_OK;
}

extern "C" int32_t gnn_layer_edge_mask_transposed(const gnn_csr* gT, const uint64_t* row_thr_key, const int32_t* row_thr_id, uint64_t seed,
                                                  int32_t layer, uint32_t* keep_t, void* stream_) {
    return mask_transposed(gT, row_thr_key, row_thr_id, seed, layer, keep_t, nullptr, nullptr, (hipStream_t)stream_);
}

extern "C" int32_t gnn_layer_edge_mask_transposed_ws(const gnn_csr* gT, const uint64_t* row_thr_key, const int32_t* row_thr_id, uint64_t seed,
                                                     int32_t layer, uint32_t* keep_t, void* ws, size_t* ws_bytes, void* stream_) {
    return mask_transposed(gT, row_thr_key, row_thr_id, seed, layer, keep_t, ws, ws_bytes, (hipStream_t)stream_);
}
