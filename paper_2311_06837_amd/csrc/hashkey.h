// Ordering keys of the sampling kernels: the seeded counter-based edge hash of the boundary sampler (paper section
// 5.3; splitmix64's output function) and lexicographic (key, id) comparison.
#pragma once
#include "common.h"

namespace gnnhot {

// splitmix64 output function: golden-ratio increment, two xor-shift-multiply rounds, xor-shift.
__host__ __device__ __forceinline__ uint64_t mix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

__device__ __forceinline__ uint64_t edge_key(uint64_t seed_hop_mixed, uint64_t v, uint64_t u) {
    return mix64(mix64(seed_hop_mixed ^ v) ^ u);
}

__device__ __forceinline__ bool in_set(const uint32_t* __restrict__ bitmap, int32_t u) {
    return (bitmap[u >> 5] >> (u & 31)) & 1u;
}

// (key, id) pairs ordered lexicographically
__device__ __forceinline__ bool pair_less(uint64_t ka, int32_t ua, uint64_t kb, int32_t ub) {
    return ka < kb || (ka == kb && ua < ub);
}

// ---- the k smallest of a row that a lane group holds in registers ------------------------------------------------
// x's minimum over each group of 16 lanes, in every lane of the group
__device__ __forceinline__ uint32_t min16(uint32_t x) {
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));   // row_ror:8
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false));
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false));
    return min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false));
}

// ... over the G lanes of a group (16 or the whole wavefront)
template <int G>
__device__ __forceinline__ uint32_t group_min(uint32_t x) {
    x = min16(x);
    if (G == 16) return x;
    return min(min((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16)),
               min((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48)));
}

// The k-th smallest (key, id) pair of a group's candidates: NP pairs per lane, bit j of `cand` = pair j is a candidate.
// `need` (uniform over the group): the group has more than k >= 1 candidates and wants the pair; the other groups of the
// wavefront only take part.  All lanes call it.
// A round of "smallest above the previous one" over 64-bit keys and ids costs some ten instructions a pair and, lane to
// lane, three LDS shuffles a step.  The rounds here see the upper halves of the keys only: a subtraction and a minimum a
// pair (what lies below `base` wraps around to the top), the lanes meet through DPP.  If the candidates up to the k-th
// upper half are exactly k, that half belongs to the pair in question; otherwise two halves are equal (about n^2 / 2^33 of
// the rows of n entries) and the rounds over whole pairs decide.
template <int NP, int G>
__device__ __forceinline__ void group_kth(const uint64_t (&key)[NP], const int32_t (&id)[NP], uint32_t cand, int32_t k, bool need,
                                          uint64_t& thr_k, int32_t& thr_u) {
    const int lane = lane_id(), first = lane / G * G;
    const uint64_t mine = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull) << first;
    uint32_t base = 0u, top = 0u;
    for (int32_t round = 0; round < k; ++round) {
        uint32_t m = ~0u;
#pragma unroll
        for (int j = 0; j < NP; ++j) m = min(m, ((cand >> j) & 1u ? (uint32_t)(key[j] >> 32) : ~0u) - base);
        top = base + group_min<G>(m);
        base = top + 1u;
    }
    int32_t kept = 0;
    bool has = false;
    uint64_t pk = 0ull;
    int32_t pu = 0;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const uint32_t half = (uint32_t)(key[j] >> 32);
        const bool c = (cand >> j) & 1u;
        kept += __popcll(__ballot(c && half <= top) & mine);
        if (c && half == top) {
            has = true;
            pk = key[j];
            pu = id[j];
        }
    }
    const uint64_t holders = __ballot(has) & mine;
    const int src = holders ? __ffsll((unsigned long long)holders) - 1 : lane;
    pk = __shfl(pk, src, kWave);
    pu = __shfl(pu, src, kWave);
    const bool tie = need && kept != k;
    if (__ballot(tie) != 0ull) {   // uniform over the wavefront
        uint64_t prev_k = 0ull;
        int32_t prev_u = -1;
        for (int32_t round = 0; round < k; ++round) {
            uint64_t best_k = ~0ull;
            int32_t best_u = 0x7fffffff;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                if (((cand >> j) & 1u) && pair_less(prev_k, prev_u, key[j], id[j]) && pair_less(key[j], id[j], best_k, best_u)) {
                    best_k = key[j];
                    best_u = id[j];
                }
            }
#pragma unroll
            for (int d = G / 2; d >= 1; d >>= 1) {
                const uint64_t ok = __shfl_xor(best_k, d, kWave);
                const int32_t ou = __shfl_xor(best_u, d, kWave);
                if (pair_less(ok, ou, best_k, best_u)) {
                    best_k = ok;
                    best_u = ou;
                }
            }
            prev_k = best_k;
            prev_u = best_u;
        }
        if (tie) {
            pk = prev_k;
            pu = prev_u;
        }
    }
    if (need) {
        thr_k = pk;
        thr_u = pu;
    }
}

// The same for a whole wavefront that holds only the upper halves: `cand` and `half` as there (~0u where there is no candidate), more
// than k >= 1 candidates in all.  True: the k candidates with halves up to `top` are the k smallest, and `id` is the k-th's;
// false: the halves do not decide.
template <int NP>
__device__ __forceinline__ bool wave_kth_half(const uint32_t (&half)[NP], const int32_t (&ids)[NP], uint32_t cand, int32_t k, uint32_t& top,
                                              int32_t& id) {
    uint32_t base = 0u;
    top = 0u;
    for (int32_t round = 0; round < k; ++round) {
        uint32_t m = ~0u;
#pragma unroll
        for (int j = 0; j < NP; ++j) m = min(m, half[j] - base);
        top = base + group_min<kWave>(m);
        base = top + 1u;
    }
    int32_t upto = 0;
    bool held = false;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const bool c = (cand >> j) & 1u;
        upto += __popcll(__ballot(c && half[j] <= top));
        const uint64_t h = __ballot(c && half[j] == top);
        if (h != 0ull) {      // uniform over the wavefront
            held = true;
            id = __builtin_amdgcn_readlane(ids[j], __ffsll((unsigned long long)h) - 1);
        }
    }
    return held && upto == k;
}

// Where the halves do not decide: the half of the k-th smallest of the same candidates, counted with repeats (a bisection), and its pair's
// rank (1, 2, ..) among the pairs that share that half.  Two or three do; rounds over all pairs, one for each that is kept, held a
// launch up by themselves (60 000 rows of 700 entries, fanout 600, three such rows: 3.0 ms instead of 2.4).
template <int NP>
__device__ __forceinline__ int32_t wave_kth_rank(const uint32_t (&half)[NP], uint32_t cand, int32_t k, uint32_t& kth) {
    auto upto = [&](uint32_t h) {
        int32_t n = 0;
#pragma unroll
        for (int j = 0; j < NP; ++j) n += __popcll(__ballot(((cand >> j) & 1u) != 0u && half[j] <= h));
        return n;
    };
    uint32_t lo = 0u, hi = ~0u;
    while (lo < hi) {      // uniform over the wavefront
        const uint32_t mid = lo + (hi - lo) / 2u;
        if (upto(mid) >= k) hi = mid;
        else lo = mid + 1u;
    }
    kth = lo;
    return k - (lo > 0u ? upto(lo - 1u) : 0);
}

// The smallest (key, id) pair over the wavefront, in every lane.
__device__ __forceinline__ void wave_min_pair(uint64_t& k, int32_t& u) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint64_t ok = __shfl_xor(k, d, kWave);
        const int32_t ou = __shfl_xor(u, d, kWave);
        if (pair_less(ok, ou, k, u)) {
            k = ok;
            u = ou;
        }
    }
}

// A key that about `want` of n uniformly distributed keys lie at or below (n >= want).
__device__ __forceinline__ uint64_t key_guess(int32_t want, int32_t n) {
    return want >= n ? ~0ull : (~0ull / (uint64_t)n) * (uint64_t)want;
}

// How far from k to aim when the k-th smallest key is wanted: aimed at k + spread keys, fewer than k lie at or below the
// guess in one of a few million rows; aimed at k - spread, k or more do about as rarely.
__host__ __device__ __forceinline__ int32_t guess_spread(int32_t k) { return 6 * (int32_t)ceilf(sqrtf((float)k)) + 10; }
__device__ __forceinline__ int32_t guess_count(int32_t k) { return k + guess_spread(k); }

// ---- a wavefront's list of (key, id) pairs in LDS: the selection step of the traversal ----

// The k-th smallest of the n (> k >= 1) distinct pairs of the list: k rounds of "smallest pair above the previous
// one".  Every lane returns the same pair.
__device__ __forceinline__ void wave_list_kth(const uint64_t* key, const int32_t* id, int32_t n, int32_t k, int lane, uint64_t& thr_k,
                                              int32_t& thr_u) {
    uint64_t prev_k = 0ull;
    int32_t prev_u = -1;
    for (int32_t round = 0; round < k; ++round) {
        uint64_t best_k = ~0ull;
        int32_t best_u = 0x7fffffff;
        for (int32_t j = lane; j < n; j += kWave) {
            const uint64_t kj = key[j];
            const int32_t uj = id[j];
            if (pair_less(prev_k, prev_u, kj, uj) && pair_less(kj, uj, best_k, best_u)) {
                best_k = kj;
                best_u = uj;
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const uint64_t ok = __shfl_xor(best_k, d, kWave);
            const int32_t ou = __shfl_xor(best_u, d, kWave);
            if (pair_less(ok, ou, best_k, best_u)) {
                best_k = ok;
                best_u = ou;
            }
        }
        prev_k = best_k;
        prev_u = best_u;
    }
    thr_k = prev_k;
    thr_u = prev_u;
}

// Drops the pairs above (thr_k, thr_u) from the list, in place and in order; returns how many are left.
__device__ __forceinline__ int32_t wave_list_keep_below(uint64_t* key, int32_t* id, int32_t n, uint64_t thr_k, int32_t thr_u, int lane) {
    const uint64_t lanes_below = (1ull << lane) - 1ull;
    int32_t out = 0;
    for (int32_t base = 0; base < n; base += kWave) {   // front to back: targets lie at or before the chunk being read
        const int32_t j = base + lane;
        const uint64_t kj = j < n ? key[j] : 0ull;
        const int32_t uj = j < n ? id[j] : 0;
        const bool keep = j < n && !pair_less(thr_k, thr_u, kj, uj);
        const uint64_t km = __ballot(keep);
        wave_lds_sync();   // the chunk has been read by every lane
        if (keep) {
            const int32_t pos = out + __popcll(km & lanes_below);
            key[pos] = kj;
            id[pos] = uj;
        }
        out += __popcll(km);
        wave_lds_sync();
    }
    return out;
}

}  // namespace gnnhot
