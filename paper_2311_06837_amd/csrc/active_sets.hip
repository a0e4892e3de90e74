// Per-layer active vertex sets: level-synchronous frontier expansion from the targets
// (paper section 6, figure 7c: step 1 extracts the multi-hop dependency from the inner
// vertices, step 4 generates the per-layer mask).
//
// Data layout.  In the workspace: bitmaps of n bits, `visited` (everything reached by the
// levels before the one being expanded, read-only while it expands; in a small graph, whose emit
// blocks read each other's words, two copies that the levels use in turn) and `frontier` (the ring
// the last level found), and `seen`, ONE BYTE per vertex (`visited` plus what the level has found
// so far).  `seen` is bytes because every lane that finds a vertex marks it: a byte takes
// a plain store of 1 - whoever comes first, the byte ends up the same - where a bit needs an atomic OR, and a ring of a few million new vertices packs those atomics onto a few thousand
// cache lines (measured: 0.60 ms of atomics for 24 M edges that discover 2.2 M vertices).
// The byte accesses are ordinary loads and stores on purpose: a stale 0 from the vector cache
// only means one more store of the same 1 (relaxed atomic loads, which bypass that cache, were
// measured 15 to 50 % slower per construction); kernel boundaries order the levels.
// A level is: expand -> count / emit, a compaction of seen & ~visited that lists the
// new ring in ascending id order without any sort, so the output does not depend on which
// wave found a vertex first; emit also writes the next visited.  Ring sizes stay on
// the device (hop_offsets); every kernel has a fixed grid and reads its bounds from there, so
// the whole construction is enqueued without a host round trip.
// With few vertices or many rings a construction is as long as its launches (about 5 us each,
// the gap included), so a level is four of them: expansion in whichever direction, its long
// rows, count, emit (which adds up the counts before its own and, for the direction switch, the
// row lengths of the ring it writes) - three where emit counts for itself (kAsSelfCount), five
// above 16M vertices, where the counts are scanned by a launch of their own (kAsSumCounts).  With a
// launch per direction, per scan and per plan it was eight: eight rings of a 1M-vertex graph
// 342 -> 269 us, two of a 10 000-vertex graph 119 -> 95 us, three of a 5M-vertex graph 688 -> 650 us
// (with the call's own host work and its copy of the ring sizes).
//
// A level expands in one of two directions; the sets are the same either way.
//   push  (from the frontier)  EDGE-parallel: a wavefront takes up to 64 frontier vertices, reads
//         their row bounds in one sweep, and then walks the concatenation of their rows 256
//         edges at a time (each lane finds the row of its edge by a binary search over the 64
//         prefix sums in LDS), so rows of 5 and rows of 500 entries keep all lanes busy alike
//         and every lane has four independent index loads and four bitmap probes in flight.
//         One probe of `seen` per edge; the byte is set if still clear.
//   pull  (from the unreached vertices; needs the transposed graph)  sixteen lanes per
//         unreached vertex scan its row of the transposed graph - the vertices that would
//         reach it - and stop at the first one that is in `frontier`.  Once the frontier is
//         most of the graph, nearly every edge of a push level points at a vertex that is
//         already in the set; the pull level only touches the few vertices still outside.
// The direction is chosen on the device, per level, from exact integer sums (made by emit):
// pull when the frontier's edges outnumber what a pull can touch at most, the transposed
// rows of the unreached vertices plus sixteen lanes for each of them.
//
// Bound: a push level reads each edge of the frontier once (4 B, streaming) and makes one
// 1-byte probe per edge into n bytes that stay in L2: the probes, not the bytes, are what
// limits it (the L2s serve a fixed number of requests per clock).
#include "common.h"
#include "hashkey.h"
#include "scan.h"
#include <type_traits>

namespace gnnhot {

constexpr int kAsWordsPerBlock = 256;   // one bitmap word per thread: 8192 vertices per block
constexpr int kAsHubDegree = 2048;      // longer rows are queued and expanded by a whole workgroup each

// A graph of up to this many blocks: emit counts the blocks before its own itself instead of reading what a count launch
// left (a block reads 9 KB per block before it: cheaper than the launch up to about 16).
constexpr int64_t kAsSelfCount = 16;
// Above this many blocks a launch turns the counts into positions: blocks that add up all counts before their own read
// half of nb^2 of them.  Three rings of a graph of 1e9 vertices took 10.1 ms that way and take 4.0 (100M: 437 -> 349 us; 10M,
// below the limit: 82, with the launch 96).
constexpr int64_t kAsSumCounts = 2048;

// Sums that every workgroup of emit adds to, dealt out to cache lines of their own above kAsOneSlot workgroups: on one address
// 12 000 of them (100M vertices) wait 0.2 ms a level for each other.  (Adding the slots up takes 4 us a level: with few
// workgroups there is one place.)  Three rings of 100M vertices with the transposed graph: 1290 -> 412 us.
constexpr int kAsSlots = 32;
constexpr int64_t kAsOneSlot = 256;
struct AsSlot {
    unsigned long long v;
    unsigned long long pad[15];
};

struct AsLevel {
    AsSlot frontier_edges[kAsSlots];     // entries of the ring's rows
    int32_t n_hubs;                      // rows queued while the ring is expanded
    int32_t pad[31];
};

struct AsCtrl {
    AsSlot reached_edges_t[kAsSlots];    // entries of the transposed rows of everything reached so far
    AsLevel level[1];                    // one per ring (L + 1 of them)
};

inline size_t as_ctrl_words(int32_t L) { return (sizeof(AsCtrl) + (size_t)L * sizeof(AsLevel)) / sizeof(int64_t); }

// The slots' sum; all lanes of the wavefront call it and get it.
__device__ __forceinline__ int64_t as_slot_sum(const AsSlot* __restrict__ slots, bool many) {
    static_assert(kAsSlots == 32, "half a wavefront");
    if (!many) return (int64_t)slots[0].v;
    unsigned long long x = lane_id() < kAsSlots ? slots[lane_id()].v : 0ull;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, kWave);
    return (int64_t)x;
}

// True when ring `ring` is expanded in the pull direction.  A pull touches at most the transposed rows of the unreached
// vertices, sixteen lanes at a time.
__device__ __forceinline__ bool as_pull_level(const AsCtrl* ctrl, const int64_t* __restrict__ hop_offsets, int32_t ring, int64_t n, int64_t nnz_t,
                                              bool many) {
    const int64_t unreached = n - hop_offsets[ring + 1];
    const int64_t unreached_edges = nnz_t - as_slot_sum(ctrl->reached_edges_t, many);
    return __builtin_amdgcn_readfirstlane((int)(as_slot_sum(ctrl->level[ring].frontier_edges, many) > unreached_edges + 16 * unreached)) != 0;
}

// Bit b of the result = byte b of the 32 bytes at p (each 0 or 1); p is 32-byte aligned.
__device__ __forceinline__ uint32_t as_mask_of_bytes(const uint8_t* __restrict__ p) {
    const uint4 a = *(const uint4*)p, b = *(const uint4*)(p + 16);
    const uint32_t x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t m = 0u;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        m |= ((x[k] & 1u) | ((x[k] >> 7) & 2u) | ((x[k] >> 14) & 4u) | ((x[k] >> 21) & 8u)) << (4 * k);
    return m;
}

__global__ __launch_bounds__(256) void as_init_kernel(int32_t* __restrict__ dist, int32_t n, uint32_t* __restrict__ visited,
                                                      uint8_t* __restrict__ seen, int64_t nw, int64_t* __restrict__ ctrl, int32_t ctrl_words,
                                                      int64_t* __restrict__ hop_offsets, int32_t L) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = tid; v < n; v += stride) dist[v] = -1;
    for (int64_t w = tid; w < nw; w += stride) {
        visited[w] = 0u;
        ((uint4*)seen)[2 * w] = make_uint4(0u, 0u, 0u, 0u);   // 32 bytes per bitmap word, the tail of the last word included
        ((uint4*)seen)[2 * w + 1] = make_uint4(0u, 0u, 0u, 0u);
    }
    for (int64_t i = tid; i < ctrl_words; i += stride) ctrl[i] = 0;
    for (int64_t i = tid; i <= L + 1; i += stride) hop_offsets[i] = 0;
}

__global__ __launch_bounds__(256) void as_seed_kernel(const int32_t* __restrict__ targets, int32_t n_targets, int32_t n,
                                                      uint8_t* __restrict__ seen) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_targets; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t v = targets[i];
        if (v >= 0 && v < n) seen[v] = 1;
    }
}

constexpr unsigned kAsPushBlocks = 2048;   // workgroups of a push level: what the chip holds at once
constexpr int kAsU = 8;   // edges per lane and step: their index loads, then their probes, are issued together

// Push level.  One wavefront per batch of up to 64 entries of the frontier list (grid-stride), edge-parallel inside
// (see the head of the file).  A step of a wavefront is a chain of dependent loads (row bounds, ids, probes: about
// 3 us), so what a level costs is the number of steps of its busiest wavefront: the batch is made as small as it can be
// while every batch still finds a wavefront of its own (a power of two, at least 1) - 29 000 frontier vertices of
// 490 entries each are 122 steps per wavefront in batches of 64 and 4 in batches of 4 (measured on the 8-level
// workload, 62 500 frontier vertices of 27 entries: 0.28 -> 0.08 ms for the level).
__device__ __forceinline__ void as_push(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                        const int32_t* __restrict__ ring_ids, const int64_t* __restrict__ hop_offsets, int32_t ring,
                                        uint8_t* __restrict__ seen, int32_t* __restrict__ hubq, AsCtrl* ctrl) {
    __shared__ int32_t s_start[4][kWave];
    __shared__ int32_t s_excl[4][kWave + 1];
    const int64_t begin = hop_offsets[ring], end = hop_offsets[ring + 1];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    int32_t* st = s_start[wave];
    int32_t* ex = s_excl[wave];
    const int64_t wave_g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)(gridDim.x < kAsPushBlocks ? gridDim.x : kAsPushBlocks) * blockDim.x) >> 6;
    if (wave_g >= n_waves) return;   // (a pull may use a larger grid)
    int batch = kWave;
    while (batch > 1 && (int64_t)(batch >> 1) * n_waves >= end - begin) batch >>= 1;
    for (int64_t b = begin + wave_g * batch; b < end; b += n_waves * batch) {   // uniform over the wavefront
        const int64_t i = b + lane;
        int32_t s = 0, len = 0;
        if (lane < batch && i < end) {
            const int32_t v = ring_ids[i];
            s = row_ptr[v];
            len = row_ptr[v + 1] - s;
            if (len > kAsHubDegree) {   // a whole workgroup of the next launch takes this row
                hubq[atomicAdd(&ctrl->level[ring].n_hubs, 1)] = v;
                len = 0;
            }
        }
        const int incl = wave_inclusive_scan(len);
        const int total = __shfl(incl, kWave - 1, kWave);
        wave_lds_sync();   // the previous batch has been read
        st[lane] = s;
        ex[lane] = incl - len;
        if (lane == kWave - 1) ex[kWave] = total;
        wave_lds_sync();
        for (int t0 = 0; t0 < total; t0 += kWave * kAsU) {
            int32_t u[kAsU];
            bool ok[kAsU];
#pragma unroll
            for (int j = 0; j < kAsU; ++j) {
                const int t = t0 + j * kWave + lane;
                ok[j] = t < total;
                int lo = 0, hi = kWave;   // ex[lo] <= t < ex[hi]: the row that holds edge t (empty rows are stepped over)
                if (ok[j]) {
#pragma unroll
                    for (int k = 0; k < 6; ++k) {
                        const int mid = (lo + hi) >> 1;
                        if (ex[mid] <= t) lo = mid;
                        else hi = mid;
                    }
                }
                u[j] = ok[j] ? col_idx[st[lo] + (t - ex[lo])] : 0;
            }
            uint8_t w[kAsU];
#pragma unroll
            for (int j = 0; j < kAsU; ++j) w[j] = seen[u[j]];   // u = 0 where the lane has no edge: a valid byte
#pragma unroll
            for (int j = 0; j < kAsU; ++j)
                if (ok[j] && !w[j]) seen[u[j]] = 1;
        }
    }
}

// Hub rows of a push level: the queued rows are cut into as many equal pieces as the grid has workgroups per row, a
// workgroup per piece (grid-stride), threads across the piece, kAsU entries per thread and step.
__device__ __forceinline__ void as_push_hubs(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                             uint8_t* __restrict__ seen, const int32_t* __restrict__ hubq, int32_t n_hubs) {
    const int32_t parts = (int32_t)gridDim.x / n_hubs > 1 ? (int32_t)gridDim.x / n_hubs : 1;
    for (int64_t job = blockIdx.x; job < (int64_t)n_hubs * parts; job += gridDim.x) {   // uniform over the workgroup
        const int32_t v = hubq[job / parts];
        const int32_t part = (int32_t)(job % parts);
        const int64_t s0 = row_ptr[v], len = row_ptr[v + 1] - s0;
        const int32_t s = (int32_t)(s0 + len * part / parts), e = (int32_t)(s0 + len * (part + 1) / parts);
        for (uint32_t base = s + threadIdx.x; base < (uint32_t)e; base += 256 * kAsU) {   // (past the end, a position may not fit an int32_t)
            int32_t u[kAsU];
            uint8_t w[kAsU];
#pragma unroll
            for (int j = 0; j < kAsU; ++j) u[j] = base + j * 256 < (uint32_t)e ? col_idx[base + j * 256] : 0;
#pragma unroll
            for (int j = 0; j < kAsU; ++j) w[j] = seen[u[j]];
#pragma unroll
            for (int j = 0; j < kAsU; ++j)
                if (base + j * 256 < (uint32_t)e && !w[j]) seen[u[j]] = 1;
        }
    }
}

// Pull level.  A wavefront per bitmap word (grid-stride), sixteen lanes per vertex: for each vertex of the word that is
// not in the set yet, scan its transposed row 64 entries at a time and stop at the first entry that is in the frontier.  A lane group
// is the only writer of its vertices' bytes in this kernel.  Rows longer than kAsHubDegree go to the queue.
__device__ __forceinline__ void as_pull(const int32_t* __restrict__ row_ptr_t, const int32_t* __restrict__ col_idx_t, int32_t n, int64_t nw,
                                        const uint32_t* __restrict__ visited, uint8_t* __restrict__ seen,
                                        const uint32_t* __restrict__ frontier, int32_t ring, int32_t* __restrict__ hubq, AsCtrl* ctrl) {
    const int lane = lane_id(), sub = lane / 16, sl = lane % 16;
    const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w < nw; w += waves) {   // uniform over the wave
        uint32_t open = ~visited[w];
        if (w == nw - 1 && (n & 31)) open &= (1u << (n & 31)) - 1u;
        // the wavefront's four lane groups share the word: group k takes its k-th, (k+4)-th, ... unreached vertex (a
        // vertex is a chain of dependent loads; four chains run side by side)
        uint32_t mine = 0u;
        for (int k = 0; open; ++k) {   // uniform over the wave
            const uint32_t lowest = open & (0u - open);
            open ^= lowest;
            if ((k & 3) == sub) mine |= lowest;
        }
        while (mine) {   // uniform over the lane group
            const int b = __ffs(mine) - 1;
            mine &= mine - 1u;
            const int32_t v = (int32_t)(w * 32 + b);
            const int32_t s = row_ptr_t[v], e = row_ptr_t[v + 1];
            if (e - s > kAsHubDegree) {
                if (sl == 0) hubq[atomicAdd(&ctrl->level[ring].n_hubs, 1)] = v;
                continue;
            }
            bool found = false;
            for (uint32_t p = s; p < (uint32_t)e && !found; p += 64) {
                int32_t u[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) u[j] = p + j * 16 + sl < (uint32_t)e ? col_idx_t[p + j * 16 + sl] : -1;
                bool hit = false;
#pragma unroll
                for (int j = 0; j < 4; ++j) hit |= u[j] >= 0 && in_set(frontier, u[j]);
                found = ((__ballot(hit) >> (sub * 16)) & 0xffffull) != 0ull;
            }
            if (found && sl == 0) seen[v] = 1;
        }
    }
}

// Long rows of a pull level: one workgroup per queued vertex, 256 entries per step, until one is in the frontier.
__device__ __forceinline__ void as_pull_hubs(const int32_t* __restrict__ row_ptr_t, const int32_t* __restrict__ col_idx_t,
                                             uint8_t* __restrict__ seen, const uint32_t* __restrict__ frontier,
                                             const int32_t* __restrict__ hubq, int32_t n_hubs) {
    for (int32_t h = blockIdx.x; h < n_hubs; h += gridDim.x) {   // uniform over the workgroup
        const int32_t v = hubq[h];
        const int32_t s = row_ptr_t[v], e = row_ptr_t[v + 1];
        for (uint32_t base = s; base < (uint32_t)e; base += 256) {
            const uint32_t p = base + threadIdx.x;
            const int hit = p < (uint32_t)e && in_set(frontier, col_idx_t[p]);
            if (__syncthreads_or(hit)) {
                if (threadIdx.x == 0) seen[v] = 1;
                break;
            }
        }
    }
}

struct AsArgs {
    const int32_t *row_ptr, *col_idx;       // the graph
    const int32_t *row_ptr_t, *col_idx_t;   // its transpose, or NULL: every level pushes
    int32_t n;
    int64_t nw, nnz_t;
    bool many;                              // workgroups of emit: the sums are in kAsSlots places
    const int32_t* ring_ids;
    const int64_t* hop_offsets;
    const uint32_t* visited;
    uint8_t* seen;
    const uint32_t* frontier;
    int32_t* hubq;
    AsCtrl* ctrl;
};

// Expansion of ring `ring`, in the direction that costs less.
__global__ __launch_bounds__(256) void as_expand_kernel(AsArgs a, int32_t ring) {
    if (a.row_ptr_t != nullptr && as_pull_level(a.ctrl, a.hop_offsets, ring, a.n, a.nnz_t, a.many))   // uniform over the grid
        as_pull(a.row_ptr_t, a.col_idx_t, a.n, a.nw, a.visited, a.seen, a.frontier, ring, a.hubq, a.ctrl);
    else
        as_push(a.row_ptr, a.col_idx, a.ring_ids, a.hop_offsets, ring, a.seen, a.hubq, a.ctrl);
}

// The rows that the expansion queued.
__global__ __launch_bounds__(256) void as_expand_hubs_kernel(AsArgs a, int32_t ring) {
    const int32_t n_hubs = a.ctrl->level[ring].n_hubs;
    if (n_hubs <= 0) return;
    if (a.row_ptr_t != nullptr && as_pull_level(a.ctrl, a.hop_offsets, ring, a.n, a.nnz_t, a.many))
        as_pull_hubs(a.row_ptr_t, a.col_idx_t, a.seen, a.frontier, a.hubq, n_hubs);
    else
        as_push_hubs(a.row_ptr, a.col_idx, a.seen, a.hubq, n_hubs);
}

__global__ __launch_bounds__(kAsWordsPerBlock) void as_count_kernel(const uint8_t* __restrict__ seen,
                                                                    const uint32_t* __restrict__ visited, int64_t nw,
                                                                    int32_t* __restrict__ blk_cnt) {
    __shared__ int s_part[kAsWordsPerBlock / kWave];
    const int64_t w = (int64_t)blockIdx.x * kAsWordsPerBlock + threadIdx.x;
    int c = 0;
    if (w < nw) c = __popc(as_mask_of_bytes(seen + 32 * w) & ~visited[w]);
    int total;
    block_exclusive_scan<kAsWordsPerBlock>(c, s_part, &total);
    if (threadIdx.x == 0) blk_cnt[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void as_scan_kernel(int32_t* __restrict__ blk_cnt, int64_t nb) {
    __shared__ int s_part[1024 / kWave];
    single_block_exclusive_scan(blk_cnt, nb, s_part);
}

// Sums over the workgroup; every thread gets them.  Two barriers.
template <int N>
__device__ __forceinline__ void as_block_sum(unsigned long long (&x)[N], unsigned long long (*s_sum)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) x[k] += __shfl_xor(x[k], d, kWave);
    if (lane_id() == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) s_sum[threadIdx.x >> 6][k] = x[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = s_sum[0][k] + s_sum[1][k] + s_sum[2][k] + s_sum[3][k];
    __syncthreads();
}

// Lists ring `ring` (seen & ~visited) in ascending id order behind the rings before it and writes the next `visited`.
// Every block adds up the counts of the blocks before it (blk_cnt NULL: counts them; scanned: finds their sum in its place of
// blk_cnt); the last one knows the ring's end.
// With row_ptr_t (a later pull is possible): the ring as a bitmap, and the exact sums the direction switch needs, the
// entries of the ring's rows and of its transposed rows (integer atomics: the totals do not depend on their order).
__global__ __launch_bounds__(kAsWordsPerBlock) void as_emit_kernel(const uint8_t* __restrict__ seen, const uint32_t* visited,
                                                                   uint32_t* visited_next, int64_t nw,
                                                                   const int32_t* __restrict__ blk_cnt, bool scanned, bool many,
                                                                   int64_t* __restrict__ hop_offsets,
                                                                   int32_t ring, int32_t* __restrict__ ring_ids, int32_t* __restrict__ dist,
                                                                   uint32_t* __restrict__ frontier, const int32_t* __restrict__ row_ptr,
                                                                   const int32_t* __restrict__ row_ptr_t, AsCtrl* ctrl) {
    static_assert(kAsWordsPerBlock == 256, "as_block_sum adds four wavefronts");
    __shared__ int s_part[kAsWordsPerBlock / kWave];
    __shared__ unsigned long long s_base[kAsWordsPerBlock / kWave][1], s_edges[kAsWordsPerBlock / kWave][2];
    __shared__ uint32_t s_fresh[kAsWordsPerBlock];
    __shared__ int s_before[kAsWordsPerBlock];
    unsigned long long base[1] = {0ull};
    if (scanned) {   // uniform over the grid
        base[0] = (unsigned long long)blk_cnt[blockIdx.x];
    } else {
        if (blk_cnt != nullptr) {
            for (int64_t b = threadIdx.x; b < blockIdx.x; b += kAsWordsPerBlock) base[0] += (unsigned long long)blk_cnt[b];
        } else {
            for (int64_t w = threadIdx.x; w < (int64_t)blockIdx.x * kAsWordsPerBlock; w += kAsWordsPerBlock)
                base[0] += (unsigned long long)__popc(as_mask_of_bytes(seen + 32 * w) & ~visited[w]);
        }
        as_block_sum(base, s_base);
    }
    const int64_t w = (int64_t)blockIdx.x * kAsWordsPerBlock + threadIdx.x;
    uint32_t fresh = 0u;
    if (w < nw) {
        const uint32_t sn = as_mask_of_bytes(seen + 32 * w), vis = visited[w];
        fresh = sn & ~vis;
        if (fresh || visited_next != visited) visited_next[w] = vis | sn;
        if (row_ptr_t != nullptr) frontier[w] = fresh;   // the ring a pull level looks for
    }
    int total;
    const int before = block_exclusive_scan<kAsWordsPerBlock>(__popc(fresh), s_part, &total);
    const int64_t begin = hop_offsets[ring] + (int64_t)base[0];
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) hop_offsets[ring + 1] = begin + total;
    if (total == 0) return;   // uniform over the workgroup
    unsigned long long edges[2] = {0ull, 0ull};   // of the ring's rows and of its transposed rows
    // vertices v[r] where in[r]: into the list at pos[r], and their rows' lengths; all loads in flight (a lane without a vertex
    // of the ring reads the first row)
    auto take = [&](auto n_const, const bool* in, const int32_t* v, const int64_t* pos) {
        constexpr int N = decltype(n_const)::value;
        bool any = false;
#pragma unroll
        for (int r = 0; r < N; ++r) {
            any |= in[r];
            if (in[r]) {
                ring_ids[pos[r]] = v[r];
                dist[v[r]] = ring;
            }
        }
        if (row_ptr_t == nullptr || __ballot(any) == 0ull) return;   // uniform over the wavefront
        int32_t lo[N], hi[N], lo_t[N], hi_t[N];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const int32_t u = in[r] ? v[r] : 0;
            lo[r] = row_ptr[u];
            hi[r] = row_ptr[u + 1];
            lo_t[r] = row_ptr_t[u];
            hi_t[r] = row_ptr_t[u + 1];
        }
#pragma unroll
        for (int r = 0; r < N; ++r) {
            edges[0] += in[r] ? (unsigned long long)(hi[r] - lo[r]) : 0ull;
            edges[1] += in[r] ? (unsigned long long)(hi_t[r] - lo_t[r]) : 0ull;
        }
    };
    constexpr int kSparse = 4, kBatch = 8;
    bool in[kBatch];
    int32_t v[kBatch];
    int64_t pos[kBatch];
    if (many && !__syncthreads_or(__popc(fresh) > kSparse)) {
        // few vertices in every word: a lane takes those of its own word (looking through all of a block's vertices for them,
        // as below, costs 20 us a level where 100M vertices have rings of a thousandth)
        uint32_t rest = fresh;
        for (int r = 0; r < kSparse && __ballot(rest != 0u) != 0ull; ++r) {   // uniform over the wavefront
            in[0] = rest != 0u;
            v[0] = (int32_t)(w * 32 + (in[0] ? __ffs(rest) - 1 : 0));
            pos[0] = begin + before + r;
            rest &= rest - 1u;
            take(std::integral_constant<int, 1>(), in, v, pos);
        }
    } else {
        // a lane per vertex, not per word (32 vertices after each other, each with its loads, took 17 us whatever the size),
        // eight vertices at a time
        s_fresh[threadIdx.x] = fresh;
        s_before[threadIdx.x] = before;
        __syncthreads();
        const int bit = (int)(threadIdx.x & 31);
        const uint32_t below = (1u << bit) - 1u;
        for (int r0 = 0; r0 < 32; r0 += kBatch) {
#pragma unroll
            for (int r = 0; r < kBatch; ++r) {
                const int k = (r0 + r) * (kAsWordsPerBlock / 32) + (int)(threadIdx.x >> 5);
                const uint32_t word = s_fresh[k];
                in[r] = (word >> bit) & 1u;
                v[r] = (int32_t)(((int64_t)blockIdx.x * kAsWordsPerBlock + k) * 32 + bit);
                pos[r] = begin + s_before[k] + __popc(word & below);
            }
            take(std::integral_constant<int, kBatch>(), in, v, pos);
        }
    }
    if (row_ptr_t != nullptr) {   // uniform over the grid
        as_block_sum(edges, s_edges);
        if (threadIdx.x == 0) {
            atomicAdd(&ctrl->level[ring].frontier_edges[many ? blockIdx.x % kAsSlots : 0].v, edges[0]);
            atomicAdd(&ctrl->reached_edges_t[many ? blockIdx.x % kAsSlots : 0].v, edges[1]);
        }
    }
}

// ---- expansion-aware traversal (paper section 5.3.1) -----------------------------------------------------------
// The same level-synchronous scheme with a thinned expansion: a traversed vertex keeps at most `fanout` of its
// not-yet-selected neighbours, those with the smallest (key, id).  `visited` is read-only while a hop expands, so
// "not yet selected" means "when the hop started" for every row, and the result does not depend on the order in
// which rows are processed.  Keys: the seeded edge hash of the boundary sampler, or (the paper's rule) the negated
// number of connections of the candidate to vertices that were unselected when the hop started.

// conn[u] = number of entries of row u that are not in `visited`; sixteen lanes per row
__global__ __launch_bounds__(256) void eas_connections_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                               int32_t n, const uint32_t* __restrict__ visited,
                                                               int32_t* __restrict__ conn) {
    const int lane = lane_id(), sub = lane / 16, sl = lane % 16;
    const int64_t groups = (int64_t)gridDim.x * (blockDim.x / 16);
    for (int64_t u = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 16; u < n; u += groups) {
        const int32_t s = row_ptr[u], e = row_ptr[u + 1];
        int32_t c = 0;
        for (uint32_t p = s; p < (uint32_t)e; p += 16) {
            const bool open = p + sl < (uint32_t)e && !in_set(visited, col_idx[p + sl]);
            c += __popcll((__ballot(open) >> (sub * 16)) & 0xffffull);
        }
        if (sl == 0) conn[u] = c;
    }
}

__device__ __forceinline__ uint64_t eas_key(int32_t rule, uint64_t seed_hop_mixed, const int32_t* __restrict__ conn, int32_t v, int32_t u) {
    return rule == 1 ? (uint64_t)(0xffffffffu - (uint32_t)conn[u]) : edge_key(seed_hop_mixed, (uint64_t)v, (uint64_t)u);
}

constexpr int kEasShortRow = 64;    // rows up to this length: sixteen lanes each; longer rows: a wavefront each
constexpr int kEasListCap = 1024;   // candidates of one long row that a wavefront keeps in LDS

// Rows of at most kEasShortRow entries: sixteen lanes per frontier vertex, four vertices per wavefront, up to four
// entries of the row per lane.  Entries, candidate flags and keys are read once and stay in registers; a row with
// more than `fanout` candidates finds the fanout-th smallest (key, id) by `fanout` rounds of "smallest pair above the
// previous one" over those registers.  Every lane runs every ballot and shuffle (no lane leaves early).
__global__ __launch_bounds__(256) void eas_expand_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                          const int32_t* __restrict__ ring_ids, const int64_t* __restrict__ hop_offsets,
                                                          int32_t ring, const uint32_t* __restrict__ visited, uint8_t* __restrict__ seen,
                                                          int32_t fanout, int32_t rule, uint64_t seed_hop_mixed,
                                                          const int32_t* __restrict__ conn) {
    constexpr int kPerLane = kEasShortRow / 16;
    const int64_t begin = hop_offsets[ring], end = hop_offsets[ring + 1];
    const int lane = lane_id(), sub = lane / 16, sl = lane % 16;
    const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    if (fanout == 0) return;   // nothing is selected
    for (int64_t base = begin + 4 * (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6); base < end; base += 4 * waves) {  // uniform over the wave
        const int64_t i = base + sub;
        int32_t v = 0, s = 0, e = 0;
        if (i < end) {
            v = ring_ids[i];
            s = row_ptr[v];
            e = row_ptr[v + 1];
            if (e - s > kEasShortRow) e = s;   // eas_expand_long_kernel takes this row
        }
        int32_t u[kPerLane];
        bool cand[kPerLane];
        uint64_t key[kPerLane];
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) u[j] = (uint32_t)s + j * 16 + sl < (uint32_t)e ? col_idx[(uint32_t)s + j * 16 + sl] : -1;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) cand[j] = u[j] >= 0 && !in_set(visited, u[j]);
        int32_t n_cand = 0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            key[j] = cand[j] ? eas_key(rule, seed_hop_mixed, conn, v, u[j]) : ~0ull;
            n_cand += __popcll((__ballot(cand[j]) >> (sub * 16)) & 0xffffull);
        }
        // threshold pair: candidates with (key, id) <= (thr_k, thr_u) are kept
        uint64_t thr_k = ~0ull;
        int32_t thr_u = 0x7fffffff;
        const bool need = n_cand > fanout;   // uniform over the 16-lane group
        if (__ballot(need) != 0ull) {        // uniform over the wavefront
            uint64_t prev_k = 0ull;
            int32_t prev_u = -1;
            for (int32_t round = 0; round < fanout; ++round) {
                uint64_t best_k = ~0ull;
                int32_t best_u = 0x7fffffff;
#pragma unroll
                for (int j = 0; j < kPerLane; ++j) {
                    if (cand[j] && pair_less(prev_k, prev_u, key[j], u[j]) && pair_less(key[j], u[j], best_k, best_u)) {
                        best_k = key[j];
                        best_u = u[j];
                    }
                }
#pragma unroll
                for (int d = 8; d >= 1; d >>= 1) {
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
            if (need) {
                thr_k = prev_k;
                thr_u = prev_u;
            }
        }
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            if (cand[j] && !pair_less(thr_k, thr_u, key[j], u[j]) && !seen[u[j]]) seen[u[j]] = 1;
        }
    }
}

// Rows longer than kEasShortRow: one wavefront per frontier vertex.  The row is read ONCE; its candidates (neighbours
// not selected when the hop started) go to a list in LDS with their keys (one key computation and, for the
// best-connected-first rule, one read of conn[] per candidate).  When the list is full it is cut down to its `fanout`
// smallest (key, id) pairs, and from then on only candidates below the largest of those are listed: a pair that is
// not among the fanout smallest of what has been read so far cannot be among the fanout smallest of the row.  At the
// end the fanout smallest pairs of the list are the row's.  (A fanout too large for this - within 64 of the list's
// capacity - takes the rounds over the row itself, re-reading it once per kept neighbour.)
__global__ __launch_bounds__(256) void eas_expand_long_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                               const int32_t* __restrict__ ring_ids,
                                                               const int64_t* __restrict__ hop_offsets, int32_t ring,
                                                               const uint32_t* __restrict__ visited, uint8_t* __restrict__ seen,
                                                               int32_t fanout, int32_t rule, uint64_t seed_hop_mixed,
                                                               const int32_t* __restrict__ conn) {
    __shared__ uint64_t s_key[4][kEasListCap];
    __shared__ int32_t s_id[4][kEasListCap];
    const int64_t begin = hop_offsets[ring], end = hop_offsets[ring + 1];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    uint64_t* key = s_key[wave];
    int32_t* id = s_id[wave];
    const uint64_t lanes_below = (1ull << lane) - 1ull;
    const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    if (fanout == 0) return;   // nothing is selected
    const bool streaming = fanout <= kEasListCap - kWave;   // the list can always be cut down far enough to take a chunk
    for (int64_t i = begin + (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6); i < end; i += waves) {   // uniform over the wave
        const int32_t v = ring_ids[i];
        const int32_t s = row_ptr[v], e = row_ptr[v + 1];
        if (e - s <= kEasShortRow) continue;
        uint64_t thr_k = ~0ull;   // pairs above (thr_k, thr_u) are out
        int32_t thr_u = 0x7fffffff;
        int32_t n_list = 0;       // pairs in the list
        int32_t n_cand = 0;       // candidates of the row (only needed when not streaming)
        for (uint32_t p = s; p < (uint32_t)e; p += kWave) {
            const uint32_t q = p + lane;
            const int32_t u = q < (uint32_t)e ? col_idx[q] : 0;
            const bool cand = q < (uint32_t)e && !in_set(visited, u);
            const uint64_t k = cand ? eas_key(rule, seed_hop_mixed, conn, v, u) : 0ull;
            bool take = cand && !pair_less(thr_k, thr_u, k, u);
            uint64_t mask = __ballot(take);
            n_cand += __popcll(__ballot(cand));
            if (streaming && n_list + __popcll(mask) > kEasListCap) {   // uniform: cut the list down to its fanout smallest
                wave_lds_sync();
                wave_list_kth(key, id, n_list, fanout, lane, thr_k, thr_u);
                n_list = wave_list_keep_below(key, id, n_list, thr_k, thr_u, lane);
                take = cand && !pair_less(thr_k, thr_u, k, u);
                mask = __ballot(take);
            }
            const int32_t pos = n_list + __popcll(mask & lanes_below);
            if (take && pos < kEasListCap) {
                key[pos] = k;
                id[pos] = u;
            }
            n_list += __popcll(mask);
        }
        wave_lds_sync();
        if (streaming || n_list <= kEasListCap) {
            if (n_list > fanout) wave_list_kth(key, id, n_list, fanout, lane, thr_k, thr_u);
            for (int32_t j = lane; j < n_list; j += kWave) {
                const int32_t u = id[j];
                if (!pair_less(thr_k, thr_u, key[j], u) && !seen[u]) seen[u] = 1;
            }
        } else {
            // more candidates than the list holds and a fanout too large to cut it down: rounds over the row itself
            if (n_cand > fanout) {
                uint64_t prev_k = 0ull;
                int32_t prev_u = -1;
                for (int32_t round = 0; round < fanout; ++round) {
                    uint64_t best_k = ~0ull;
                    int32_t best_u = 0x7fffffff;
                    for (uint32_t p = (uint32_t)s + lane; p < (uint32_t)e; p += kWave) {
                        const int32_t u = col_idx[p];
                        if (in_set(visited, u)) continue;
                        const uint64_t k = eas_key(rule, seed_hop_mixed, conn, v, u);
                        if (pair_less(prev_k, prev_u, k, u) && pair_less(k, u, best_k, best_u)) {
                            best_k = k;
                            best_u = u;
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
            for (uint32_t p = (uint32_t)s + lane; p < (uint32_t)e; p += kWave) {
                const int32_t u = col_idx[p];
                if (in_set(visited, u)) continue;
                if (!pair_less(thr_k, thr_u, eas_key(rule, seed_hop_mixed, conn, v, u), u) && !seen[u]) seen[u] = 1;
            }
        }
        wave_lds_sync();   // the lists are read before the next row overwrites them
    }
}

// ---- small graphs: all levels in one launch, by one workgroup -------------------------------------------------------
// A construction of a small graph is as long as its launches, so here one workgroup keeps the bitmaps in LDS (a word a thread)
// and walks the frontier's rows edge-parallel, 8192 edges a step; the row of an edge is a rank among the bits of rows'
// beginnings (a search over the rows' prefix sums is ten dependent LDS reads an edge: 65 us of kernel where this takes 41).
// One compute unit walks what it takes the others to hide, so entries and vertices count against it, levels for it.  The whole call, and
// the GPU's share (us, a launch per part of a level with the transposed graph / this one):
//   two levels: 2000 vertices of degree 5 71 / 32, 34 / 13; 10 000 of 10 78 / 55, 41 / 36; 15 000 of 8 80 / 63, 43 / 44; 30 000 of 2 81 / 59, 46 / 39,
//   of 4 83 / 74, 46 / 54; three: 20 000 of 5 94 / 75, 56 / 56; 30 000 of 4 97 / 95, 60 / 75; 32 000 around one hub, 96 000 entries, 83 / 102, 42 / 82
//   eight: 12 000 of 10 142 / 75, 100 / 55; 32 000 of 4 151 / 118, 112 / 99
// With the transposed graph a level behind which few vertices are left starts from those (10 000 of 10, two levels 61.5 -> 51.7; 15 000 of 8
// 69.8 -> 58.4; 5000 of 20, three 64.4 -> 52.2), and nothing is looked for once all are reached.  Theirs are not always the fewer entries:
// as_pull_pays.
static bool as_takes_small(int32_t n, int64_t nnz, int32_t L) { return nnz + 3 * (int64_t)n <= 168000 || L >= 5; }
constexpr int32_t kAsSmallRows = 32 * 1024;
constexpr int64_t kAsSmallEntries = (int64_t)1 << 17;

// Whether a level of a small graph starts from the `left` unreached vertices, which have `edges` transposed entries: a vertex costs as
// much as four entries.  The ring's `count` vertices stand for their share of the entries of all `total` reached ones.
// us, from the ring / from the last vertices: 3900 vertices with all of 101 000 entries behind 8100 17.1 / 32.6, 1000 of 100 behind 11 000 of
// one 27.0 / 31.9, 4000 of 20 behind 20 000 38.3 / 41.8; but 3000 of 26 behind 25 000 43.3 / 41.7, 2000 of 40 behind 18 000 of one 38.7 / 31.7.
// The question costs 2.5 where the answer is no: it is asked once their rows' bounds are there.
__device__ __forceinline__ bool as_pull_pays(int32_t edges, int32_t left, int32_t count, int32_t total, int32_t nnz) {
    return (float)edges + 4.f * (float)left <= (float)(nnz - edges) * (float)count / (float)total + 4.f * (float)count;
}

template <bool BOTH>     // with the transposed graph
__global__ __launch_bounds__(1024) void as_small_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                        const int32_t* __restrict__ row_ptr_t, const int32_t* __restrict__ col_idx_t, int32_t n,
                                                        int32_t nnz, const int32_t* __restrict__ targets, int32_t n_targets, int32_t L,
                                                        int32_t* __restrict__ dist, int32_t* ring_ids, int64_t* __restrict__ hop_offsets) {
    constexpr int kRows = 4096, kPer = kRows / 1024, kWords = (int)(kAsSmallEntries / 32), kU = 8, kRowBit = 18, kRow = 1 << kRowBit;
    static_assert(kAsSmallEntries < kRow && (int64_t)kRows << kRowBit <= INT32_MAX, "edges and rows share an int");
    __shared__ uint32_t s_seen[1024], s_new[1024];
    __shared__ int32_t s_at[1024];
    __shared__ int32_t s_first[kRows];        // of the rows with entries: position of the first, less the edges before it
    __shared__ uint32_t s_begin[kWords];      // bit: the edge begins a row
    __shared__ uint16_t s_rank[kWords];       // rows that begin before the word's edges
    __shared__ uint16_t s_left[BOTH ? kRows : 1];        // unreached vertices, then those of them with entries
    __shared__ int s_part[16];
    const int tid = (int)threadIdx.x;
    s_seen[tid] = 0u;
    for (int32_t v = tid; v < n; v += 1024) dist[v] = -1;
    if (tid == 0) hop_offsets[0] = 0;
    __syncthreads();
    for (int32_t i = tid; i < n_targets; i += 1024) {
        const int32_t v = targets[i];
        if (v >= 0 && v < n) atomicOr(&s_seen[v >> 5], 1u << (v & 31));
    }
    __syncthreads();
    uint32_t visited = 0u;      // of the thread's 32 vertices
    int32_t total = 0;
    for (int32_t ring = 0;; ++ring) {
        const uint32_t found = s_seen[tid] & ~visited;
        visited |= found;
        int count;
        const int before = block_exclusive_scan<1024>(__popc(found), s_part, &count);
        const int32_t begin = total;
        total += count;
        s_new[tid] = found;
        s_at[tid] = begin + before;
        if (tid == 0) hop_offsets[ring + 1] = total;
        __syncthreads();
        for (int32_t v = tid; v < n; v += 1024) {
            const uint32_t w = s_new[v >> 5], bit = 1u << (v & 31);
            if ((w & bit) == 0u) continue;
            ring_ids[s_at[v >> 5] + __popc(w & (bit - 1u))] = v;
            dist[v] = ring;
        }
        if (ring == L) break;
        if (count == 0 || total == n) {      // nothing more is reached
            for (int32_t r = ring + 1 + tid; r <= L; r += 1024) hop_offsets[r + 1] = total;
            break;
        }
        // From the unreached vertices instead, where few are left: a transposed row with an entry in the ring is reached.
        const int32_t left = n - total;
        const bool pull = BOTH && left <= kRows && 2 * left < count;      // uniform
        if (pull) {
            uint32_t rest = ~visited & (tid * 32 + 32 <= n ? ~0u : tid * 32 < n ? (1u << (n & 31)) - 1u : 0u);
            int place, all;
            place = block_exclusive_scan<1024>(__popc(rest), s_part, &all);
            for (; rest; rest &= rest - 1u) s_left[place++] = (uint16_t)(tid * 32 + __ffs(rest) - 1);
        }
        __syncthreads();       // the ring's ids are there
        auto expand = [&](auto from_left, const int32_t* __restrict__ rows, const int32_t* __restrict__ cols, int32_t from, int32_t end) -> bool {
            constexpr bool kLeft = decltype(from_left)::value;
            for (int32_t c0 = from; c0 < end; c0 += kRows) {
                int32_t s[kPer], len[kPer], v[kPer], sum = 0;
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const int32_t i = c0 + tid * kPer + k < end ? c0 + tid * kPer + k : from;
                    v[k] = kLeft ? (int32_t)s_left[i] : ring_ids[i];
                }
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    s[k] = rows[v[k]];
                    len[k] = rows[v[k] + 1] - s[k];
                }
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    if (c0 + tid * kPer + k >= end) len[k] = 0;
                    sum += len[k] | (len[k] > 0 ? kRow : 0);      // edges (2^17 at most) and rows with some (4096: 2^30), in one sum
                }
                int all;
                int at = block_exclusive_scan<1024>(sum, s_part, &all);
                const int edges = all & (kRow - 1), words = (edges + 31) / 32;
                if (kLeft && !as_pull_pays(edges, left, count, total, nnz)) return false;      // uniform (one chunk: nothing has been changed)
                for (int w = tid; w < words; w += 1024) s_begin[w] = 0u;
                __syncthreads();
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    if (len[k] == 0) continue;
                    const int off = at & (kRow - 1);
                    s_first[at >> kRowBit] = s[k] - off;
                    if (kLeft) s_left[at >> kRowBit] = (uint16_t)v[k];      // (one chunk: all have been read)
                    atomicOr(&s_begin[off >> 5], 1u << (off & 31));
                    at += len[k] | kRow;
                }
                __syncthreads();
                const int each = (words + 1023) / 1024;              // words a thread, one after the other
                int mine = 0, rank_all;
                for (int w = tid * each; w < (tid + 1) * each && w < words; ++w) mine += __popc(s_begin[w]);
                int rank = block_exclusive_scan<1024>(mine, s_part, &rank_all);
                for (int w = tid * each; w < (tid + 1) * each && w < words; ++w) {
                    s_rank[w] = (uint16_t)rank;
                    rank += __popc(s_begin[w]);
                }
                __syncthreads();
                for (int32_t e0 = tid; e0 < edges; e0 += kU * 1024) {
                    int32_t u[kU];
                    int row[kU];
#pragma unroll
                    for (int j = 0; j < kU; ++j) {
                        const int32_t e = e0 + j * 1024 < edges ? e0 + j * 1024 : edges - 1;
                        row[j] = s_rank[e >> 5] + __popc(s_begin[e >> 5] & (~0u >> (31 - (e & 31)))) - 1;
                        u[j] = cols[s_first[row[j]] + e];
                    }
#pragma unroll
                    for (int j = 0; j < kU; ++j) {
                        if (kLeft) {
                            if ((s_new[u[j] >> 5] >> (u[j] & 31) & 1u) == 0u) continue;
                            u[j] = s_left[row[j]];
                        }
                        const uint32_t bit = 1u << (u[j] & 31);
                        if ((s_seen[u[j] >> 5] & bit) == 0u) atomicOr(&s_seen[u[j] >> 5], bit);
                    }
                }
                __syncthreads();
            }
            return true;
        };
        if (!(BOTH && pull && expand(std::true_type{}, row_ptr_t, col_idx_t, 0, left))) expand(std::false_type{}, row_ptr, col_idx, begin, total);
    }
}

// count (unless the blocks are few), scan (if they are many) and emit
static int32_t as_emit(const uint8_t* seen, const uint32_t* visited, uint32_t* visited_next, int64_t nw, int64_t nb, int32_t* blk_cnt,
                       int64_t* hop_offsets, int32_t ring, int32_t* ring_ids, int32_t* dist, uint32_t* frontier, const int32_t* row_ptr,
                       const int32_t* row_ptr_t, AsCtrl* ctrl, hipStream_t stream) {
    if (nb > kAsSelfCount) {
        as_count_kernel<<<(int)nb, kAsWordsPerBlock, 0, stream>>>(seen, visited, nw, blk_cnt);
        GNN_LAUNCH_CHECK("as_count_kernel");
    }
    if (nb > kAsSumCounts) {
        as_scan_kernel<<<1, 1024, 0, stream>>>(blk_cnt, nb);
        GNN_LAUNCH_CHECK("as_scan_kernel");
    }
    as_emit_kernel<<<(int)nb, kAsWordsPerBlock, 0, stream>>>(seen, visited, visited_next, nw, nb > kAsSelfCount ? blk_cnt : nullptr,
                                                             nb > kAsSumCounts, nb > kAsOneSlot, hop_offsets, ring, ring_ids, dist, frontier, row_ptr, row_ptr_t, ctrl);
    GNN_LAUNCH_CHECK("as_emit_kernel");
    return GNN_OK;
}

}  // namespace gnnhot

using namespace gnnhot;

extern "C" int32_t gnn_build_active_sets(const gnn_csr* g, const gnn_csr* gt, const int32_t* targets, int32_t n_targets, int32_t L,
                                         int32_t* dist, int32_t* ring_ids, int64_t* hop_offsets, int64_t* hop_offsets_host,
                                         void* ws, size_t* ws_bytes, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_CHECK(check_csr(g, "g"));
    GNN_REQUIRE(g->n_rows == g->n_cols, GNN_ERR_SHAPE, "active sets need a square graph (%d x %d)", g->n_rows, g->n_cols);
    if (gt != nullptr) {
        GNN_CHECK(check_csr(gt, "gt"));
        GNN_REQUIRE(gt->n_rows == g->n_rows && gt->n_cols == g->n_cols && gt->nnz == g->nnz, GNN_ERR_SHAPE,
                    "gt (%d x %d, %lld entries) is not the transpose of g (%d x %d, %lld entries)", gt->n_rows, gt->n_cols,
                    (long long)gt->nnz, g->n_rows, g->n_cols, (long long)g->nnz);
    }
    GNN_REQUIRE(L >= 1 && L <= 1024, GNN_ERR_INVALID_ARG, "L = %d out of range [1, 1024]", L);
    GNN_REQUIRE(n_targets >= 0, GNN_ERR_INVALID_ARG, "n_targets < 0");
    const int32_t n = g->n_rows;
    const int64_t nw = ((int64_t)n + 31) / 32;
    const int64_t nb = nw > 0 ? (nw + kAsWordsPerBlock - 1) / kAsWordsPerBlock : 1;

    WsCarver carve(ws);
    uint32_t* visited[2];
    visited[0] = carve.take<uint32_t>((size_t)nw + 1);
    visited[1] = nb > kAsSelfCount ? visited[0] : carve.take<uint32_t>((size_t)nw + 1);
    uint8_t* seen = carve.take<uint8_t>((size_t)nw * 32 + 32);
    uint32_t* frontier = carve.take<uint32_t>((size_t)nw + 1);
    int32_t* blk_cnt = carve.take<int32_t>((size_t)nb + 1);
    int32_t* hubq = carve.take<int32_t>((size_t)n + 1);
    const size_t ctrl_words = as_ctrl_words(L);
    int64_t* ctrl = carve.take<int64_t>(ctrl_words);
    bool query;
    GNN_CHECK(ws_protocol(ws, ws_bytes, carve.used, &query));
    if (query) return GNN_OK;

    GNN_REQUIRE(hop_offsets != nullptr, GNN_ERR_INVALID_ARG, "hop_offsets is NULL");
    GNN_REQUIRE(n == 0 || (dist != nullptr && ring_ids != nullptr), GNN_ERR_INVALID_ARG, "dist / ring_ids is NULL");
    GNN_REQUIRE(n_targets == 0 || targets != nullptr, GNN_ERR_INVALID_ARG, "targets is NULL");

    const bool small = n > 0 && n <= kAsSmallRows && g->nnz <= kAsSmallEntries && as_takes_small(n, g->nnz, L);
    if (small) {
        if (gt != nullptr) as_small_kernel<true><<<1, 1024, 0, stream>>>(g->row_ptr, g->col_idx, gt->row_ptr, gt->col_idx, n, (int32_t)g->nnz, targets, n_targets, L, dist, ring_ids, hop_offsets);
        else as_small_kernel<false><<<1, 1024, 0, stream>>>(g->row_ptr, g->col_idx, nullptr, nullptr, n, (int32_t)g->nnz, targets, n_targets, L, dist, ring_ids, hop_offsets);
        GNN_LAUNCH_CHECK("as_small_kernel");
    } else {
        as_init_kernel<<<grid_for(n > L + 2 ? n : L + 2, 256, 2048), 256, 0, stream>>>(dist, n, visited[0], seen, nw, ctrl, (int32_t)ctrl_words,
                                                                                       hop_offsets, L);
        GNN_LAUNCH_CHECK("as_init_kernel");
    }
    if (n > 0 && !small) {
        if (n_targets > 0) {
            as_seed_kernel<<<grid_for(n_targets, 256, 2048), 256, 0, stream>>>(targets, n_targets, n, seen);
            GNN_LAUNCH_CHECK("as_seed_kernel");
        }
        AsArgs a;
        a.row_ptr = g->row_ptr; a.col_idx = g->col_idx;
        a.row_ptr_t = gt != nullptr ? gt->row_ptr : nullptr; a.col_idx_t = gt != nullptr ? gt->col_idx : nullptr;
        a.n = n; a.nw = nw; a.nnz_t = gt != nullptr ? gt->nnz : 0; a.many = nb > kAsOneSlot;
        a.ring_ids = ring_ids; a.hop_offsets = hop_offsets; a.seen = seen; a.frontier = frontier; a.hubq = hubq; a.ctrl = (AsCtrl*)ctrl;
        const int pull_grid = gt != nullptr ? grid_for(nw * kWave, 256, 8192) : 1;   // a wavefront per 32 vertices
        const int grid = pull_grid > (int)kAsPushBlocks ? pull_grid : (int)kAsPushBlocks;
        for (int32_t ring = 0; ring <= L; ++ring) {
            a.visited = visited[ring & 1];
            if (ring > 0) {
                as_expand_kernel<<<grid, 256, 0, stream>>>(a, ring - 1);
                GNN_LAUNCH_CHECK("as_expand_kernel");
                if (g->nnz > kAsHubDegree) {   // else no row is long enough to be queued
                    as_expand_hubs_kernel<<<grid_for(g->nnz / kAsHubDegree * 16, 1, 2048), 256, 0, stream>>>(a, ring - 1);
                    GNN_LAUNCH_CHECK("as_expand_hubs_kernel");
                }
            }
            GNN_CHECK(as_emit(seen, visited[ring & 1], visited[(ring + 1) & 1], nw, nb, blk_cnt, hop_offsets, ring, ring_ids, dist, frontier,
                              a.row_ptr, a.row_ptr_t, (AsCtrl*)ctrl, stream));
        }
    }
    if (hop_offsets_host != nullptr) {
        GNN_HIP(hipMemcpyAsync(hop_offsets_host, hop_offsets, sizeof(int64_t) * (size_t)(L + 2), hipMemcpyDeviceToHost, stream));
        GNN_HIP(hipStreamSynchronize(stream));
    }
    return GNN_OK;
}

extern "C" int32_t gnn_eas_traverse(const gnn_csr* g, const int32_t* targets, int32_t n_targets, int32_t hops, int32_t fanout,
                                    int32_t rule, uint64_t seed, int32_t* dist, int32_t* ring_ids, int64_t* hop_offsets,
                                    int64_t* hop_offsets_host, void* ws, size_t* ws_bytes, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    GNN_CHECK(check_csr(g, "g"));
    GNN_REQUIRE(g->n_rows == g->n_cols, GNN_ERR_SHAPE, "the traversal needs a square graph (%d x %d)", g->n_rows, g->n_cols);
    GNN_REQUIRE(hops >= 1 && hops <= 1024, GNN_ERR_INVALID_ARG, "hops = %d out of range [1, 1024]", hops);
    GNN_REQUIRE(fanout >= 0, GNN_ERR_INVALID_ARG, "fanout < 0");
    GNN_REQUIRE(rule == GNN_EAS_HASH || rule == GNN_EAS_DEGREE, GNN_ERR_INVALID_ARG, "unknown selection rule %d", rule);
    GNN_REQUIRE(n_targets >= 0, GNN_ERR_INVALID_ARG, "n_targets < 0");
    const int32_t n = g->n_rows;
    const int64_t nw = ((int64_t)n + 31) / 32;
    const int64_t nb = nw > 0 ? (nw + kAsWordsPerBlock - 1) / kAsWordsPerBlock : 1;

    WsCarver carve(ws);
    uint32_t* visited2[2];
    visited2[0] = carve.take<uint32_t>((size_t)nw + 1);
    visited2[1] = nb > kAsSelfCount ? visited2[0] : carve.take<uint32_t>((size_t)nw + 1);
    uint8_t* seen = carve.take<uint8_t>((size_t)nw * 32 + 32);
    int32_t* blk_cnt = carve.take<int32_t>((size_t)nb + 1);
    int32_t* conn = carve.take<int32_t>(rule == GNN_EAS_DEGREE ? (size_t)n + 1 : 1);
    bool query;
    GNN_CHECK(ws_protocol(ws, ws_bytes, carve.used, &query));
    if (query) return GNN_OK;

    GNN_REQUIRE(hop_offsets != nullptr, GNN_ERR_INVALID_ARG, "hop_offsets is NULL");
    GNN_REQUIRE(n == 0 || (dist != nullptr && ring_ids != nullptr), GNN_ERR_INVALID_ARG, "dist / ring_ids is NULL");
    GNN_REQUIRE(n_targets == 0 || targets != nullptr, GNN_ERR_INVALID_ARG, "targets is NULL");

    as_init_kernel<<<grid_for(n > hops + 2 ? n : hops + 2, 256, 2048), 256, 0, stream>>>(dist, n, visited2[0], seen, nw, nullptr, 0, hop_offsets, hops);
    GNN_LAUNCH_CHECK("as_init_kernel");
    if (n > 0) {
        if (n_targets > 0) {
            as_seed_kernel<<<grid_for(n_targets, 256, 2048), 256, 0, stream>>>(targets, n_targets, n, seen);
            GNN_LAUNCH_CHECK("as_seed_kernel");
        }
        for (int32_t ring = 0; ring <= hops; ++ring) {
            const uint32_t* visited = visited2[ring & 1];
            if (ring > 0) {
                if (rule == GNN_EAS_DEGREE) {
                    eas_connections_kernel<<<grid_for((int64_t)n * 16, 256, 1 << 16), 256, 0, stream>>>(g->row_ptr, g->col_idx, n, visited, conn);
                    GNN_LAUNCH_CHECK("eas_connections_kernel");
                }
                eas_expand_kernel<<<2048, 256, 0, stream>>>(g->row_ptr, g->col_idx, ring_ids, hop_offsets, ring - 1, visited, seen, fanout,
                                                            rule, mix64(seed + (uint64_t)ring), conn);
                GNN_LAUNCH_CHECK("eas_expand_kernel");
                eas_expand_long_kernel<<<2048, 256, 0, stream>>>(g->row_ptr, g->col_idx, ring_ids, hop_offsets, ring - 1, visited, seen, fanout,
                                                                 rule, mix64(seed + (uint64_t)ring), conn);
                GNN_LAUNCH_CHECK("eas_expand_long_kernel");
            }
            GNN_CHECK(as_emit(seen, visited, visited2[(ring + 1) & 1], nw, nb, blk_cnt, hop_offsets, ring, ring_ids, dist, nullptr, nullptr,
                              nullptr, nullptr, stream));
        }
    }
    if (hop_offsets_host != nullptr) {
        GNN_HIP(hipMemcpyAsync(hop_offsets_host, hop_offsets, sizeof(int64_t) * (size_t)(hops + 2), hipMemcpyDeviceToHost, stream));
        GNN_HIP(hipStreamSynchronize(stream));
    }
    return GNN_OK;
}
