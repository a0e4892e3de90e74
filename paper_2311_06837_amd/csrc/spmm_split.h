// Split route of the aggregation: entries whose neighbour is among the most frequent ones ("hot") are added up from a table
// that fits the L2 of a compute die, the rest by the row kernel.
//
// What bounds the row kernel on a graph far larger than the caches is the path between L2 and the fabric: whole rows gathered at
// random arrive at 7.3 to 7.8 TB/s whatever the kernel does, out of an L2 at 27 to 31 (measured, 256 floats a row).  In a
// power-law graph a few ten thousand neighbours hold half of the entries, but a die's 4 MB hold only 4096 rows of 1 KB, and
// the other rows passing through push those out.  So the feature axis is cut into slabs of 32 floats (one cache line) and a
// die works on one slab at a time: 65 535 rows of a slab are 8 MB, the most frequent half of which stays in L2.  The slab
// rows are copied side by side (slab-major): gathered in place, 1 KB apart, 32 768 lines run at 18 TB/s, side by side at 27.
//
// Launches of a call:
//   split_degrees   lengths of the rows of the graph, as a histogram per workgroup: in a symmetric graph the length of row u is
//                   also how often u is a neighbour
//   split_assign    the longest rows that fit the table become hot: a slot number per neighbour (0: not hot)
//   split_table     copies the hot rows (times the neighbour scale), and looks 65 536 entries up: the route goes on only if
//                   enough of them are hot (a graph that is not symmetric, or not skewed, runs as before)
//   split_entries   per chunk of 8192 entries: every row's hot entries as slot numbers, padded to fours with the zero row,
//                   one row after the other; its other ids moved together to the row's start
//   split_sum       32 groups of eight lanes share a chunk's fours evenly; the sums of a row ("parts": one for every
//                   group that has some of the row) go to a plane of floats
//   spmm_rows       the row kernel over the other ids; a row starts from the sum of its parts
// No atomics on sums: which entries meet in which sum depends on the graph alone, and so do the results, bit for bit.
//
// Measured, fp32, rows of 50 (us): 1.2 M x 256 columns, 61 M entries, 55 % of them hot: row kernel alone 8900; now
// 6880 = 50 (first three) + 380 + 1650 (35 GB out of the table) + 4800 (row kernel, 33 GB from the fabric at 6.8 TB/s).  2.45 M x 100
// columns: 9900; now 8250 = 50 + 790 + 1550 + 5850.  A table of 32 768 rows gathers faster (27 TB/s, not 23) but leaves more to
// the fabric (gathers alone 1.08 + 4.45 ms, not 1.51 + 3.74); 131 072 rows 2.2 + 3.07.  Hot and other rows in one kernel, slab by
// slab: 6.8 ms gathers alone (the others push the hot ones out, whatever the cache hint of their loads).
#pragma once
#include "scan.h"
#include "spmm_fours.h"

namespace gnnhot {

constexpr int kSplitChunk = 8192;        // entries per chunk
constexpr int kSplitWords = kSplitChunk / 64;
constexpr int kSplitGroups = 32;         // lane groups that share a chunk
constexpr int kSplitSlots = 65535;       // hot neighbours at most; slot 0 is a row of zeros
constexpr int kSplitCols = 32;           // floats of a slab: one cache line
constexpr int kSplitBlocks = 256;        // workgroups of the passes over the neighbours
constexpr int kSplitBins = 256;          // bins of the histogram of row lengths: eight an octave
constexpr int kSplitSamples = 65536;
constexpr int kSplitMaxSpan = 32768;     // rows that a chunk may span
constexpr int kSplitSampleBlocks = kSplitSamples / 256;
// A row's hot entries in a chunk are split off only if they are at least so many: a part is written and read once more, which
// costs about as much as gathering this many rows.
constexpr int kSplitMin = 4;
// Hot entries among the samples from which the route goes on: about a fifth of all entries make up for what it costs
// (256 columns, 50 entries a row), a quarter at 100 columns.
constexpr int kSplitMinShare = kSplitSamples / 4;
constexpr int kSplitTableBlocks = 2048;
// slot numbers of a chunk at most: a row of k >= 4 hot entries takes at most 1.75 k
constexpr int kSplitStage = kSplitChunk / 4 * 7;
constexpr int kSplitQuadWords = (kSplitStage / 4 + 63) / 64;
static_assert(kSplitMin >= 4, "kSplitStage counts on it");

struct SplitRow {        // of a row with entries: its parts and its other entries in the chunk where it starts
    int32_t part;
    uint16_t n_parts;
    uint16_t n_cold;
};
struct SplitChunk {
    int32_t part0;       // part of the chunk's first four
    int32_t n_quads;
    uint16_t head_parts, head_cold;   // of the row that began in an earlier chunk
    int32_t pad;
};

// Slot of neighbour u < n_nbr, 0 if it is not hot.  A bit and a count per 32 neighbours (600 KB for 2.4 million) stay in L2, slot
// numbers themselves would not: split_entries 0.61 -> 0.53 ms for 61 M entries of 1.2 M neighbours, 1.33 -> 1.09 for 125 M of 2.4 M.
__device__ __forceinline__ uint32_t split_slot(const uint2 w, int32_t u) {
    const uint32_t bit = 1u << (u & 31);
    return (w.x & bit) != 0 ? w.y + __popc(w.x & (bit - 1u)) : 0u;
}

struct SplitArgs {
    const int32_t* row_ptr;
    const int32_t* col_idx;
    int32_t n_active;        // rows 0 .. n_active - 1
    int32_t n_nbr;           // neighbours that may be hot: ids below this are gathered and have a row
    int32_t limit;           // entries >= limit are dropped (rows sorted by column), or INT32_MAX
    int64_t n_chunks;
    const void* X;           // floats
    int64_t ldx;
    int32_t F, n_slabs;
    const float* nbr_scale;
    // workspace
    int32_t* hist;           // [kSplitBlocks][kSplitBins]
    int32_t* hits;           // [kSplitSampleBlocks]
    int32_t* ctrl;           // [0] hot neighbours, [1] 1: the route goes on
    int32_t* first_row;      // [n_chunks + 1] row that holds a chunk's first entry; at the end the last row with entries
    uint2* slot;             // [ceil(n_nbr / 32)] x: bit: hot, y: slot of the first of them
    int32_t* hot;            // [kSplitSlots + 1] neighbour of a slot
    float* table;            // [n_slabs][kSplitSlots + 1][kSplitCols]
    uint16_t* stream;        // [n_chunks][kSplitStage]
    uint64_t* ends;          // [n_chunks][kSplitQuadWords] bit: the four is the last of its row
    uint16_t* before;        // [n_chunks][kSplitGroups] rows that end before a group's first four
    int32_t* cold;           // [n_chunks * kSplitChunk]
    SplitRow* rows;          // [n_active]
    SplitChunk* chunks;      // [n_chunks]
    float* plane;            // [n_parts][n_slabs][kSplitCols]
    int64_t n_parts;
};

__device__ __forceinline__ int split_bin(int32_t len) {
    return len <= 0 ? 0 : (int)(__float_as_uint((float)len) >> 20) - (127 << 3) + 1;     // at most 249
}

__device__ __forceinline__ void split_range(int32_t n, int32_t& lo, int32_t& hi) {      // the neighbours of a workgroup
    const int32_t per = ((n + kSplitBlocks - 1) / kSplitBlocks + 63) / 64 * 64;
    const int64_t a = (int64_t)blockIdx.x * per, b = a + per;
    lo = (int32_t)(a < n ? a : n);
    hi = (int32_t)(b < n ? b : n);
}

static __global__ __launch_bounds__(1024) void split_degrees_kernel(SplitArgs a) {
    __shared__ int32_t s_bin[kSplitBins];
    for (int i = threadIdx.x; i < kSplitBins; i += 1024) s_bin[i] = 0;
    __syncthreads();
    int32_t lo, hi;
    split_range(a.n_nbr, lo, hi);
    for (int32_t u = lo + (int)threadIdx.x; u < hi; u += 1024) atomicAdd(&s_bin[split_bin(a.row_ptr[u + 1] - a.row_ptr[u])], 1);
    split_range(a.n_active, lo, hi);
    const int32_t m0 = a.row_ptr[0];
    for (int32_t r = lo + (int)threadIdx.x; r < hi; r += 1024) {
        const int64_t x = a.row_ptr[r], y = a.row_ptr[r + 1];
        for (int64_t c = x == m0 ? x / kSplitChunk : (x + kSplitChunk - 1) / kSplitChunk; c * kSplitChunk < y && y > x; ++c) a.first_row[c] = r;
        if (y > x && y == a.row_ptr[a.n_active]) a.first_row[a.n_chunks] = r;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSplitBins; i += 1024) a.hist[(int64_t)blockIdx.x * kSplitBins + i] = s_bin[i];
}

static __global__ __launch_bounds__(1024) void split_assign_kernel(SplitArgs a) {
    __shared__ int32_t s_all[4][kSplitBins], s_mine[4][kSplitBins];
    __shared__ int s_scan[16];
    __shared__ int32_t s_least, s_base, s_count;
    const int tid = (int)threadIdx.x, bin = tid & (kSplitBins - 1), part = tid / kSplitBins;
    static_assert(kSplitBins == 256 && kSplitBlocks % 4 == 0, "four threads a bin");
    int32_t all = 0, mine = 0;     // neighbours of the bin, and those of them before this workgroup's range
#pragma unroll 16
    for (int j = part * (kSplitBlocks / 4); j < (part + 1) * (kSplitBlocks / 4); ++j) {
        const int32_t c = a.hist[(int64_t)j * kSplitBins + bin];
        all += c;
        if (j < (int)blockIdx.x) mine += c;
    }
    s_all[part][bin] = all;
    s_mine[part][bin] = mine;
    if (tid == 0) s_least = kSplitBins;
    __syncthreads();
    // from the longest rows down: thread t holds bin 255 - t
    int32_t n = 0, m = 0;
    if (tid < kSplitBins) {
        for (int q = 0; q < 4; ++q) {
            n += s_all[q][kSplitBins - 1 - tid];
            m += s_mine[q][kSplitBins - 1 - tid];
        }
    }
    int total, all_len, hot_len;
    const int before = block_exclusive_scan<1024>(n, s_scan, &total);
    const bool fits = tid < kSplitBins - 1 && before + n <= kSplitSlots;      // (bin 0: rows without entries)
    if (fits) atomicMin(&s_least, kSplitBins - 1 - tid);
    __syncthreads();
    int least = s_least;
    // entries of the bin, at least (below nnz in all).  In a symmetric graph these are also the entries that name them: too few
    // of them in the table, and nothing is taken
    const int len = tid < kSplitBins - 1 ? n * (int)__uint_as_float((uint32_t)(kSplitBins - 2 - tid + (127 << 3)) << 20) : 0;
    block_exclusive_scan<1024>(len, s_scan, &all_len);
    block_exclusive_scan<1024>(kSplitBins - 1 - tid >= least ? len : 0, s_scan, &hot_len);
    if ((int64_t)hot_len * kSplitSamples < (int64_t)all_len * kSplitMinShare) least = kSplitBins;
    const bool taken = tid < kSplitBins && kSplitBins - 1 - tid >= least;
    block_exclusive_scan<1024>(taken ? m : 0, s_scan, &total);
    if (tid == 0) s_base = total;
    block_exclusive_scan<1024>(taken ? n : 0, s_scan, &total);
    if (tid == 0) s_count = total;
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) a.ctrl[0] = s_count;
    int32_t lo, hi;
    split_range(a.n_nbr, lo, hi);
    int32_t base = s_base + 1;
    for (int32_t u0 = lo; u0 < hi; u0 += 1024) {
        const int32_t u = u0 + tid;
        const bool hot = u < hi && split_bin(a.row_ptr[u + 1] - a.row_ptr[u]) >= least;
        const int rank = block_exclusive_scan<1024>(hot ? 1 : 0, s_scan, &total);
        const uint64_t bits = __ballot(hot);
        if (u < hi && (u & 31) == 0) a.slot[u >> 5] = make_uint2((uint32_t)(bits >> (u & 32)), (uint32_t)(base + rank));
        if (hot) a.hot[base + rank] = u;
        base += total;
    }
}

// Last row with entries in a chunk that has some.
__device__ __forceinline__ int32_t split_last_row(const SplitArgs& a, int64_t chunk, int64_t m) {
    return (chunk + 1) * kSplitChunk < m ? a.first_row[chunk + 1] : a.first_row[a.n_chunks];
}

// Slab s of the table: 8 lanes a row, 16 bytes a lane.  The blocks behind those of the table look at samples.
static __global__ __launch_bounds__(256) void split_table_kernel(SplitArgs a) {
    constexpr int table_blocks = kSplitTableBlocks;
    const int n_hot = a.ctrl[0];
    if ((int)blockIdx.x >= table_blocks) {
        __shared__ int s_scan[4];
        const int64_t m = a.row_ptr[a.n_active];
        const int64_t i = (int64_t)((int)blockIdx.x - table_blocks) * 256 + threadIdx.x;
        int hit = 0, total;
        if (m > 0) {
            const int32_t u = a.col_idx[(i * m) / kSplitSamples];
            hit = u < a.n_nbr && u < a.limit && split_slot(a.slot[u >> 5], u) != 0;
        }
        // a chunk that spans very many rows (nearly all of them empty) would be walked by one workgroup: not this route
        for (int64_t c = i; c < a.n_chunks; c += kSplitSamples) {
            const int64_t e0 = c * kSplitChunk;
            if (e0 < m && e0 + kSplitChunk > a.row_ptr[0] && split_last_row(a, c, m) - a.first_row[c] > kSplitMaxSpan) hit = -2 * kSplitSamples;
        }
        block_exclusive_scan<256>(hit, s_scan, &total);
        if (threadIdx.x == 0) a.hits[(int)blockIdx.x - table_blocks] = total;
        return;
    }
    const int64_t per_row = (int64_t)a.n_slabs * 8;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < (int64_t)(n_hot + 1) * per_row; t += (int64_t)table_blocks * 256) {
        const int32_t row = (int32_t)(t / per_row);
        const int32_t c = (int32_t)(t % per_row) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row > 0 && c < a.F) {
            const int32_t u = a.hot[row];
            const float w = a.nbr_scale ? a.nbr_scale[u] : 1.f;
            v = *(const float4*)((const float*)a.X + (int64_t)u * a.ldx + c);
            v.x *= w; v.y *= w; v.z *= w; v.w *= w;
        }
        *(float4*)(a.table + ((int64_t)(c / kSplitCols) * (kSplitSlots + 1) + row) * kSplitCols + c % kSplitCols) = v;
    }
}

// Per workgroup a chunk of entries.  The rows of a chunk are a few hundred, so the work between two barriers is short and the
// barriers count: all sums over words are taken by one wavefront, the rows are visited once (again only where a chunk has more
// than 1024).  61 M entries of 1.2 M neighbours, 50 a row: 0.38 ms, 125 M of 2.4 M 0.79 (0.53 / 1.09 with a block-wide sum at
// every step and a search for the chunk's first row: that code also spilled).
template <bool CUT>
__global__ __launch_bounds__(1024, 8) void split_entries_kernel(SplitArgs a) {
    constexpr int NE = kSplitChunk / 1024, NW = kSplitWords;
    __shared__ uint64_t s_hot[NW + 1], s_kept[CUT ? NW + 1 : 1], s_start[NW], s_end[64];
    __shared__ int s_hot_pre[NW + 1], s_kept_pre[CUT ? NW + 1 : 1], s_start_pre[NW], s_end_pre[64];
    __shared__ uint32_t s_row[kSplitChunk + 1];      // of the chunk's j-th row: hot entries before it, and << 16 where its slots go (all ones: not split)
    __shared__ __attribute__((aligned(16))) uint16_t s_stage[kSplitStage];
    __shared__ int s_scan[16];
    static_assert(NW == 128 && kSplitQuadWords <= 64 && kSplitSampleBlocks == 256, "sums over words by one wavefront");
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int64_t chunk = blockIdx.x;
    // does the route go on?  (every wavefront adds up the same numbers)
    int hits = a.hits[lane] + a.hits[lane + 64] + a.hits[lane + 128] + a.hits[lane + 192];
    hits = __shfl(wave_inclusive_scan(hits), 63, kWave);
    const bool on = hits >= kSplitMinShare;
    if (chunk == 0 && tid == 0) a.ctrl[1] = on ? 1 : 0;
    if (!on) return;
    const int64_t m = a.row_ptr[a.n_active], m0 = a.row_ptr[0];
    const int64_t e0 = chunk * kSplitChunk;
    if (e0 >= m || e0 + kSplitChunk <= m0) {
        if (tid == 0) a.chunks[chunk] = SplitChunk{0, 0, 0, 0, 0};
        return;
    }
    const int n = (int)(m - e0 < kSplitChunk ? m - e0 : kSplitChunk), n0 = (int)(m0 > e0 ? m0 - e0 : 0);
    const int32_t r0 = a.first_row[chunk];
    const int32_t r_end = split_last_row(a, chunk, m) + 1;      // rows with entries here lie in [r0, r_end)
    const uint32_t n_rows = (uint32_t)(r_end - r0);
    const bool few = n_rows <= 1024;
    // ---- the entries: id, or slot of a hot one, in registers; which they are as bits
    const int32_t* const ids = a.col_idx + e0;     // (uniform: a lane's place is a dword beside it)
    int32_t* const cold = a.cold + e0;
    int32_t u[NE];
    uint64_t hot[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) u[i] = ids[i * 1024 + tid < n ? (uint32_t)(i * 1024 + tid) : (uint32_t)(n - 1)];
    if (tid < NW) s_start[tid] = 0;
    if (tid < 64) s_end[tid] = 0;
    uint2 w[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) w[i] = *(const uint2*)((const char*)a.slot + ((uint32_t)(u[i] < a.n_nbr ? u[i] : 0) >> 5 << 3));
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const bool in = i * 1024 + tid < n && i * 1024 + tid >= n0, kept = in && (!CUT || u[i] < a.limit);
        const uint32_t q = kept && u[i] < a.n_nbr ? split_slot(w[i], u[i]) : 0u;
        hot[i] = __ballot(q != 0);
        if (q != 0) u[i] = (int32_t)q;
        if (lane == 0) s_hot[i * 16 + wave] = hot[i];
        if (CUT) {
            const uint64_t k = __ballot(kept);
            if (lane == 0) s_kept[i * 16 + wave] = k;
        }
    }
    // words' counts before each of NW words (and behind the last), by one wavefront
    auto prefix = [&](const uint64_t* words, int* pre, bool total) {
        const int c0 = __popcll(words[2 * lane]), c1 = __popcll(words[2 * lane + 1]);
        const int inc = wave_inclusive_scan(c0 + c1);
        pre[2 * lane] = inc - c0 - c1;
        pre[2 * lane + 1] = inc - c1;
        if (total && lane == 63) pre[NW] = inc;
    };
    __syncthreads();
    if (wave == 0) {
        if (lane == 0) s_hot[NW] = 0;
        prefix(s_hot, s_hot_pre, true);
    }
    if (CUT && wave == 1) {
        if (lane == 0) s_kept[NW] = 0;
        prefix(s_kept, s_kept_pre, true);
    }
    __syncthreads();
    // hot entries among the first x of the chunk, kept ones, rows that start at or before x
    auto hot_rank = [&](int x) { return s_hot_pre[x >> 6] + __popcll(s_hot[x >> 6] & ((1ull << (x & 63)) - 1ull)); };
    auto kept_rank = [&](int x) { return CUT ? s_kept_pre[x >> 6] + __popcll(s_kept[x >> 6] & ((1ull << (x & 63)) - 1ull)) : x; };
    auto start_rank = [&](int x) { return s_start_pre[x >> 6] + __popcll(s_start[x >> 6] & (~0ull >> (63 - (x & 63)))); };
    // ---- the rows, 1024 at a time: f(row, starts here, first entry, end, has entries here)
    const int32_t* const ptr = a.row_ptr + r0;
    auto visit = [&](uint32_t r, auto f) {
        int x = n, y = n;              // where the row's entries lie in the chunk
        bool starts = true;
        if (r < n_rows) {
            const int64_t s = (int64_t)ptr[r] - e0, e = (int64_t)ptr[r + 1] - e0;
            starts = s >= 0;
            x = s < 0 ? 0 : (int)(s < n ? s : n);
            y = (int)(e < n ? e : n);
        }
        f(r, starts, x, y, y > x);
    };
    int fours = 0, n_quads;
    for (uint32_t r = tid; r < n_rows; r += 1024)
        visit(r, [&](uint32_t, bool starts, int x, int y, bool in) {
            if (!in) return;
            if (starts) atomicOr((unsigned long long*)&s_start[x >> 6], 1ull << (x & 63));
            const int k = hot_rank(y) - hot_rank(x);
            if (k >= kSplitMin) fours += ((k + 3) / 4) << 16 | 1;
        });
    const int at0 = block_exclusive_scan<1024>(fours, s_scan, &n_quads);     // fours << 16 | split rows before this thread's
    n_quads >>= 16;
    if (wave == 0) prefix(s_start, s_start_pre, false);
    for (int q = tid; q < (n_quads + 1) / 2; q += 1024) *(uint4*)(s_stage + q * 8) = make_uint4(0, 0, 0, 0);   // (kSplitStage: whole eights)
    __syncthreads();
    const int per = (n_quads + kSplitGroups - 1) / kSplitGroups;     // fours of a group
    const int32_t part0 = (int32_t)(r0 + chunk * (kSplitGroups + 1));
    int run = 0;
    int head_parts = 0, head_cold = 0;
    for (uint32_t r = 0; r < n_rows; r += 1024) {
        visit(r + tid, [&](uint32_t row, bool starts, int x, int y, bool in) {
            const int h0 = in ? hot_rank(x) : 0, k = in ? hot_rank(y) - h0 : 0;
            const bool split = k >= kSplitMin;
            int at = at0;
            if (!few) {
                int total;
                at = run + block_exclusive_scan<1024>(split ? ((k + 3) / 4) << 16 | 1 : 0, s_scan, &total);
                run += total;
            }
            if (!in) return;
            const int q0 = at >> 16, i = at & 0xffff, q1 = q0 + (k + 3) / 4;
            const int j = starts ? start_rank(x) : 0;
            s_row[j] = (uint32_t)h0 | (split ? (uint32_t)(q0 * 4) : 0xffffu) << 16;
            const int n_cold = kept_rank(y) - kept_rank(x) - (split ? k : 0);
            int n_parts = 0, first = 0;
            if (split) {
                first = i + q0 / per;
                n_parts = (q1 - 1) / per - q0 / per + 1;
                atomicOr((unsigned long long*)&s_end[(q1 - 1) >> 6], 1ull << ((q1 - 1) & 63));
            }
            if (starts) {
                a.rows[r0 + row] = SplitRow{part0 + first, (uint16_t)n_parts, (uint16_t)n_cold};
            } else {                                                 // row r0: thread 0 in the first step
                head_parts = n_parts;
                head_cold = n_cold;
            }
        });
    }
    if (tid == 0) a.chunks[chunk] = SplitChunk{part0, n_quads, (uint16_t)head_parts, (uint16_t)head_cold, 0};
    __syncthreads();
    // ---- entries to their places: the masks of a step's 64 entries are the wavefront's own
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int x = i * 1024 + tid;
        const uint64_t starts = s_start[i * 16 + wave];
        const int j = s_start_pre[i * 16 + wave] + __popcll(starts & (below << 1 | 1ull)), hot_before = s_hot_pre[i * 16 + wave] + __popcll(hot[i] & below);
        if (x < n && x >= n0) {
            const uint32_t d = s_row[j];
            const int rank = hot_before - (int)(d & 0xffffu), dst = (int)(d >> 16);
            const bool is_hot = (hot[i] >> lane) & 1ull;
            const bool whole = dst == 0xffff;                        // the row is not split
            int32_t v = u[i];
            if (whole && is_hot) v = ids[(uint32_t)x];
            if (!whole && is_hot) s_stage[dst + rank] = (uint16_t)v;
            else cold[(uint32_t)(whole ? x : x - rank)] = v;
        }
    }
    if (wave == 15) {      // rows that end before every group's first four
        const uint64_t w = s_end[lane];
        const int c = __popcll(w);
        s_end_pre[lane] = wave_inclusive_scan(c) - c;
        if (lane < kSplitQuadWords) a.ends[chunk * kSplitQuadWords + lane] = w;
        wave_lds_sync();
        const int q = lane * per;
        if (lane < kSplitGroups && q < n_quads)
            a.before[chunk * kSplitGroups + lane] = (uint16_t)(s_end_pre[q >> 6] + __popcll(s_end[q >> 6] & ((1ull << (q & 63)) - 1ull)));
    }
    __syncthreads();
    for (int q = tid; q < (n_quads + 1) / 2; q += 1024) *(uint4*)(a.stream + chunk * kSplitStage + q * 8) = *(const uint4*)(s_stage + q * 8);
}

// Lane j of every group of eight, to all of its group (no bank conflicts, no memory: the lanes' crossbar).
template <int J>
__device__ __forceinline__ uint32_t split_bcast(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x18 | (J << 5));
}

template <int J>
__device__ __forceinline__ void split_load(const char* tab, uint32_t lane_off, uint32_t ex, uint32_t ey, float4 (&x)[4]) {
    const uint32_t p = split_bcast<J>(ex), q = split_bcast<J>(ey);
    x[0] = *(const float4*)(tab + ((p & 0xffffu) * (kSplitCols * 4) + lane_off));
    x[1] = *(const float4*)(tab + ((p >> 16) * (kSplitCols * 4) + lane_off));
    x[2] = *(const float4*)(tab + ((q & 0xffffu) * (kSplitCols * 4) + lane_off));
    x[3] = *(const float4*)(tab + ((q >> 16) * (kSplitCols * 4) + lane_off));
}

__device__ __forceinline__ void split_add(float4& s, const float4 (&x)[4]) {
    s.x += (x[0].x + x[1].x) + (x[2].x + x[3].x);
    s.y += (x[0].y + x[1].y) + (x[2].y + x[3].y);
    s.z += (x[0].z + x[1].z) + (x[2].z + x[3].z);
    s.w += (x[0].w + x[1].w) + (x[2].w + x[3].w);
}

// Workgroup b runs on die b mod 8 and takes unit b / 8 of the die's: the units (slab, chunk) of the chunks in use are dealt to the
// dies in eight stretches, slab by slab, so a die meets few slabs, one after the other, at any width.  A lane of eight holds every eighth
// four of its group's stretch and hands it round; a load of 1 KB (eight table rows) costs about seven vector instructions
// where the vector cache takes as long as sixteen.
static __global__ __launch_bounds__(256, 6) void split_sum_kernel(SplitArgs a) {
    if (a.ctrl[1] == 0) return;
    const int64_t used = ((int64_t)a.row_ptr[a.n_active] + kSplitChunk - 1) / kSplitChunk;
    const int64_t units = used * a.n_slabs, per_die = (units + 7) / 8;
    const int64_t unit = (int64_t)(blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_die || unit >= units) return;
    const int slab = (int)(unit / used);
    const int64_t chunk = unit - (int64_t)slab * used;
    const SplitChunk info = a.chunks[chunk];
    if (info.n_quads == 0) return;
    const int lane = lane_id(), sl = lane & 7, g = (int)(threadIdx.x >> 3);
    const int per = (info.n_quads + kSplitGroups - 1) / kSplitGroups;
    const int lo = g * per;
    int cnt = info.n_quads - lo;
    cnt = cnt < 0 ? 0 : (cnt < per ? cnt : per);
    const char* tab = (const char*)(a.table + (int64_t)slab * (kSplitSlots + 1) * kSplitCols);
    const uint32_t lane_off = (uint32_t)sl * 16u;
    const uint2* stream = (const uint2*)(a.stream + chunk * kSplitStage);
    const uint32_t* ends = (const uint32_t*)(a.ends + chunk * kSplitQuadWords);
    const int64_t step = (int64_t)a.n_slabs * kSplitCols;
    float* out = a.plane + (info.part0 + g + (cnt > 0 ? (int)a.before[chunk * kSplitGroups + g] : 0)) * step + slab * kSplitCols + sl * 4;
    uint2 e = make_uint2(0, 0);
    uint32_t w = 0;
    if (sl < cnt) {
        e = stream[lo + sl];
        w = ends[(lo + sl) >> 5];
    }
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q = 0; q < per; q += 8) {
        const uint32_t ex = e.x, ey = e.y;
        const bool mine = q + sl < cnt && (((w >> ((lo + q + sl) & 31)) & 1u) != 0u || q + sl == cnt - 1);
        const uint32_t stores = (uint32_t)(__ballot(mine) >> (lane & 56)) & 0xffu;      // bit j: the group stores after its j-th four
        e = make_uint2(0, 0);
        if (q + 8 + sl < cnt) {
            e = stream[lo + q + 8 + sl];
            w = ends[(lo + q + 8 + sl) >> 5];
        }
        auto done = [&](int j) {
            if ((stores >> j) & 1u) {
                // past the L2s, which are to keep the table (us, without / with: 1.2 M rows of 50, 256 columns 7059 / 6917; 100 k of 60, 602 1139 / 1105)
                __builtin_nontemporal_store(FourRaw{__float_as_uint(s.x), __float_as_uint(s.y), __float_as_uint(s.z), __float_as_uint(s.w)}, (FourRaw*)out);
                out += step;
                s = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        };
        float4 x[4], y[4];
        split_load<0>(tab, lane_off, ex, ey, x);
        split_load<1>(tab, lane_off, ex, ey, y);
        split_add(s, x); done(0);
        split_load<2>(tab, lane_off, ex, ey, x);
        split_add(s, y); done(1);
        split_load<3>(tab, lane_off, ex, ey, y);
        split_add(s, x); done(2);
        split_load<4>(tab, lane_off, ex, ey, x);
        split_add(s, y); done(3);
        split_load<5>(tab, lane_off, ex, ey, y);
        split_add(s, x); done(4);
        split_load<6>(tab, lane_off, ex, ey, x);
        split_add(s, y); done(5);
        split_load<7>(tab, lane_off, ex, ey, y);
        split_add(s, x); done(6);
        split_add(s, y); done(7);
    }
}

}  // namespace gnnhot
