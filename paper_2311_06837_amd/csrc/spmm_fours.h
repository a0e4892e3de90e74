// Column-blocked aggregation over the first rows of a graph (no row list, and enough of them: fours_pay): the entries that a
// workgroup gathers are laid out once a call as a stream of fours and summed up slab by slab.
//
// A slab is one cache line of every row (32 floats or 64 bfloat16), so a die's block of 32 768 neighbours on average stays in its 4 MB L2
// (65 535 at most, 8 MB, where few ids hold most entries and the others share a block), and a load of 1 KB (eight rows) takes the
// vector cache as long as sixteen vector instructions.  What the ids cost is therefore paid once a call and not once a slab:
//   spmm_fours_kernel      per (chunk of rows, block): every row's entries in the block as ids of 16 bits relative to the block's first, in
//                          fours that belong to one row; what is left of a row's last four names no id.  A row without
//                          entries there has one four all the same, so the rows of a chunk follow each other.
//   spmm_slabs_kernel      the gathered rows slab by slab, times the neighbour scale in float (lines side by side: gathered in
//                          place, 1 KB apart, a slab's lines use a part of the L2's sets)
//   spmm_four_sums_kernel  32 groups of eight lanes share a chunk's fours evenly.  The buffer descriptor ends with the block's last
//                          row: a place without id reads zeros and no memory.  A row end is a bit, tested four by four; a row cut
//                          by stretches is added up behind the only barrier, in stream order.
// The sums go to plane `block mod 8`; they depend on the graph and the call alone, bit for bit.
//
// What bounds the sums: 16 clocks of the vector cache a load (3.3 ms of the 5.0 below), the row ends (0.4), L2 misses (6 % of the
// requests at 233 000 rows, where a die's block just fits: 0.5).  Measured, 256 columns, the whole call, us, 256-byte slabs whose ids are
// staged anew for every slab (spmm_stream_kernel) -> now:
//   fp32, 490 entries a row: 233 000 rows 6200 -> 5730 (sums 5000, planes 370, fours 175, cut points 90, slabs 70), 165 000 4250 -> 3510, 70 000 1600
//     -> 1480; 200 000 rows of 160 2620 -> 2030, of 80 1770 -> 1390; bf16, 233 000 3730 -> 3340, with a neighbour scale 5270 -> 4430
// Of 233 000 rows: ids of 16 bits staged in LDS piece by piece, 256-byte slabs 5930, 128-byte 5910; rows gathered in place 5600 for the sums
// alone; plane stores that stay in L2 5920 instead of 5775; 9 to 16 blocks instead of 8 5930 to 6450 (more planes and row ends for
// fewer misses); seven workgroups a CU 5780, five 5720, four 5630 (but with two passes, 420 000 rows, 8620, 8700, 9040), two 6850; stages of 48 or 32
// fours 1 % slower; streams read past the caches 2 % faster here, 4 to 10 % slower at other sizes.
#pragma once
#include "scan.h"

namespace gnnhot {

typedef uint32_t FourRaw __attribute__((ext_vector_type(4)));

constexpr int kFourGroups = 32;          // lane groups of a workgroup
constexpr int kFourBytes = 128;          // of a slab
constexpr int kFourMaxRows = 1024;       // rows of a chunk
constexpr int kFourEdges = 7168;         // entries of a (chunk, block) that the host aims for: one stage of every group
constexpr int kFourStage = 64;           // fours of a group that are staged at a time
constexpr int kFourPad = 20;             // 16-byte places that keep a fifth or sixth workgroup from a CU
constexpr uint32_t kNoId = 0xffffu;
constexpr int kRawBuffer = 0x00027000;    // buffer descriptor, last word: dwords, bounds in bytes; a load beyond them returns zeros
constexpr int kBlockIds = 65535;         // ids of a block at most

struct FourArgs {
    const int32_t* row_ptr;
    const int32_t* ids;        // col_idx or its filtered copy
    const int32_t* seg;        // [n_active][n_blocks + 1] cut points of every row
    const int32_t* seg_end;    // nullable, [n_active][n_blocks]: block j ends here instead (filtered copy)
    const int32_t* bounds;     // [n_blocks + 1] first id of every block
    int32_t n_active, n_blocks, block0;
    int32_t rows_per_wg;
    const void* X;             // the gathered matrix: rows of ldx elements, the first n_src of them in use
    int64_t ldx;
    int32_t F, n_src;
    const float* nbr_scale;    // nullable; float: applied to the copied rows, bfloat16: a factor per entry
    char* slabs;               // [slabs of F][n_src][kFourBytes]
    float* part;               // 8 planes of [n_active][ldp]
    int64_t ldp;
    int32_t accumulate;        // add to the planes
    // the streams
    uint2* at;                 // [n_chunks][n_blocks] x: place of the stream, in 32 fours, y: fours
    uint2* stream;
    float4* w;                 // factors of a four
    uint32_t* ends;            // bit: the four is the last of its row
    uint16_t* before;          // [n_chunks][n_blocks][kFourGroups] rows that end before a group's first four
};

// Places (of 32 fours) that the streams of a call take at most: a four and a last one for every row, 64 more a stream.
static inline size_t four_places(int64_t nnz, int64_t n_active, int64_t n_chunks, int64_t n_blocks) {
    return (size_t)((nnz / 4 + n_active * n_blocks + 64 * n_chunks * n_blocks) / 32 + 4);
}

// Copies the gathered rows (times the neighbour scale, float) slab by slab.
template <int DT>
static __global__ __launch_bounds__(256) void spmm_slabs_kernel(FourArgs a) {
    constexpr int ES = DT == GNN_F32 ? 4 : 2, VE = 16 / ES, W = kFourBytes / ES;
    const int per_row = (a.F + W - 1) / W * (W / VE);
    const int64_t total = (int64_t)a.n_src * per_row;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        const int64_t u = t / per_row;
        const int32_t c = (int32_t)(t % per_row) * VE;
        uint4 x = make_uint4(0, 0, 0, 0);
        if (c < a.F) x = *(const uint4*)((const char*)a.X + (u * a.ldx + c) * ES);
        if (DT == GNN_F32 && a.nbr_scale) {
            const float f = a.nbr_scale[u];
            x.x = __float_as_uint(__uint_as_float(x.x) * f);
            x.y = __float_as_uint(__uint_as_float(x.y) * f);
            x.z = __float_as_uint(__uint_as_float(x.z) * f);
            x.w = __float_as_uint(__uint_as_float(x.w) * f);
        }
        *(uint4*)(a.slabs + ((int64_t)(c / W) * a.n_src + u) * kFourBytes + c % W * ES) = x;
    }
}

// Fours of a group: whole eights.
__device__ __forceinline__ int four_stretch(int n_fours) { return ((n_fours + kFourGroups - 1) / kFourGroups + 7) / 8 * 8; }

template <bool SCALED>
static __global__ __launch_bounds__(256) void spmm_fours_kernel(FourArgs a) {
    constexpr int R = kFourMaxRows / 256;        // consecutive rows of a thread
    __shared__ int32_t s_at[kFourMaxRows + 1], s_first[kFourMaxRows], s_len[kFourMaxRows];
    __shared__ int s_scan[4];
    const int tid = (int)threadIdx.x, lane = lane_id();
    const int64_t chunk = blockIdx.x / (uint32_t)a.n_blocks;
    const int block = (int)(blockIdx.x % (uint32_t)a.n_blocks);
    const int64_t chunk0 = chunk * a.rows_per_wg;
    const int n_rows = (int)(((int64_t)a.n_active - chunk0) < a.rows_per_wg ? ((int64_t)a.n_active - chunk0) : a.rows_per_wg);
    int before = 0, fours[R], sum = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int r = tid * R + i;
        fours[i] = 0;
        if (r < n_rows) {
            const int64_t v = chunk0 + r;
            const int32_t* cut = a.seg + v * (a.n_blocks + 1);
            const int32_t first = cut[block], len = (a.seg_end ? a.seg_end[v * a.n_blocks + block] : cut[block + 1]) - first;
            before += first - cut[0];
            fours[i] = len > 4 ? (len + 3) / 4 : 1;
            s_first[r] = first;
            s_len[r] = len;
        }
        sum += fours[i];
    }
    int n_fours, n_before;
    int at = block_exclusive_scan<256>(sum, s_scan, &n_fours);
    block_exclusive_scan<256>(before, s_scan, &n_before);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (tid * R + i < n_rows) s_at[tid * R + i] = at;
        at += fours[i];
    }
    if (tid == 0) s_at[n_rows] = n_fours;
    __syncthreads();
    // the streams in order: room for the rows before (a quarter of their entries and a four each) and 64 fours a stream for whole words
    const int64_t room = ((int64_t)a.row_ptr[chunk0] + n_before) / 4 + chunk0 * a.n_blocks + (int64_t)block * n_rows;
    const int64_t place = (room + 31) / 32 + 2 * (int64_t)blockIdx.x;
    if (tid == 0) a.at[blockIdx.x] = make_uint2((uint32_t)place, (uint32_t)n_fours);
    auto row_of = [&](int t) {
        int x = 0, y = n_rows;
        while (y - x > 1) {
            const int m = (x + y) >> 1;
            if (s_at[m] <= t) x = m;
            else y = m;
        }
        return x;
    };
    const int per = four_stretch(n_fours);
    if (tid < kFourGroups) a.before[(int64_t)blockIdx.x * kFourGroups + tid] = (uint16_t)(tid * per < n_fours ? row_of(tid * per) : 0);
    const uint32_t id0 = (uint32_t)a.bounds[block];
    uint2* const stream = a.stream + place * 32;
    uint32_t* const ends = a.ends + place;
    for (int t0 = tid - lane; t0 < n_fours; t0 += 256) {     // uniform over the wavefront
        const int t = t0 + lane < n_fours ? t0 + lane : n_fours - 1;
        const int x = row_of(t);
        const int k = (t - s_at[x]) * 4, left = s_len[x] - k;
        const int32_t* const p = a.ids + s_first[x];
        uint32_t u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = (uint32_t)(i < left ? p[k + i] : 0);
        float f[4];
        if (SCALED) {
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = i < left ? a.nbr_scale[u[i]] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = i < left ? u[i] - id0 : kNoId;
        const uint64_t last = __ballot(t + 1 == s_at[x + 1]);
        if (t0 + lane < n_fours) {
            stream[t] = make_uint2(u[0] | u[1] << 16, u[2] | u[3] << 16);
            if (SCALED) a.w[place * 32 + t] = make_float4(f[0], f[1], f[2], f[3]);
            if ((lane & 31) == 0) ends[t >> 5] = (uint32_t)(last >> (lane & 32));
        }
    }
}

typedef uint64_t FourBits __attribute__((aligned(1)));

template <bool SCALED>
struct FourLoads {
    FourRaw x[4];
    float w[SCALED ? 4 : 1];
};

template <bool SCALED>
__device__ __forceinline__ void four_load(__amdgpu_buffer_rsrc_t rows, uint32_t lane_off, uint32_t p, uint32_t q, const FourRaw* w, FourLoads<SCALED>& l) {
    const uint32_t id[4] = {p & 0xffffu, p >> 16, q & 0xffffu, q >> 16};
#pragma unroll
    for (int i = 0; i < 4; ++i) l.x[i] = __builtin_amdgcn_raw_buffer_load_b128(rows, id[i] * kFourBytes + lane_off, 0, 0);
    if constexpr (SCALED) {
        const FourRaw f = *w;
#pragma unroll
        for (int i = 0; i < 4; ++i) l.w[i] = __uint_as_float(f[i]);
    }
}

template <bool SCALED>
__device__ __forceinline__ void four_add(float (&s)[4], const FourLoads<SCALED>& l) {      // floats
#pragma unroll
    for (int k = 0; k < 4; ++k)
        s[k] += (__uint_as_float(l.x[0][k]) + __uint_as_float(l.x[1][k])) + (__uint_as_float(l.x[2][k]) + __uint_as_float(l.x[3][k]));
}

template <bool SCALED>
__device__ __forceinline__ void four_add(float (&s)[8], const FourLoads<SCALED>& l) {      // bfloat16
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float lo = bf16lo(l.x[i][k]), hi = bf16hi(l.x[i][k]);
            s[2 * k] = SCALED ? fmaf(l.w[SCALED ? i : 0], lo, s[2 * k]) : s[2 * k] + lo;
            s[2 * k + 1] = SCALED ? fmaf(l.w[SCALED ? i : 0], hi, s[2 * k + 1]) : s[2 * k + 1] + hi;
        }
    }
}

template <int DT, bool SCALED>
static __global__ __launch_bounds__(256, 4) void spmm_four_sums_kernel(FourArgs a) {
    constexpr int ES = DT == GNN_F32 ? 4 : 2, VE = 16 / ES, W = kFourBytes / ES;
    __shared__ __attribute__((aligned(16))) float s_head[kFourGroups][W];
    __shared__ int32_t s_head_row[kFourGroups];
    constexpr int S = SCALED ? kFourStage / 2 : kFourStage;      // fours of a group that are staged at a time
    __shared__ FourRaw s_stage[kFourGroups][S / 2 + 1 + kFourPad];      // (the odd row length puts the groups on different banks)
    __shared__ FourRaw s_w[SCALED ? kFourGroups : 1][SCALED ? S + 1 : 1];
    const int lane = lane_id(), sl = lane & 7, g = (int)(threadIdx.x >> 3);
    const int die = (int)(blockIdx.x & 7), block = a.block0 + die, slab = (int)blockIdx.y;     // (workgroup b runs on die b mod 8)
    const int64_t chunk = blockIdx.x >> 3;
    const int64_t which = chunk * a.n_blocks + block;
    const uint2 at = a.at[which];
    const int n_fours = (int)at.y, per = four_stretch(n_fours);
    const int lo = g * per;
    int cnt = n_fours - lo;
    cnt = cnt < 0 ? 0 : (cnt < per ? cnt : per);
    // the block's rows in the slab; a place without id lies beyond them
    const int32_t id0 = a.bounds[block], id1 = a.bounds[block + 1];
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(a.slabs + ((int64_t)slab * a.n_src + id0) * kFourBytes, 0,
                                                                          (uint32_t)(id1 - id0) * kFourBytes, kRawBuffer);
    const int32_t col = slab * W + sl * VE;
    const bool col_ok = col < a.F;
    const uint32_t lane_off = (uint32_t)sl * 16u;
    const uint2* const stream = a.stream + (int64_t)at.x * 32;
    const FourRaw* const factors = SCALED ? (const FourRaw*)a.w + (int64_t)at.x * 32 : nullptr;
    const uint8_t* const ends = (const uint8_t*)(a.ends + at.x);
    const int64_t chunk0 = chunk * a.rows_per_wg;
    float* const out = a.part + ((int64_t)die * a.n_active + chunk0) * a.ldp + col;
    int row = a.before[which * kFourGroups + g], head_row = -1;
    // does the stretch begin inside a row?
    bool cut = cnt > 0 && lo > 0 && ((ends[(lo > 0 ? lo - 1 : 0) >> 3] >> ((lo - 1) & 7)) & 1u) == 0u;
    bool open = false;            // s holds fours of a row that has not ended
    float s[VE];
#pragma unroll
    for (int k = 0; k < VE; ++k) s[k] = 0.f;
    auto store = [&](int r) {
        float* const q = out + (int64_t)r * a.ldp;
#pragma unroll
        for (int k = 0; k < VE; k += 4) {
            float4 v = make_float4(s[k], s[k + 1], s[k + 2], s[k + 3]);
            if (a.accumulate) {
                const float4 old = *(const float4*)(q + k);
                v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
            }
            __builtin_nontemporal_store(FourRaw{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)}, (FourRaw*)(q + k));
        }
    };
    auto head = [&]() {
        head_row = row;
#pragma unroll
        for (int k = 0; k < VE; ++k) s_head[g][sl * VE + k] = s[k];
        cut = false;
    };
    for (int q0 = 0; q0 < per; q0 += S) {
        // a wavefront stages the next S fours of its own groups: loads retire in order, so those of the rows wait for these once a
        // stage only
        FourRaw e[S / 16];
        // bit j: a row ends with the group's j-th four of the stage
        const uint64_t last = q0 < cnt ? *(const FourBits*)(ends + ((lo + q0) >> 3)) : 0ull;
#pragma unroll
        for (int i = 0; i < S / 16; ++i) {
            const int q = q0 + 16 * i + 2 * sl;
            e[i] = FourRaw{~0u, ~0u, ~0u, ~0u};
            if (q < cnt) e[i] = *(const FourRaw*)(stream + lo + q);
            if (q + 1 >= cnt) e[i][2] = e[i][3] = ~0u;
        }
        if constexpr (SCALED) {
            FourRaw f[S / 8];
#pragma unroll
            for (int i = 0; i < S / 8; ++i) f[i] = q0 + 8 * i + sl < cnt ? factors[lo + q0 + 8 * i + sl] : FourRaw{0u, 0u, 0u, 0u};
            wave_lds_sync();
#pragma unroll
            for (int i = 0; i < S / 8; ++i) s_w[g][8 * i + sl] = f[i];
        } else {
            wave_lds_sync();
        }
#pragma unroll
        for (int i = 0; i < S / 16; ++i) s_stage[g][8 * i + sl] = e[i];
        wave_lds_sync();
#pragma unroll 1
        for (int q = q0; q < per && q < q0 + S; q += 8) {
            const int left = cnt - q < 8 ? cnt - q : 8;
            uint32_t stores = 0;
            if (left > 0) {
                stores = (uint32_t)(last >> (q - q0)) & ((1u << left) - 1u);
                open = ((stores >> (left - 1)) & 1u) == 0u;
            }
            const FourRaw* const st = &s_stage[g][(q - q0) / 2];
            const FourRaw* const wt = SCALED ? &s_w[SCALED ? g : 0][SCALED ? q - q0 : 0] : nullptr;
            auto done = [&](int j) {
                if ((stores >> j) & 1u) {
                    if (cut) head();
                    else if (col_ok) store(row);
                    ++row;
#pragma unroll
                    for (int k = 0; k < VE; ++k) s[k] = 0.f;
                }
            };
            FourLoads<SCALED> x, y;
            four_load(rows, lane_off, st[0][0], st[0][1], wt + 0, x);
            four_load(rows, lane_off, st[0][2], st[0][3], wt + 1, y);
            four_add(s, x); done(0);
            four_load(rows, lane_off, st[1][0], st[1][1], wt + 2, x);
            four_add(s, y); done(1);
            four_load(rows, lane_off, st[1][2], st[1][3], wt + 3, y);
            four_add(s, x); done(2);
            four_load(rows, lane_off, st[2][0], st[2][1], wt + 4, x);
            four_add(s, y); done(3);
            four_load(rows, lane_off, st[2][2], st[2][3], wt + 5, y);
            four_add(s, x); done(4);
            four_load(rows, lane_off, st[3][0], st[3][1], wt + 6, x);
            four_add(s, y); done(5);
            four_load(rows, lane_off, st[3][2], st[3][3], wt + 7, y);
            four_add(s, x); done(6);
            four_add(s, y); done(7);
        }
    }
    if (open && cut) {            // the whole stretch lies inside a row
        head();
        open = false;
    }
    if (sl == 0) s_head_row[g] = head_row;
    __syncthreads();
    if (open) {                   // the row goes on in the stretches behind
        for (int h = g + 1; h < kFourGroups && s_head_row[h] == row; ++h)
#pragma unroll
            for (int k = 0; k < VE; ++k) s[k] += s_head[h][sl * VE + k];
        if (col_ok) store(row);
    }
}

}  // namespace gnnhot
