// Row kernel for short rows of a graph far larger than the caches (included by spmm.hip, which defines SpmmArgs and Elem).
//
// The general row kernel gives a row of up to 512 bytes to 16 or 32 lanes, tile by tile: between two rows of a group its loads
// drain, and with rows of 5 to 20 entries a group is between rows half of its time.  Here a whole wavefront spans the row
// (4 or 8 bytes a lane) and walks its eight rows as ONE stream of entries with U loads in flight throughout: what is
// uniform - the neighbour, the end of a row - is in scalar registers, a load takes its row's offset as a scalar operand, and
// the end of a row is a scalar branch that stores and goes on.  The small loads cost vector-cache time, which only a graph
// out of the fabric has to spare.
// Measured (bf16, 128 columns, us, before / after): 810 k rows of 24 643 / 603, 720 k of 8 352 / 269, 2.1 M of 10 1038 / 842;
// fp32, 64 columns: 720 k of 8 326 / 262.  Rounds of 8 loads at 4 bytes a lane 618 (of 16 590), 16 or 32 rows a
// wavefront 605 / 670, rows shared by the workgroup from 64 / 128 / 512 entries on 620 / 606 / 613.
#pragma once
#include "common.h"

namespace gnnhot {

constexpr int kWaveRows = 32;          // rows of the list per wavefront at most
// Rows of more entries are shared by the workgroup's wavefronts.  A row below is one chain of additions: in fp32 no longer
// than a row of one lane group's in the general kernel, in bf16, where the rounding of the result is what counts, longer.
template <int DT>
constexpr int kWaveHub = DT == GNN_F32 ? 64 : 256;

template <int BPL>
struct WaveRaw;
template <> struct WaveRaw<4> { using T = uint32_t; };
template <> struct WaveRaw<8> { typedef uint32_t T __attribute__((ext_vector_type(2))); };

// A row (index `row`, `bytes` bytes a row) of a matrix, BPL bytes a lane.  OFF32: the matrix spans less than 4 GB, the row's offset is
// a scalar operand of the load and no address is computed.
template <int BPL, bool OFF32>
__device__ __forceinline__ typename WaveRaw<BPL>::T wave_load(const void* base, uint32_t row, int64_t bytes, uint32_t lane_off) {
    if constexpr (OFF32) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00020000);
        const int off = (int)(row * (uint32_t)bytes);
        if constexpr (BPL == 4) return __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, off, 0);
        if constexpr (BPL == 8) return __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, off, 0);
    } else {
        return *(const typename WaveRaw<BPL>::T*)((const char*)base + (int64_t)row * bytes + lane_off);
    }
}

template <int DT, int BPL>
__device__ __forceinline__ void wave_unpack(const typename WaveRaw<BPL>::T& r, float (&v)[BPL / (DT == GNN_F32 ? 4 : 2)]) {
#pragma unroll
    for (int i = 0; i < BPL / 4; ++i) {
        uint32_t x;
        if constexpr (BPL == 4) x = r;
        else x = r[i];
        if constexpr (DT == GNN_F32) {
            v[i] = __uint_as_float(x);
        } else {
            v[2 * i] = bf16lo(x);
            v[2 * i + 1] = bf16hi(x);
        }
    }
}

template <int DT, int BPL, int U, bool OFF32, bool SCALED>
__global__ __launch_bounds__(256, BPL == 4 ? 8 : 7) void spmm_wave_kernel(SpmmArgs a) {
    constexpr int ES = DT == GNN_F32 ? 4 : 2, VE = BPL / ES, W = 64 * VE;
    using Raw = typename WaveRaw<BPL>::T;
    static_assert(64 % U == 0, "whole rounds");
    __shared__ int32_t s_hub[4 * kWaveRows], s_hub_s[4 * kWaveRows], s_hub_n[4 * kWaveRows];
    __shared__ float s_hub_sc[4 * kWaveRows];
    __shared__ int s_hubs[4];
    __shared__ float s_red[4][W];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int R = a.rows_per_group;
    const int64_t base = ((int64_t)blockIdx.x * 4 + wave) * R;
    const int col = lane * VE;
    const bool col_ok = col < a.F;
    const uint32_t lane_off = col_ok ? (uint32_t)(lane * BPL) : 0u;
    const int64_t xb = a.ldx * ES;

    // ---- the wavefront's rows, one per lane
    int32_t v = 0, s = 0, len = 0;
    float sc = 1.f;
    bool hub = false;
    const bool mine = lane < R && base + lane < a.n_active;
    if (mine) {
        v = a.rows ? a.rows[base + lane] : (int32_t)(base + lane);
        s = a.row_ptr[v];
        int32_t e = a.row_ptr[v + 1];
        if (a.cut_id >= 0) e = row_lower_bound(a.col_idx, s, e, a.cut_id);
        len = e - s;
        sc = a.out_scale ? a.out_scale[v] : 1.f;
        hub = len > kWaveHub<DT>;
    }
    const uint64_t hubs = __ballot(hub);
    if (hub) {
        const int k = wave * kWaveRows + __popcll(hubs & ((1ull << lane) - 1ull));
        s_hub[k] = v; s_hub_s[k] = s; s_hub_n[k] = len; s_hub_sc[k] = sc;
    }
    if (lane == 0) s_hubs[wave] = __popcll(hubs);
    int items = mine && !hub ? len : 0;
    uint64_t none = __ballot(mine && !hub && items == 0);
    int end = wave_inclusive_scan(items), start = end - items;
    int T = __builtin_amdgcn_readlane(end, 63);

    float acc[VE];
#pragma unroll
    for (int k = 0; k < VE; ++k) acc[k] = 0.f;
    auto store = [&](int32_t row, const float (&o)[VE]) {
        if (!col_ok) return;
        char* q = (char*)a.Y + (int64_t)row * (a.ldy * ES) + lane * BPL;
        if (a.F - col >= VE) {
            Raw r;
#pragma unroll
            for (int i = 0; i < BPL / 4; ++i) {
                uint32_t x;
                if constexpr (DT == GNN_F32) x = __float_as_uint(o[i]);
                else x = pack_bf16(o[2 * i], o[2 * i + 1]);
                if constexpr (BPL == 4) r = x;
                else r[i] = x;
            }
            *(Raw*)q = r;
        } else {
#pragma unroll
            for (int k = 0; k < VE; ++k) {
                if (k < a.F - col) {
                    if constexpr (DT == GNN_F32) ((float*)q)[k] = o[k];
                    else ((uint16_t*)q)[k] = f32_to_bf16(o[k]);
                }
            }
        }
    };
    int hub_row = -1;              // >= 0: the stream is this wavefront's quarter of a long row, summed 64 entries at a time
    // The rows' entries as one stream, 64 at a time, a lane an entry: its neighbour, and of which lane's row it is (| 0x80: the
    // last of that row).
    struct Items { uint32_t nbr; uint32_t slot; };
    auto fetch = [&](int t0) -> Items {
        const int t = t0 + lane < T ? t0 + lane : T - 1;
        int lo = 0;
#pragma unroll
        for (int d = kWaveRows / 2; d > 0; d >>= 1)
            if (__shfl(end, lo + d - 1, kWave) <= t) lo += d;
        const int row_start = __shfl(start, lo, kWave), row_end = __shfl(end, lo, kWave), first = __shfl(s, lo, kWave);   // (by all lanes)
        Items it;
        it.slot = (uint32_t)lo | (t0 + lane < T && (t + 1 == row_end || (hub_row >= 0 && lane == 63)) ? 0x80u : 0u);
        it.nbr = (uint32_t)a.col_idx[first + (t - row_start)];
        return it;
    };
    auto issue = [&](uint32_t nbr) { return wave_load<BPL, OFF32>(a.X, nbr, xb, lane_off); };
    for (int q = -1;;) {
        if (T > 0) {
            Items cur = fetch(0);
            float w_c = 1.f, w_n = 1.f;
            if constexpr (SCALED) { w_c = a.nbr_scale[cur.nbr]; }
            Items nxt = fetch(64);
            Raw x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = issue(__builtin_amdgcn_readlane(cur.nbr, u));
            int t0 = 0;
            do {
                if constexpr (SCALED) { w_n = a.nbr_scale[nxt.nbr]; }
                const Items after = fetch(t0 + 128);
                const uint64_t last = __ballot((cur.slot & 0x80u) != 0);
                const int stop = T - t0 < 64 ? T - t0 : 64;
#pragma unroll 1
                for (int j0 = 0, more = 1; more != 0; j0 += U) {     // at least once: what was fetched before is then known to be older than U loads
                    more = j0 + U < stop;
                    const bool wrap = j0 + U == 64;
                    const uint32_t nbr_s = wrap ? nxt.nbr : cur.nbr;
                    const int js = (j0 + U) & 63;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        float t[VE];
                        wave_unpack<DT, BPL>(x[u], t);
                        const float w = SCALED ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w_c), j0 + u)) : 1.f;
#pragma unroll
                        for (int k = 0; k < VE; ++k) acc[k] = SCALED ? fmaf(w, t[k], acc[k]) : acc[k] + t[k];
                        if ((last >> (j0 + u)) & 1ull) {      // uniform
                            if (hub_row >= 0) {
#pragma unroll
                                for (int k = 0; k < VE; ++k) s_red[wave][col + k] += acc[k];
                            } else {
                                const int slot = __builtin_amdgcn_readlane((int)cur.slot, j0 + u) & 0x7f;
                                const float scale = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sc), slot));
                                float o[VE];
#pragma unroll
                                for (int k = 0; k < VE; ++k) o[k] = acc[k] * scale;
                                store(__builtin_amdgcn_readlane(v, slot), o);
                            }
#pragma unroll
                            for (int k = 0; k < VE; ++k) acc[k] = 0.f;
                        }
                        x[u] = issue(__builtin_amdgcn_readlane(nbr_s, js + u));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                cur = nxt; nxt = after; w_c = w_n;
#pragma unroll
                for (int k = 0; k < VE; ++k) acc[k] = t0 + 64 < T ? acc[k] : 0.f;      // (items past the end)
                t0 += 64;
            } while (t0 < T);
        }
        __syncthreads();
        if (hub_row >= 0) {
            const float scale = s_hub_sc[q];
            for (int c = (int)threadIdx.x; c < W; c += 256) {
                if (c < a.F) {
                    float o[1] = {((s_red[0][c] + s_red[1][c]) + (s_red[2][c] + s_red[3][c])) * scale};
                    Elem<DT, 1>::store(a.Y, (int64_t)hub_row * a.ldy + c, o, 1, false);
                }
            }
            __syncthreads();
        }
        // ---- the next long row of the workgroup: a quarter of its entries, in whole batches
        ++q;
        while (q < 4 * kWaveRows && (q & (kWaveRows - 1)) >= s_hubs[q / kWaveRows]) q = (q | (kWaveRows - 1)) + 1;
        if (q >= 4 * kWaveRows) break;
        hub_row = s_hub[q];
        const int n = s_hub_n[q], per = (n + 255) / 256 * 64;
        s = s_hub_s[q] + wave * per;
        len = n - wave * per < per ? n - wave * per : per;
        if (len < 0) len = 0;
#pragma unroll
        for (int k = 0; k < VE; ++k) s_red[wave][col + k] = 0.f;
        T = end = len;
        start = 0;
    }
    // ---- rows without any item are zero
    while (none != 0) {
        const int l = __builtin_ctzll(none);
        none &= none - 1;
        float o[VE];
#pragma unroll
        for (int k = 0; k < VE; ++k) o[k] = 0.f;
        store(a.rows ? a.rows[base + l] : (int32_t)(base + l), o);
    }
}

// Where the line lies (us, general / this kernel, rows of the call; bf16 128 columns, fp32 64): rows of 20: 1.3 M 1009 / 908 and 957 /
// 935, 560 k 389 / 355 and 368 / 341, 240 k 190 / 193 and 176 / 184; of 12: 240 k 138 / 120 and 122 / 116; of 6: 960 k 442 / 305 and
// 410 / 302, 200 k 98 / 85 and 87 / 83, 107 k 57 / 63 and 50 / 56; of 35: 1.5 M 1607 / 1628 and 1572 / 1634.  8 bytes a lane
// (bf16 256 columns, fp32 128): rows of 8 640 / 539 and 605 / 527, of 20 748 / 728 and 718 / 732.  Rows of 128 bytes or less leave half of
// the lanes idle, rows of 1 KB are not slower in the general kernel.
static bool wave_rows_apply(const gnn_csr* g, int32_t n_active, int32_t F, int32_t dtype, bool vec_ok, bool filter, bool plain_store) {
    const int64_t avg = g->nnz / (g->n_rows > 0 ? g->n_rows : 1), bytes = (int64_t)F * (dtype == GNN_F32 ? 4 : 2);
    return vec_ok && !filter && plain_store && bytes > 128 && bytes <= 512 && avg <= (bytes <= 256 ? 24 : 16) &&
           n_active >= 25000 * (avg < 4 ? 4 : avg);
}

template <int DT, int BPL, int U>
static int32_t launch_wave(const SpmmArgs& a, hipStream_t stream) {
    SpmmArgs b = a;
    b.rows_per_group = 8;
    const unsigned grid = (unsigned)(((int64_t)a.n_active + 4 * b.rows_per_group - 1) / (4 * b.rows_per_group));
    if (a.x_row_bytes != 0) {      // less than 4 GB
        if (a.nbr_scale) spmm_wave_kernel<DT, BPL, U, true, true><<<grid, 256, 0, stream>>>(b);
        else spmm_wave_kernel<DT, BPL, U, true, false><<<grid, 256, 0, stream>>>(b);
    } else {
        if (a.nbr_scale) spmm_wave_kernel<DT, BPL, U, false, true><<<grid, 256, 0, stream>>>(b);
        else spmm_wave_kernel<DT, BPL, U, false, false><<<grid, 256, 0, stream>>>(b);
    }
    GNN_LAUNCH_CHECK("spmm_wave_kernel");
    return GNN_OK;
}

template <int DT>
static int32_t launch_wave_rows(const SpmmArgs& a, hipStream_t stream) {
    return a.F * (DT == GNN_F32 ? 4 : 2) <= 256 ? launch_wave<DT, 4, 16>(a, stream) : launch_wave<DT, 8, 8>(a, stream);
}

}  // namespace gnnhot
