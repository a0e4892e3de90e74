// Row-length classes of the kernels that walk whole CSR rows: rows of up to kRowShort entries stay with the sixteen lanes
// that found them, rows of up to kRowMedium are left to a launch with a wavefront per row, longer ones to a launch with a
// workgroup per row.  (On power-law graphs a few per cent of the rows hold most of the entries; sixteen lanes that walk
// a row of 10 000 entries keep their launch alive long after every other row is done.)  The rows that a workgroup
// leaves are collected in LDS lists and appended to the two queues with ONE global atomic per workgroup: one
// atomic per row on a single counter serialised such a launch (184 000 of them took 1.4 ms).  The order of a queue depends
// on timing, so what is done with a row must depend on the row alone.
#pragma once
#include "common.h"

namespace gnnhot {

constexpr int kRowLanes = 16;                  // lanes per short row
constexpr int kRowShort = 4 * kRowLanes;       // rows up to this length stay with their sixteen lanes
constexpr int kRowMedium = 16 * kWave;         // rows up to this length get a wavefront, longer ones a workgroup
constexpr int kRowsPerWg = 256 / kRowLanes;    // rows one workgroup of 256 threads takes per step
// Workgroups of a launch that fills the queues: what the chip holds at a time.  Each ends with an atomic on one address, some 9 ns one
// after the other (ex_fill_kernel of 1 M rows, 20 M entries, us: 4096 workgroups with an atomic a class 243, with one for both
// 215, 2048 140; 1024 are too few: 3 M vertices of degree 10, three rings, the whole extraction 1311 / 1238 / 1430).
constexpr int kRowGrid = 2048;
// Entries of a workgroup's LDS list of medium rows; what does not fit goes out one by one, on one address: 3 M rows of 100, lists of 1024 /
// 2048, sampling 25.1 / 4.7 ms, extraction 27.1 / 6.7.  Of rows above kRowMedium a graph of 2^31 entries has 2 M at most, 1024 a workgroup.
constexpr int kRowListCap = 2048, kHubListCap = 1024;

// Workgroups of a launch over n rows of nnz entries that takes rows_a_step of them at a time: at_least, fewer for few rows, more where the
// lists (to 7/8, the rows are dealt in turn) would not hold the medium rows there can be.  5 M rows of 100, sampling 25.9 -> 7.7 ms, extraction 30.3 -> 12.2;
// of 15, none more: with 2442 workgroups for its 1.1 M the extraction would take 2.13 ms instead of 1.84.
inline int queue_grid(int64_t n, int64_t nnz, int rows_a_step, int at_least = kRowGrid) {
    const int64_t queued = nnz / (kRowShort + 1) < n ? nnz / (kRowShort + 1) : n;
    const int64_t full = (queued + kRowListCap / 8 * 7 - 1) / (kRowListCap / 8 * 7);
    return grid_for(n, rows_a_step, full > at_least ? (int)full : at_least);
}

struct __attribute__((aligned(8))) RowCtrl {
    int32_t n_medium;        // the first two as one 64-bit word: row_lists_flush
    int32_t n_hub;
    int32_t pad[6];
};

struct RowLists {
    int32_t med[kRowListCap], hub[kHubListCap];
    int32_t n_med, n_hub, base_med, base_hub;
};

__device__ __forceinline__ void row_lists_init(RowLists& L) {
    if (threadIdx.x == 0) L.n_med = L.n_hub = 0;
    __syncthreads();
}

// one lane per row calls this
__device__ __forceinline__ void row_lists_push(RowLists& L, int32_t i, int32_t len, int32_t* __restrict__ medq, int32_t* __restrict__ hubq,
                                               RowCtrl* ctrl) {
    if (len <= kRowMedium) {
        const int pos = atomicAdd(&L.n_med, 1);
        if (pos < kRowListCap) L.med[pos] = i;
        else medq[atomicAdd(&ctrl->n_medium, 1)] = i;
    } else {
        const int pos = atomicAdd(&L.n_hub, 1);
        if (pos < kHubListCap) L.hub[pos] = i;
        else hubq[atomicAdd(&ctrl->n_hub, 1)] = i;
    }
}

// every thread of the workgroup calls this once, after its last push
__device__ __forceinline__ void row_lists_flush(RowLists& L, int32_t* __restrict__ medq, int32_t* __restrict__ hubq, RowCtrl* ctrl) {
    __syncthreads();
    const int nm = L.n_med < kRowListCap ? L.n_med : kRowListCap, nh = L.n_hub < kHubListCap ? L.n_hub : kHubListCap;
    if (threadIdx.x == 0 && nm + nh > 0) {      // both counters at once: one atomic on one address
        const unsigned long long base = atomicAdd((unsigned long long*)ctrl, (unsigned long long)(uint32_t)nh << 32 | (uint32_t)nm);
        L.base_med = (int32_t)(uint32_t)base;
        L.base_hub = (int32_t)(uint32_t)(base >> 32);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nm; k += blockDim.x) medq[L.base_med + k] = L.med[k];
    for (int k = threadIdx.x; k < nh; k += blockDim.x) hubq[L.base_hub + k] = L.hub[k];
}

// The rows i, i + step, .. of a list, with their bounds fetched ahead: four dependent loads lie between a place of the list and the
// first probe of a row's entries (id, bounds, entries, probe), and short rows are nothing but these.  While a row is worked on, the
// next one's bounds and the id of the one after that are on their way.
struct RowWalk {
    const int32_t* ids;        // vertex of a place of the list
    const int32_t* rp;
    int32_t n;                 // vertices: ids outside have no entries
    int64_t n_rows, step;      // places
    int32_t v, s, e;           // the row in hand
    int32_t v_next, s_next, e_next;

    __device__ __forceinline__ int32_t id(int64_t i) const { return i < n_rows ? ids[i] : -1; }
    __device__ __forceinline__ void bounds(int32_t u, int32_t& from, int32_t& to) const {
        const bool in = u >= 0 && u < n;
        from = rp[in ? u : 0];
        to = rp[in ? u + 1 : 0];
    }
    __device__ __forceinline__ void begin(int64_t i) {
        v = id(i);
        v_next = id(i + step);
        bounds(v, s, e);
    }
    // called with the row at place i in hand, before its entries are asked for
    __device__ __forceinline__ int32_t ahead(int64_t i) {
        bounds(v_next, s_next, e_next);
        return id(i + 2 * step);
    }
    __device__ __forceinline__ void next(int32_t v_after) {
        v = v_next;
        s = s_next;
        e = e_next;
        v_next = v_after;
    }
};

// the 16 bits of a ballot that belong to lane group `sub` of the wavefront
__device__ __forceinline__ uint32_t group_ballot(bool p, int sub) {
    return (uint32_t)((__ballot(p) >> (sub * kRowLanes)) & 0xffffu);
}

}  // namespace gnnhot
