// Row-length classes of the kernels that walk whole CSR rows: rows of up to kRowShort entries stay with the sixteen lanes
// that found them, rows of up to kRowMedium are left to a launch with a wavefront per row, longer ones to a launch with a
// workgroup per row.  (On power-law graphs a few per cent of the rows hold most of the entries; sixteen lanes that walk
// a row of 10 000 entries keep their launch alive long after every other row is done.)  The rows that a workgroup
// leaves are collected in LDS lists and appended to the two queues with ONE global atomic per workgroup and class: one
// atomic per row on a single counter serialised such a launch (184 000 of them took 1.4 ms).  The order of a queue depends
// on timing, so what is done with a row must depend on the row alone.
#pragma once
#include "common.h"

namespace gnnhot {

constexpr int kRowLanes = 16;                  // lanes per short row
constexpr int kRowShort = 4 * kRowLanes;       // rows up to this length stay with their sixteen lanes
constexpr int kRowMedium = 16 * kWave;         // rows up to this length get a wavefront, longer ones a workgroup
constexpr int kRowsPerWg = 256 / kRowLanes;    // rows one workgroup of 256 threads takes per step
constexpr int kRowListCap = 1024;              // entries of a workgroup's LDS list per class; what does not fit goes out one by one

struct RowCtrl {
    int32_t n_medium;
    int32_t n_hub;
    int32_t pad[6];
};

struct RowLists {
    int32_t med[kRowListCap], hub[kRowListCap];
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
        if (pos < kRowListCap) L.hub[pos] = i;
        else hubq[atomicAdd(&ctrl->n_hub, 1)] = i;
    }
}

// every thread of the workgroup calls this once, after its last push
__device__ __forceinline__ void row_lists_flush(RowLists& L, int32_t* __restrict__ medq, int32_t* __restrict__ hubq, RowCtrl* ctrl) {
    __syncthreads();
    const int nm = L.n_med < kRowListCap ? L.n_med : kRowListCap, nh = L.n_hub < kRowListCap ? L.n_hub : kRowListCap;
    if (threadIdx.x == 0) {
        L.base_med = nm ? atomicAdd(&ctrl->n_medium, nm) : 0;
        L.base_hub = nh ? atomicAdd(&ctrl->n_hub, nh) : 0;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nm; k += blockDim.x) medq[L.base_med + k] = L.med[k];
    for (int k = threadIdx.x; k < nh; k += blockDim.x) hubq[L.base_hub + k] = L.hub[k];
}

// the 16 bits of a ballot that belong to lane group `sub` of the wavefront
__device__ __forceinline__ uint32_t group_ballot(bool p, int sub) {
    return (uint32_t)((__ballot(p) >> (sub * kRowLanes)) & 0xffffu);
}

}  // namespace gnnhot
