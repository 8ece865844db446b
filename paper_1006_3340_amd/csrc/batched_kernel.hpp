// batched_kernel.hpp -- the persistent kernel of one register bucket.
//
// Work items are (structure, block of 256 paths) of the structures whose rates
// fit the bucket NMAX, structure by structure; a grid sized to the kernel's resident capacity pulls
// items from a device counter until none are left.  Each structure keeps its
// own precompute tables (laid out for its bucket) behind a per-structure
// argument block.  Instantiated per bucket in batched_b*.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "lll_device.hpp"
#include "lll_internal.hpp"
#include "path_kernel.hpp"

namespace lll {
namespace batch {

using detail::cptr;
using detail::PathArgs;

// The structures of a bucket in the order of their items, and what a pass sets.
struct BatchWork {
    cptr<int> order;
    int n_items, blocks_each;
    int64_t n_paths;
    uint32_t key0, key1;
};

// Copy of a trivially copyable struct read word by word through the constant
// address space (uniform address: scalar loads).
template <typename T>
__device__ __forceinline__ T load_uniform(cptr<T> p) {
    static_assert(sizeof(T) % 4 == 0, "word-sized struct");
    T v;
    const cptr<uint32_t> w = (cptr<uint32_t>)(p);
    uint32_t *d = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
    for (int i = 0; i < static_cast<int>(sizeof(T) / 4); ++i) d[i] = w[i];
    return v;
}

template <int NMAX, int SCHEME>
__global__ void __launch_bounds__(kBlock) batched_kernel(cptr<PathArgs<float>> args,
                                                         BatchWork work,
                                                         int *__restrict__ counter) {
    // The block shares one item (its four wavefronts then stream the same
    // step tables through the CU's scalar cache).  With the state in LDS the
    // item index travels through the first word of that array, which no
    // simulation touches between the two barriers (so the block's LDS stays
    // at the state's size).
    int *slot;
    if constexpr (detail::kStateInLds<float, NMAX, SCHEME>) {
        slot = reinterpret_cast<int *>(detail::state_lds<float, NMAX>());
    } else {
        __shared__ int s_item;
        slot = &s_item;
    }
    for (;;) {
        if (threadIdx.x == 0) *slot = atomicAdd(counter, 1);
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(*slot);
        __syncthreads();
        if (item >= work.n_items) return;  // same value in every lane of the block
        const int at = item / work.blocks_each;
        PathArgs<float> a = load_uniform<PathArgs<float>>(args + work.order[at]);
        a.n_paths = work.n_paths;
        a.key0 = work.key0;
        a.key1 = work.key1;
        const int64_t gid =
            static_cast<int64_t>(item - at * work.blocks_each) * kBlock + threadIdx.x;
        const int64_t wave_first = gid - (threadIdx.x % kWave);
        if (wave_first < a.n_paths)
            detail::simulate<float, NMAX, SCHEME, true, detail::kAnyProduct>(a, gid);
    }
}

template <int NMAX, int SCHEME>
hipError_t launch_bucket_t(cptr<PathArgs<float>> args, const BatchWork &work, int *counter,
                           hipStream_t st) {
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batched_kernel<NMAX, SCHEME>,
                                                         kBlock, 0);
    if (e != hipSuccess) return e;
    const int grid = std::max(1, std::min(cus * std::max(per_cu, 1), work.n_items));
    hipLaunchKernelGGL((batched_kernel<NMAX, SCHEME>), dim3(grid), dim3(kBlock), 0, st, args,
                       work, counter);
    return hipGetLastError();
}

// The persistent launch of one bucket (the counter starts at zero).
template <int NMAX>
hipError_t launch_bucket(int scheme, cptr<PathArgs<float>> args, const BatchWork &work,
                         int *counter, hipStream_t st) {
    switch (scheme) {
        case kFull: return launch_bucket_t<NMAX, kFull>(args, work, counter, st);
        case kPicard: return launch_bucket_t<NMAX, kPicard>(args, work, counter, st);
        default: return launch_bucket_t<NMAX, kFrozen>(args, work, counter, st);
    }
}

#define LLL_BATCH_BUCKET_DECL(EXT, NMAX)                                                          \
    EXT template hipError_t launch_bucket<NMAX>(int, cptr<PathArgs<float>>, const BatchWork &,    \
                                                int *, hipStream_t);
#ifndef LLL_BATCH_BUCKET_TU
LLL_BATCH_BUCKET_DECL(extern, 8)
LLL_BATCH_BUCKET_DECL(extern, 16)
LLL_BATCH_BUCKET_DECL(extern, 24)
LLL_BATCH_BUCKET_DECL(extern, 32)
LLL_BATCH_BUCKET_DECL(extern, 40)
#endif

}  // namespace batch
}  // namespace lll
