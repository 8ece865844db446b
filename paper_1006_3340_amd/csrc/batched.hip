// batched.hip -- many independent term structures, one persistent launch per
// register bucket.
//
// Every structure is planned in the smallest bucket that holds its rates (8,
// 16, 24, 32 or 40 slots), so its path kernel runs at that bucket's register
// and LDS footprint.  Work items are (structure, block of 256 paths), the
// structures of a bucket by decreasing cost (N^2 s per path);
// each bucket's persistent kernel pulls its items from its own device counter.
// The buckets' launches run concurrently on the batch's side streams (forked
// from and joined back into the caller's stream), so a bucket that runs out
// of items leaves its compute units to the others instead of idling them.  The
// argument blocks and the order go to the device with the first pass; set-up and
// reduction of all structures are one launch each kernel.  64 structures of 2^18
// paths take 114.5 ms a pass, 105 of them the longest bucket's kernel; with 320
// set-up and reduction launches and an item list sorted and uploaded per pass
// they took over 140.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "batched_kernel.hpp"
#include "lll_internal.hpp"

namespace lll {

using batch::BatchWork;
using detail::PathArgs;

namespace {

constexpr int kBuckets[kBatchBuckets] = {40, 32, 24, 16, 8};

int bucket_index(int nmax) {
    for (int b = 0; b < kBatchBuckets; ++b)
        if (kBuckets[b] == nmax) return b;
    return -1;
}

hipError_t launch_one(int nmax, int scheme, detail::cptr<PathArgs<float>> args,
                      const BatchWork &w, int *counter, hipStream_t st) {
    switch (nmax) {
        case 8: return batch::launch_bucket<8>(scheme, args, w, counter, st);
        case 16: return batch::launch_bucket<16>(scheme, args, w, counter, st);
        case 24: return batch::launch_bucket<24>(scheme, args, w, counter, st);
        case 32: return batch::launch_bucket<32>(scheme, args, w, counter, st);
        case 40: return batch::launch_bucket<40>(scheme, args, w, counter, st);
        default: return hipErrorInvalidValue;
    }
}

__global__ void zero_counters_kernel(int *counter) {
    if (threadIdx.x < kBatchBuckets) counter[64 * threadIdx.x] = 0;
}

const PassArgs *batch_pass_args(const lll_batch &b) {
    return reinterpret_cast<const PassArgs *>(static_cast<const PathArgs<float> *>(b.args) +
                                              b.plans.size());
}

}  // namespace

size_t batch_item_bytes() { return sizeof(int); }
size_t batch_args_bytes() { return sizeof(PathArgs<float>) + sizeof(PassArgs); }

// Argument blocks and order of the structures (largest bucket first, decreasing
// cost inside a bucket) on the device, once; then the set-up of all structures.
hipError_t batch_prepare(lll_batch &b, int64_t n_paths_each, uint64_t seed, hipStream_t st) {
    const size_t n = b.plans.size();
    int max_N = 0, max_K = 0;
    for (const lll_plan *p : b.plans) {
        max_N = std::max(max_N, p->N);
        max_K = std::max(max_K, p->K);
    }
    if (!b.laid_out) {
        std::vector<PathArgs<float>> args(n);
        std::vector<PassArgs> pass(n);
        std::vector<int> order(n);
        for (size_t i = 0; i < n; ++i) {
            args[i] = detail::make_args<float>(*b.plans[i], 0, 0, 0, nullptr);
            pass[i] = pass_args(*b.plans[i]);
            order[i] = static_cast<int>(i);
            if (bucket_index(b.plans[i]->nmax) < 0) return hipErrorInvalidValue;
        }
        std::stable_sort(order.begin(), order.end(), [&](int i, int j) {
            const lll_plan &px = *b.plans[i], &py = *b.plans[j];
            const int bx = bucket_index(px.nmax), by = bucket_index(py.nmax);
            if (bx != by) return bx < by;
            return (int64_t)px.N * px.N * px.s > (int64_t)py.N * py.N * py.s;
        });
        for (int k = 0; k < kBatchBuckets; ++k) b.bucket_begin[k] = b.bucket_end[k] = 0;
        for (size_t i = 0; i < n; ++i) {
            const int k = bucket_index(b.plans[order[i]]->nmax);
            if (b.bucket_end[k] == 0) b.bucket_begin[k] = static_cast<int>(i);
            b.bucket_end[k] = static_cast<int>(i) + 1;
        }
        hipError_t e = hipMemcpyAsync(b.args, args.data(), n * sizeof(PathArgs<float>),
                                      hipMemcpyHostToDevice, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(const_cast<PassArgs *>(batch_pass_args(b)), pass.data(),
                               n * sizeof(PassArgs), hipMemcpyHostToDevice, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(b.items, order.data(), n * sizeof(int), hipMemcpyHostToDevice, st);
        // the host vectors die at return: make the copies complete first
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        b.laid_out = true;
    }
    b.pass_paths = n_paths_each;
    b.pass_seed = seed;
    return launch_precompute_batch(batch_pass_args(b), static_cast<int>(n), max_N, max_K, st);
}

// One persistent launch per bucket present: the largest on the caller's
// stream, the others on side streams that wait for the caller's stream and
// that the caller's stream waits for in turn; then the reductions (outside the
// timed launch).
hipError_t launch_batched(const lll_batch &b, int scheme, hipStream_t st) {
    const auto args = detail::as_const(static_cast<const PathArgs<float> *>(b.args));
    const int blocks = static_cast<int>((b.pass_paths + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, st, b.counter);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipEventRecord(b.fork, st);
    bool first = true;
    for (int k = 0; k < kBatchBuckets && e == hipSuccess; ++k) {
        const int n = b.bucket_end[k] - b.bucket_begin[k];
        if (n <= 0) continue;
        hipStream_t s = first ? st : b.side[k];
        if (!first) e = hipStreamWaitEvent(s, b.fork, 0);
        BatchWork w;
        w.order = detail::as_const(static_cast<const int *>(b.items) + b.bucket_begin[k]);
        w.n_items = n * blocks;
        w.blocks_each = blocks;
        w.n_paths = b.pass_paths;
        w.key0 = static_cast<uint32_t>(b.pass_seed & 0xFFFFFFFFull);
        w.key1 = static_cast<uint32_t>(b.pass_seed >> 32);
        if (e == hipSuccess)
            e = launch_one(kBuckets[k], scheme, args, w, b.counter + 64 * k, s);
        if (e == hipSuccess && !first) e = hipEventRecord(b.join[k], s);
        if (e == hipSuccess && !first) e = hipStreamWaitEvent(st, b.join[k], 0);
        first = false;
    }
    if (e == hipSuccess && b.timing) e = hipEventRecord(b.ev[1], st);
    if (e == hipSuccess)
        e = launch_reduce_batch(batch_pass_args(b), static_cast<int>(b.plans.size()), b.pass_paths,
                                st);
    return e;
}

}  // namespace lll
