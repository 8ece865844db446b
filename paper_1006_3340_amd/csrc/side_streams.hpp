// side_streams.hpp -- launches beside the caller's stream (host code only).
#pragma once

#include <hip/hip_runtime_api.h>

namespace lll {

constexpr int kSideStreams = 3;  // with the caller's stream, the device's four queues
struct SideStreams {             // default priority
    hipStream_t side[kSideStreams] = {};
    hipEvent_t fork = nullptr, join[kSideStreams] = {};
};

// launch(i, stream) for i = 0 .. n - 1 round the caller's stream st and the side streams:
// these start after what st holds now, and st goes on after all of them.  So too after a
// launch that failed: what was queued before it still uses the plan's buffers, and the
// caller's next pass on st must find them free.
template <typename F>
hipError_t run_beside(const SideStreams &ss, hipStream_t st, int n, F &&launch) {
    hipError_t e = hipEventRecord(ss.fork, st);
    int forked = 0;
    while (e == hipSuccess && forked < kSideStreams)
        if ((e = hipStreamWaitEvent(ss.side[forked], ss.fork, 0)) == hipSuccess) ++forked;
    for (int i = 0; i < n && e == hipSuccess; ++i) {
        const int s = i % (kSideStreams + 1);
        e = launch(i, s == 0 ? st : ss.side[s - 1]);
    }
    for (int i = 0; i < forked; ++i) {
        hipError_t j = hipEventRecord(ss.join[i], ss.side[i]);
        if (j == hipSuccess) j = hipStreamWaitEvent(st, ss.join[i], 0);
        if (j != hipSuccess) (void)hipStreamSynchronize(ss.side[i]);  // wait here instead
        if (e == hipSuccess) e = j;
    }
    return e;
}

}  // namespace lll
