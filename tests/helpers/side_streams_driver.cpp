// run_beside (side_streams.hpp) on stand-ins of the HIP calls: which stream waits for what
// when a launch or one of the calls fails.  Prints "ok" and exits 0.
#include <cstdio>
#include <cstdint>
#include <map>
#include <vector>

#include "side_streams.hpp"

namespace {

std::map<hipStream_t, std::vector<int>> queued;   // launches of each stream
std::map<hipEvent_t, std::vector<int>> recorded;  // launches an event stands for
std::vector<int> caller_waits;                    // launches the caller's stream waits for
std::vector<hipStream_t> host_waited;
int failing_call = -1, calls = 0;

template <typename T>
T handle(uintptr_t v) { return reinterpret_cast<T>(v); }
const hipStream_t kCaller = handle<hipStream_t>(1);

bool fails() { return calls++ == failing_call; }

}  // namespace

extern "C" {
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (fails()) return hipErrorUnknown;
    recorded[e] = queued[s];
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned int) {
    if (fails()) return hipErrorUnknown;
    if (s == kCaller) caller_waits.insert(caller_waits.end(), recorded[e].begin(), recorded[e].end());
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    host_waited.push_back(s);
    return hipSuccess;
}
}

int main() {
    lll::SideStreams ss;
    ss.fork = handle<hipEvent_t>(10);
    for (int i = 0; i < lll::kSideStreams; ++i) {
        ss.side[i] = handle<hipStream_t>(2 + i);
        ss.join[i] = handle<hipEvent_t>(11 + i);
    }
    int bad = 0;
    // no failure (-1), a failing launch, a failing HIP call
    for (int n : {1, 4, 11})
        for (int fail_at = -1; fail_at < n; ++fail_at)
            for (failing_call = -1; failing_call < 1 + 3 * lll::kSideStreams; ++failing_call) {
                queued.clear(), recorded.clear(), caller_waits.clear(), host_waited.clear();
                calls = 0;
                const hipError_t e = lll::run_beside(ss, kCaller, n, [&](int i, hipStream_t s) {
                    if (i == fail_at) return hipErrorLaunchFailure;
                    queued[s].push_back(i);
                    return hipSuccess;
                });
                std::vector<int> waited = caller_waits;
                for (hipStream_t s : host_waited)
                    waited.insert(waited.end(), queued[s].begin(), queued[s].end());
                for (int i = 0; i < lll::kSideStreams; ++i)
                    for (int launch : queued[ss.side[i]]) {
                        bool found = false;
                        for (int w : waited) found = found || w == launch;
                        if (!found) {
                            std::printf("n %d, launch %d failed, call %d failed: %d not waited for\n",
                                        n, fail_at, failing_call, launch);
                            bad = 1;
                        }
                    }
                const bool failed = fail_at >= 0 || (failing_call >= 0 && failing_call < calls);
                if ((e != hipSuccess) != failed) {
                    std::printf("n %d, launch %d, call %d: status %d\n", n, fail_at, failing_call, e);
                    bad = 1;
                }
                if (!failed && static_cast<int>(queued[kCaller].size()) != (n + 3) / 4) bad = 1;
            }
    std::printf(bad ? "FAILED\n" : "ok\n");
    return bad;
}
