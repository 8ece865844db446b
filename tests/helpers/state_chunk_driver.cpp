// alloc_state_chunk (state_chunk.hpp): which chunks of paths it asks for with a given
// amount of free memory and an allocator that takes up to `limit` bytes.  Arguments: bytes per
// path, max paths, free bytes, limit; prints the chunk and the number of requests.
#include <cstdio>
#include <cstdlib>

#include "state_chunk.hpp"

int main(int, char **argv) {
    const int64_t per = std::atoll(argv[1]), paths = std::atoll(argv[2]);
    const int64_t limit = std::atoll(argv[4]);
    int requests = 0;
    hipError_t e = hipSuccess;
    const int64_t chunk = lll::alloc_state_chunk(
        per, paths, std::atoll(argv[3]),
        [&](int64_t n) {
            ++requests;
            return n * per <= limit ? hipSuccess : hipErrorOutOfMemory;
        },
        e);
    std::printf("%lld %d %d\n", static_cast<long long>(chunk), requests, e == hipSuccess);
    return 0;
}
