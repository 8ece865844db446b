// state_chunk.hpp -- how many paths' states a Greeks pass keeps at once (host code only).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace lll {

// The states of the forward pass, the increments, the fixings and the carried adjoint
// take 4 (s N (N+1) / 2 + K + 2 N) bytes per path (34 KB at 40 rates and 10 steps a period).
// Paths go in chunks whose states keep within kStateBytes: at those sizes a
// vector-Jacobian product of 2^18 paths takes 9.4 ms in one chunk of 8.6 GiB, 11.9 ms within
// 8 GiB, 16.4 within 4 and 25.5 within 2 (few wavefronts a launch, many launches).  With longer
// periods 16 GiB too would be few wavefronts, so a chunk takes kFillPaths paths all the
// same: 2^17 paths at 250 steps take 399 ms, 673 within 16 GiB.  A plan keeps its states,
// so it asks for at most 1 / kFreeShare of the memory that is free.
constexpr int64_t kStateBytes = int64_t(16) << 30;
constexpr int64_t kFillPaths = 32768;
constexpr int64_t kFreeShare = 4;
constexpr int64_t kChunkWave = 64;  // chunks are whole wavefronts: the sums do not depend on them

inline int64_t state_chunk(int64_t bytes_per_path, int64_t max_paths, int64_t free_bytes) {
    const int64_t all = (max_paths + kChunkWave - 1) / kChunkWave * kChunkWave;
    int64_t chunk = kStateBytes / bytes_per_path;
    if (chunk < kFillPaths) chunk = kFillPaths;
    if (chunk > free_bytes / kFreeShare / bytes_per_path)
        chunk = free_bytes / kFreeShare / bytes_per_path;
    chunk = chunk / kChunkWave * kChunkWave;
    if (chunk < kChunkWave) chunk = kChunkWave;
    if (chunk >= all) return all;
    const int64_t parts = (all + chunk - 1) / chunk;  // even chunks
    return ((all + parts - 1) / parts + kChunkWave - 1) / kChunkWave * kChunkWave;
}

// alloc(paths) with the chunk above, or where that does not fit, half as many paths at
// a time down to one wavefront; the paths of the allocation that succeeded, or 0 and its error.
template <typename Alloc>
int64_t alloc_state_chunk(int64_t bytes_per_path, int64_t max_paths, int64_t free_bytes,
                          Alloc &&alloc, hipError_t &e) {
    for (int64_t chunk = state_chunk(bytes_per_path, max_paths, free_bytes);;
         chunk = (chunk / 2 + kChunkWave - 1) / kChunkWave * kChunkWave) {
        e = alloc(chunk);
        if (e == hipSuccess) return chunk;
        if (e != hipErrorOutOfMemory || chunk <= kChunkWave) return 0;
    }
}

}  // namespace lll
