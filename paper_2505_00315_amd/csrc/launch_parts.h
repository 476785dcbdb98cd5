// Launch geometry of kernels whose blocks are independent and may number more
// than one launch can hold.  Plain C++ (no HIP), so that a CPU test can check it.
#pragma once

#include <stdint.h>

namespace mosa {

// Threads of a launch in one dimension stay below 2^32 (a launch of more is
// refused), so blocks [0, blocks) of `threads` threads each go out as
// consecutive launches launch(first, count); the kernel adds `first` to its
// block index.  One launch up to 2^32 / threads blocks.  Returns nonzero, and
// stops, at the first launch that does.
template <class F>
int launch_parts(uint64_t blocks, uint32_t threads, F launch) {
    const uint64_t most = 0xffffffffull / threads;
    for (uint64_t first = 0; first < blocks; first += most) {
        const uint64_t left = blocks - first;
        if (const int e = launch((uint32_t)first, (uint32_t)(left < most ? left : most))) return e;
    }
    return 0;
}

// fp32 attention: waves that share the loop over one block of 16 rows, up to
// max_waves (a power of two), fewer when the head has fewer blocks to share out.
inline int f32_attn_waves(int n, int max_waves) {
    const int nb = (n + 15) / 16;
    int nw = 1;
    while (nw < max_waves && 2 * nw <= nb) nw *= 2;
    return nw;
}

}  // namespace mosa
