// Workgroup LDS deposit cache of the transport kernel: the line lookup
// shared by the transport and the roofline replay (device code only).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"

namespace pmc {

// The cache holds lines of kLine neighbouring tally elements (64 bytes: the
// tally's innermost axis is z, the direction the beams run), each with one key.
// The memory side works one FP64 atomic request per 64-byte line, about 23.7
// thousand million a second whether it adds one double or eight: a line
// flushed by eight neighbouring lanes costs one request.  In an epoch of the
// 2000-spot field (32 iterations of 1024 lanes, 30,300 deposits) 9,950 single
// sums left 12,200 to 15,900 requests; the 1,755 lines that fit in the same LDS
// leave 4,900 to 6,900, half-size lines (3,316) as many, lines along x 13,000 to
// 16,800.  Launches: that field (1e7 histories) 17.8 ms with single sums, 15.3
// with lines; 2e6 histories of 444 spots with LET_d 6.7 and 3.6.

// hash of a line's index (and, in a batch, its plan): a 24-bit product, at full
// rate; linear probing after it found more free lines than after a 32-bit
// product or a mixed key
__device__ __forceinline__ uint32_t line_hash(uint32_t line, uint32_t plan = 0u)
{
    return ((line ^ (plan << 18)) & 0xFFFFFFu) * 0x9E3779u;
}

// The line of a workgroup's LDS cache that holds key, claiming a free one on
// the way (compare-and-swap), trying `probes` consecutive lines from the key's
// hash position; -1 when all are taken by other keys.
template <typename Key>
__device__ __forceinline__ int cache_line(Key* ckey, Key key, uint32_t h, uint32_t n_lines, int probes)
{
    constexpr Key kEmpty = ~Key(0);
    uint32_t at = ((h >> 16) * (n_lines & 0xFFFFu)) >> 16;   // (n_lines < 2^14)
    auto take = [&](uint32_t l) {
        Key held = ckey[l];
        if (held == kEmpty) {
            held = atomicCAS(&ckey[l], kEmpty, key);
            if (held == kEmpty) held = key;
        }
        return held == key;
    };
    bool hit = take(at);
    // further lines by linear probing
    for (int probe = 1; !hit && probe < probes; ++probe) {
        at = at + 1u == n_lines ? 0u : at + 1u;
        hit = take(at);
    }
    return hit ? (int)at : -1;
}

}  // namespace pmc
