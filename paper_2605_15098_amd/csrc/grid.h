// Launch shapes, apart from the HIP headers.
#pragma once

#include <algorithm>
#include <cstdint>

namespace svk {

// The runtime refuses a launch of 2^32 threads or more in one dimension, which
// a thread per 16 bytes reaches with a state of 64 GiB. Half of that, a power of
// two, keeps every launch a whole number of tiles.
constexpr uint64_t kLaunchThreads = 1ull << 31;

// Runs launch(first, count) over work-groups 0 .. groups - 1 of `threads`
// threads: one launch, or several in a row where one would be refused. A kernel
// launched through this takes its number as first + blockIdx.x. Zero is the
// launches' success.
template <typename F> auto split_launch(uint64_t groups, unsigned threads, F &&launch) -> decltype(launch(uint64_t(0), 0u))
{
    const uint64_t most = kLaunchThreads / threads;
    decltype(launch(uint64_t(0), 0u)) e{};
    for (uint64_t first = 0; first < groups && e == decltype(e){}; first += most)
        e = launch(first, (unsigned)std::min(most, groups - first));
    return e;
}

}  // namespace svk
