// The rules by which launches get their shape, as plain host functions: the launchers apply them and
// the tests check them without a GPU.  Not part of the public ABI.
#pragma once

#include "eager_internal.h"

namespace eager {

// A grid must hold fewer than 2^32 threads in total; a launch beyond that is not refused
// by the runtime, its thread count wraps.  Every launcher stays at or below 2^31, and a round at
// one workgroup more: a run of 2^33 elements is 2^31 threads, and one that ends just below it
// needs a wavefront for its ragged tail besides.
constexpr long long kMaxGridThreads = 1ll << 31;
constexpr long long kMaxRoundThreads = kMaxGridThreads + 256;
constexpr long long kMaxRunElements = 1ll << 33;

// Workgroups of a round over n elements: a wavefront per tile, one more for the ragged tail.
inline long long round_workgroups(long long n, bool bf16, int block)
{
    const long long nvec = bf16 ? slot_nvec<true>(n) : slot_nvec<false>(n);
    const long long waves = (nvec + 63) / 64 + (nvec * 4 < n ? 1 : 0);
    const int per = block / 64;
    return (waves + per - 1) / per;
}

}  // namespace eager
