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

// Threads of the workgroup that finishes a bucket's statistics.  1024 make fewest trips to memory and
// are best while the chip holds most of the buckets' workgroups at once; with many buckets, which
// are then small, four times as many workgroups of 256 run at a time.  (Norms, finish and update of
// the layer-wise rule behind a round, 1024 and 256 threads: 600 buckets in 40 M elements 403 and 407
// us, 800 in 36 M 366 and 363, 1000 in 20 M 219 and 216, 2000 in 16 M 181 and 171; a round of two
// processes with norms, 65536 buckets in 4 M elements, 290 and 147 us.)  It also bounds the grid: 2^32 threads are more than
// 16 M buckets, or 262 k where one of them takes all the slices of a first stage.
inline int finish_threads(int n_buckets) { return n_buckets > 768 ? 256 : 1024; }

// Whether the norms pass of the layer-wise rule works in groups of 8 tiles: from 50 M elements, with
// 32 k elements per bucket on average.  A group that buckets share goes through its tiles one by one
// (4 M elements in buckets of 3000, the three kernels of the rule: 41 us in groups, 29.7 by tiles), and
// below 50 M elements even whole groups leave too few wavefronts (2.3 M in 161 buckets 26.8 and 17.2;
// 40 M in 600 190 and 179).  Above: 67 M in one bucket behind a round 632 and 644, 200 M in 2000 909 and
// 943, 140 M in 3000 637 and 670, 64 M in 400 both 292; but 268 M in one bucket 1190 and 1184.
inline bool norms_grouped(long long tiles, int n_buckets)
{
    return tiles >= 3 << 16 && tiles >= 128ll * n_buckets;
}

}  // namespace eager
