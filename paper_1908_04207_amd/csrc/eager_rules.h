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

// Bytes a launch of a round moves per element: every stream read once by its type, the copies, and
// w and v read and written or the receive buffer written.
inline long long round_bytes(const SlotArgs &s, bool update)
{
    long long bytes = update ? 16 : 4;
    for (int k = 0; k < s.h.n_sum + s.h.n_copy; ++k) {
        const bool copy = (s.slot[k] & kSlotCopy) != 0, skip = (s.slot[k] & kKindMask) == kSkip && !copy;
        if (!skip) bytes += ((s.slot[k] & kSlotBf16) ? 2 : 4) + (copy ? 4 : 0);
    }
    return bytes;
}

// A run that moves at most this is bound by latency: everything at once, no cap (chunk_kernel).  Beyond
// it is a stream (burst_kernel): from 96 MiB where it only reads fp32 streams, from 112 MiB where bursts
// are shorter (bf16) or copies follow them.  Both sides, chunks and bursts, one state in a loop: 8
// processes on time, fp32, 96 MiB 18.3 and 15.0 us, 112 MiB 21.4 and 19.3, 16 processes 112 MiB 19.8 and 17.6;
// 3 processes, 1 late, 88 MiB 13.9 and 18.1, 100 MiB 15.7 and 17.9; 8 processes, 4 late, 100 MiB 17.1 and
// 18.6; 16 on time with bf16 gradients 100 MiB 16.2 and 19.2.
inline bool small_round(const SlotArgs &s, bool update)
{
    bool reads_fp32 = s.h.n_copy == 0;
    for (int k = 0; k < s.h.n_sum; ++k) reads_fp32 = reads_fp32 && !(s.slot[k] & kSlotBf16);
    return s.h.n * round_bytes(s, update) <= (reads_fp32 ? 96ll : 112ll) << 20;
}

// Accesses of a small run are plain where the whole model moves no more than 56 MiB in a round: its
// arrays then stay in the last-level cache from round to round.  Small runs of a larger model are
// streamed.  Both sides, plain and streamed, one state in a loop: 8 processes, 4 late, 40 MiB 6.4
// and 7.7 us; 16 processes, all on time, 64 MiB 12.0 and 10.4, 8 processes 11.4 and 9.9; with cold buffers
// 9.9 and 10.6 at 40 MiB, 14.1 and 13.6 at 64.
constexpr long long kPlainRoundBytes = 56ll << 20;

}  // namespace eager
