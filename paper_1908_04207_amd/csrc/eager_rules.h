// The rules by which launches get their shape, as plain host functions: the launchers apply them and
// the tests check them without a GPU.  Not part of the public ABI.
#pragma once

#include "eager_internal.h"

#include <algorithm>

namespace eager {

constexpr int kCus = 256;

// Occupancy is capped with LDS, which is handed out in units of 1280 bytes: a cap of w workgroups per
// CU realises floor(128 / floor(128 / w)) of them, so 32 (which is no cap for workgroups of one
// wavefront), 25, 21, 18, 16, 14, 12, 11, 10, 9 ... exist and the counts between run as the next one up.
constexpr int kLdsPerCu = 160 * 1024;
constexpr int kLdsUnit = 1280;
constexpr int kLdsUnits = kLdsPerCu / kLdsUnit;

// A grid must hold fewer than 2^32 threads in total; a launch beyond that is not refused
// by the runtime, its thread count wraps.  Every launcher stays at or below 2^31, and a round at
// one workgroup more: a run of 2^33 elements is 2^31 threads, and one that ends just below it
// needs a wavefront for its ragged tail besides.
constexpr long long kMaxGridThreads = 1ll << 31;
constexpr long long kMaxRoundThreads = kMaxGridThreads + 256;
constexpr long long kMaxRunElements = 1ll << 33;

// Elements by which a launch steps back from the first element of its run: its tiles then begin at multiples
// of 64 elements of the arena - whole cache lines of 128 bytes, of bf16 streams too, where the arena begins at
// one - and the first tile leaves out what stands before the run.  Buckets begin at any 16 bytes.  A tile that does not
// begin at a line shares lines with the next one, which another XCD reads and writes: both fetch it, and
// both write a part of it.  (Ranges that begin 32 bytes behind a line, time over that of the bytes and a launch, before
// and now: 8 processes, 4 late, 0.5, 1, 4 and 8 M elements 1.24 1.17 1.13 1.05 and 1.16 1.09 1.05 0.98; 12, 11 late, 1.26 1.17
// 1.12 1.11 and 1.14 1.07 1.04 1.02; bf16, 16, 8 late, 1.38 1.25 1.20 1.14 and 1.26 1.16 1.11 1.05.)
constexpr long long kTileAlign = 64, kAlignFrom = 1024;
inline long long run_back(long long e0, long long n)
{
    return n < kAlignFrom || n > kMaxRunElements - kTileAlign ? 0 : e0 % kTileAlign;
}

// A lane of a wavefront on a tile of such a launch, `left` > 0 lane-vectors before the run ends and `skip` of the first tile
// standing in front of it: lanes without a lane-vector of their own take the nearest of the run.  Offsets count from the first
// lane-vector of the tile that belongs to the run, so that 0 - what all lanes of a SKIP load - lies inside it too.
// (In 32 bits, which hold the 2^31 lane-vectors of the largest run: with few streams what a wavefront does before its
// first load counts.  One stream of 280 M elements into the receive buffer 474 us without a look at `skip`, 482 with it in 64
// bits, 465 in 32.)
struct LanePlace {
    unsigned first;        // lane-vector of the launch that offsets count from
    unsigned at;           // offset, in lane-vectors
    bool in;               // the lane's own lane-vector belongs to the run
    bool held;             // it does, or stands in front of it
};
constexpr LanePlace place_lane(unsigned lane, unsigned tile, unsigned left, unsigned skip)
{
    const unsigned last = left > 64u ? 63u : left - 1u, first = tile == 0u ? skip : 0u;
    const unsigned up = lane > first ? lane : first, lv = up < last ? up : last;
    return {tile * 64u + first, lv - first, lv == lane, lane <= last};
}

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
// processes with norms, 65536 buckets in 4 M elements, 290 and 147 us.)  It also bounds the grid: 2^32
// threads are 16 M buckets; finish_slices keeps below.
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

constexpr int kNormsTiles = 8;         // records of norms_kernel come in groups of so many

// Whether 2 or 3 slices are worth it.  Not where one workgroup has the records in about a trip, nor where those of the other
// buckets that have nothing to do (n slices are n workgroups to every bucket) do not all fit the chip beside them; of
// 256 threads, which take more trips, up to 1536 buckets.  Two processes with norms, one bucket of 1.1, 2 and 3.1 M elements among
// small ones, one workgroup to a bucket and slices: 64 buckets 9.5 13.4 16.5 and 9.6 11.2 14.6 us, 161 10.0 13.7 17.8 and 10.9
// 12.7 15.7, 600 10.8 14.4 18.5 and 12.4 15.6 19.5, 1000 12.3 15.7 20.5 and 12.4 14.9 17.7, 3000 15.4 18.5 23.3 and 16.6 19.8 24.0;
// every 8th of 200 and of 400 of 2.5 M, the finishing kernel alone 9.9 15.7 and 11.2 17.8.
inline bool few_slices(long long records, long long slices, int buckets)
{
    if (finish_threads(buckets) < 1024) return records > 5632 && buckets <= 1536;
    return records > (buckets <= 64 ? 5632 : 7168) && slices * buckets < 2 * kCus;
}

// The slices of the finishing kernel, for the largest of the launch's `buckets`: 4096 records to a workgroup - one in 8 where
// they come in groups - which is one trip to memory for 1024 threads and two for 256, or as many more as 64 slices come to.
// Half or a quarter as many are faster while that makes no more workgroups than CUs, most of which have nothing to do where
// the other buckets are small (1 bucket of 12 k records 5.4 us with 4096, 5.0 with 1024; but up to 4 k in slices, 1.5 M elements in 22 buckets, norms and layer-wise step
// 27.6 us, 26.0 with one workgroup to a bucket; 5 of up to 50 k 6.3 and 5.7; but 48 of up to 20 k 6.4 and 11.0).  A first launch for
// the slices and a second for the totals, which this was, took 8.9, 9.6 and 9.7; and 7.8 for 161 of up to 9 k, 6.7 now.
// Two or three slices are a trip less and a count of arrivals more: see few_slices.
// Groups: 800 buckets of 10 k elements and one of 70 M 26.6 us in 64 slices, 14.5 in 9.  Slices of the largest bucket's
// records, not of the run's: 8 buckets of 273 k each 19.8 us in 8 slices, 13.6 in 64 (two launches 16.9).
inline void finish_slices(StatsArgs &a, int buckets, bool grouped)
{
    const long long unit = grouped ? kNormsTiles : 1, most = (a.largest + unit - 1) / unit;
    // (a grid of more threads than a launch takes would wrap: 131072 buckets times 64 slices are just as many)
    const long long fits = kMaxGridThreads / (static_cast<long long>(finish_threads(buckets)) * buckets);
    const long long room = std::min<long long>(std::max(fits, 1ll), kStatsMaxSlices);
    long long per = kStatsRecordsPerSlice, n = std::max((most + per - 1) / per, 1ll);
    if (n <= 3 && !few_slices(most, n, buckets)) n = 1;
    if (n >= room) {
        n = room;
        per = (most + n - 1) / n;
    }
    while (n > 1 && n < room && per > 1024 && 2 * n * buckets <= kCus) {
        n = std::min(2 * n, room);
        per = n < room ? per / 2 : (most + n - 1) / n;
    }
    a.slices = static_cast<int>(n);
    a.per_slice = static_cast<int>((per * unit + kNormsTiles - 1) / kNormsTiles * kNormsTiles);
}

// Whether the update with a rate per bucket takes a workgroup per bucket, whose u, w and v wait in its registers between
// the norms and the update: one launch instead of three, 20 bytes per element instead of 28.  Up to 16384 elements in the
// largest bucket; a workgroup of 1024 threads has a CU to itself, so that beyond 4096 many buckets must not be tiny.  Three
// launches and this: one bucket of 256, 4096, 16384 elements 6.0 6.7 6.7 and 2.4 3.6 5.3 us; 64 of up to 1024 10.3 and 3.1;
// 16384 of 1024 111 and 57, of up to 4096 121 and 73, of up to 16384 402 and 319; 512 of 16384 51 and 33; but one of
// 16384 among 1024 of 256 10.2 and 12.5, among 4096 of 256 16.5 and 39.
// `ends`: the most elements from a bucket's last whole lane-vector to the next bucket of the run, padding included, one to a
// lane of its workgroup.  (Padding in the registers beside the bucket's own makes one of 4096 with 8 behind it a case of
// workgroups of 1024 threads: 4096 of up to 4096 53 us, 42 with three launches, 22 in this way.)
constexpr int kBucketEnd = 256;
inline bool rate_by_bucket(long long largest, long long ends, long long elements, int buckets)
{
    if (ends > kBucketEnd || buckets > 1 << 21) return false;
    return largest <= 4096 || (largest <= 16384 && (buckets <= 512 || elements >= 1024ll * buckets));
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

// Whether a run is bound by latency - everything at once, no cap (chunk_kernel) - and not a stream
// (burst_kernel).  A stream begins at 96 MiB moved where the run only reads fp32 streams, at 112 MiB where
// bursts are shorter (bf16) or copies follow them, and at 56 MiB where one or two bf16 streams are all
// there is, which a wavefront takes in one burst anyway.  Both sides, chunks and bursts, one state in a
// loop: 8 processes on time, fp32, 96 MiB 15.2 and 16.7 us, 112 MiB 17.7 and 17.8, into the receive buffer 96
// MiB 17.4 and 16.4; 16 processes 96 MiB 16.7 and 16.1, 112 MiB 20.0 and 17.8; 3 processes, 1 late, 100 MiB 15.2 and
// 17.4, 128 MiB 22.0 and 21.8; 8 processes, 4 late, 100 MiB 15.8 and 18.1, 112 MiB 18.6 and 19.6; 16 on time with
// bf16 gradients 100 MiB 16.9 and 19.4, 128 MiB 21.5 and 23.2.  One bf16 stream 80 MiB 15.1 and 16.5, two 13.4 and 13.4:
// the line at 56 MiB was drawn when chunks were filled up with loads (17.1 and 16.6, 14.4 and 13.3).
inline bool small_round(const SlotArgs &s, long long bytes_per_element)
{
    const long long moved = s.h.n * bytes_per_element;
    if (moved <= 56ll << 20) return true;
    if (moved > 112ll << 20) return false;
    if (s.h.n_copy) return true;
    bool bf16 = false;
    for (int k = 0; k < s.h.n_sum; ++k) bf16 = bf16 || (s.slot[k] & kSlotBf16);
    return bf16 ? s.h.n_sum > 2 : moved <= 96ll << 20;
}

// Accesses of a small run are plain where the whole model moves no more than 56 MiB in a round: its
// arrays then stay in the last-level cache from round to round.  Small runs of a larger model are
// streamed.  Both sides, plain and streamed, one state in a loop: 8 processes, 4 late, 40 MiB 6.4
// and 7.7 us; 16 processes, all on time, 64 MiB 12.0 and 10.4, 8 processes 11.4 and 9.9; with cold buffers
// 9.9 and 10.6 at 40 MiB, 14.1 and 13.6 at 64.
constexpr long long kPlainRoundBytes = 56ll << 20;

// Resident wavefronts per CU of the weight-view kernels when the caller leaves it open, -1: no cap.  Half of the traffic is
// stores: few, as for the rounds.  What counts is the KiB of loads in flight per CU, about 38 for the update (1 + 2 per
// view loads per lane, views in chunks of 8) and 26 for the average (one load per view).  25.6 M elements, update: 8 views
// 550 us with 2, 540 with 3, but 4 M 87 and 95; 10 views 708 with 2, 686 with 3, 688 with 4, uncapped 776; 16 views 1093,
// 1144, 1185, 1261; average: 4 views 127.4 with 8, 124.7 with 6, 130.4 with 5, uncapped 139; 6 views 191.0 with 5, 187.9 with 4, 211 with 3; 8 views 255.6 with 4,
// 257.6 with 3; 12 views 393 and 388; 2 views 62 with 16, 65 with 12.
// The average of more than 16 views, whose kernel has 16 loads in flight: 17 views of 0.4, 1 and 25.6 M elements 10.6 26.7 561 us
// with 4, 11.7 27.6 595 with 3; 40 of 0.4, 1 and 4 M 23.6 60.4 239 and 24.6 59.2 213.
// Up to 6 tiles per CU there is no cap (update of 8 views of 200 k elements 5.7 us with 3 and 5.3 without; average of 64 of 390 k 36.8
// and 31.6), but for updates of more than 24 views (48 and 64 of 390 k 51 and 70 us with 2, 55 and 75 without).
inline long long views_tiles(long long n) { return std::max((n / 4 + 63) / 64, 1ll); }
inline int views_sgd_waves(int n_views, long long n)
{
    if (n_views <= 24 && views_tiles(n) <= 6 * kCus) return -1;
    const int loads = 1 + 2 * (n_views < 8 ? n_views : 8);
    return std::max((38 + loads / 2) / loads, n_views > 8 && n_views <= 12 ? 3 : 2);
}
inline int views_average_waves(int n_views, long long n)
{
    if (n_views == 1 || views_tiles(n) <= 6 * kCus) return -1;
    if (n_views < 4) return 32 / n_views;
    const bool three = n_views > 16 ? n_views >= 24 && n >= 1 << 20 : n_views >= 12;
    return std::max(26 / n_views, three ? 3 : 4);
}

// Whether the average streams its views past the caches.  Up to 56 MiB plain accesses are faster (see kPlainRoundBytes) from 4 views on,
// of 4 to 8 not below 28 MiB (4: 32), where the views just fit the second-level caches: 1 and 2 views streamed and plain, 18 to 30 MB 4.2
// to 5.5 and 4.5 to 6.6 us, 34 MB 4.6 and 5.5 (2 views); 4 views of 24 MB 4.4 and 4.5, of 52 MB 7.7 and 6.7; 8 views 4.1 4.4 and 8.1 6.7;
// 16 views 4.5 4.6 and 9.1 6.9.
inline bool views_average_streamed(int n_views, long long n)
{
    const long long bytes = n * 8 * n_views;
    return bytes > kPlainRoundBytes || n_views < 4 || (n_views <= 8 && bytes < (n_views == 4 ? 32ll : 28ll) << 20);
}

// Slots of the sum without what fills them up.
inline int sum_terms(const SlotArgs &s)
{
    int n = s.h.n_sum;
    while (n > 0 && (s.slot[n - 1] & kKindMask) == kSkip) --n;
    return n;
}

// The same round for the kernel of small runs: elements [first, first + n) of the run.  `A` has room for
// the list (slots that fill it up are left out).
inline bool chunk_fits(const SlotArgs &s, int slots, int copies)
{
    return s.h.n_sum + s.h.n_copy <= slots && s.h.n_copy <= copies;
}
template <typename A>
void fill_chunk(const SlotArgs &s, bool any_order, long long first, long long n, A &a)
{
    const long long e = s.h.e0 + first;
    auto at = [e](float *p) { return p ? p + e : nullptr; };
    a.h.w = at(s.h.w);
    a.h.v = at(s.h.v);
    a.h.recv = at(s.h.recv);
    a.h.n = static_cast<unsigned>(n);
    a.h.inv_P = s.h.inv_P;
    a.h.neg_lr = s.h.neg_lr;
    a.h.mu = s.h.mu;
    a.h.wd = s.h.wd;
    a.h.nesterov = s.h.nesterov;
    a.h.form = first == 0 ? s.h.skip * 4 << kFormBits : 0;
    for (ChunkBits &b : a.bits) b = ChunkBits{0u, 0u, 0u, 0u};
    int k = 0;
    auto push = [&](unsigned long long slot, unsigned ChunkBits::*what) {
        const bool bf = (slot & kSlotBf16) != 0;
        const unsigned bit = 1u << (k % kChunkWord);
        ChunkBits &b = a.bits[k / kChunkWord];
        if (what) b.*what |= bit;
        if (bf) b.bf |= bit;
        a.slot[k++] = (slot & ~static_cast<unsigned long long>(kSlotTag)) +
                      static_cast<unsigned long long>(e) * (bf ? 2 : 4);
    };
    const int terms = sum_terms(s);
    auto term = [&](int j) {
        const unsigned kind = static_cast<unsigned>(s.slot[j]) & kKindMask;
        push(s.slot[j], kind == kAdd ? nullptr : kind == kPair ? &ChunkBits::pair : &ChunkBits::hold);
    };
    if (any_order) {
        for (unsigned long long type : {0ull, static_cast<unsigned long long>(kSlotBf16)})
            for (int j = 0; j < terms; ++j)
                if ((s.slot[j] & kSlotBf16) == type) term(j);
    } else {
        for (int j = 0; j < terms; ++j) term(j);
    }
    a.h.n_sum = k;
    a.h.dst_first = k & ~7;
    for (int j = 0; j < s.h.n_copy; ++j) {
        a.dst[k - a.h.dst_first] = s.dst[s.h.n_sum + j] + e;
        push(s.slot[s.h.n_sum + j], &ChunkBits::copy);
    }
    a.h.n_slots = k;
    a.h.first = a.bits[0];
}

// Whether the kernel of short lists can take a small run.  (Statistics have arguments of their own; a launch is within
// 32-bit offsets.)
inline bool short_round(const SlotArgs &s)
{
    return !s.stats.stats && sum_terms(s) + s.h.n_copy <= 16 && s.h.n_copy <= kShortCopies && s.h.n <= kChunkElements;
}
template <int SLOTS>
void fill_short(const SlotArgs &s, bool any_order, int form, ShortArgs<SLOTS> &a)
{
    const long long e = s.h.e0;
    auto at = [e](float *p) { return p ? p + e : nullptr; };
    a.w = at(s.h.w);
    a.v = at(s.h.v);
    a.recv = at(s.h.recv);
    a.n = static_cast<unsigned>(s.h.n);
    a.inv_P = s.h.inv_P;
    a.neg_lr = s.h.neg_lr;
    a.mu = s.h.mu;
    a.wd = s.h.wd;
    auto base = [e](unsigned long long slot) {
        return (slot & ~static_cast<unsigned long long>(kSlotTag)) + static_cast<unsigned long long>(e) * (slot & kSlotBf16 ? 2 : 4);
    };
    const int terms = sum_terms(s);
    unsigned bits = 0u;
    int k = 0;
    auto term = [&](int j) {
        const unsigned long long slot = s.slot[j];
        bits |= ((slot & kKindMask) == kPair ? 1u << k : 0u) | (slot & kSlotBf16 ? 0x10000u << k : 0u);
        a.slot[k++] = base(slot);
    };
    if (any_order) {                 // all fp32 streams before the bf16 ones
        for (int j = 0; j < terms; ++j)
            if (!(s.slot[j] & kSlotBf16)) term(j);
        for (int j = 0; j < terms; ++j)
            if (s.slot[j] & kSlotBf16) term(j);
    } else {
        for (int j = 0; j < terms; ++j) term(j);
    }
    const int first = std::max(terms, a.kHalf);           // of the copies
    k = first;
    for (int j = 0; j < s.h.n_copy; ++j) {
        const unsigned long long slot = s.slot[s.h.n_sum + j];
        a.dst[k - a.kHalf] = s.dst[s.h.n_sum + j] + e;
        bits |= slot & kSlotBf16 ? 0x10000u << k : 0u;
        a.slot[k++] = base(slot);
    }
    a.bits = bits;
    a.copies = (1u << k) - (1u << first);
    a.shape = static_cast<unsigned>(terms | (k - a.kHalf) << 8 | (s.h.nesterov ? 1 << 16 : 0) | form << kShortForm) |
              static_cast<unsigned>(s.h.skip * 4) << kShortSkip;
}

// Whether a lane of such a launch owns one element and not four: four times the wavefronts with a
// quarter of the arithmetic each, and up to 32 slots in one trip to memory instead of 16.  From 9 slots
// on, up to 128 k elements (one launch after another, 4 elements to a lane and 1): 8 processes, 4 late, 4096
// elements 2.96 and 2.86 us, 65536 3.47 and 3.52, 131072 4.54 and 4.35, 262144 5.69 and 6.00; 16 processes, 8
// late, 4096 4.24 and 3.28, 131072 5.93 and 5.16, 262144 8.4 and 9.1; but with 3 slots 2.60 and 2.66, 2.87 and
// 3.12.  Up to 32 k where more than 40 bf16 gradients are copied (64 processes, 63 late, bf16: 32 k elements 15.7
// and 15.8 us, 64 k 16.5 and 20.3, 128 k 20.8 and 27.9; 48 processes, 47 late, 128 k 15.7 and 18.4; but 64 processes,
// 32 late, 128 k 13.4 and 13.2, and with fp32 gradients, 63 late, 20.2 and 18.4).  (By-products are kept per 256 elements,
// so a launch with them is never narrow; nor is one whose loads in flight the caller has set: chunk, 0 where it
// has not.)
inline bool chunk_narrow(long long n, int slots, int copies, bool bf16, bool stats, int chunk)
{
    return chunk == 0 && !stats && slots > 8 && n <= (bf16 && copies > 40 ? 1ll << 15 : 1ll << 17);
}

// Wavefronts that a CU holds of a kernel with so many vector registers: 512 on each of its 4 SIMDs, handed out in
// eights.
inline int resident_waves(int registers)
{
    const int each = (registers + 7) / 8 * 8;
    return registers < 1 ? 0 : each <= 64 ? 32 : 4 * (512 / each);
}

// Whether the copies' stores of such a launch go out one at a time.  Where all its wavefronts are resident at once
// (`resident` per CU, 20 or 16 in chunks of 16) that keeps the stores of the first behind the loads of the last, and the memory side reads for a
// while and then writes.  It takes 6 copies to pay, 5 with bf16 gradients, a list in flight as a whole (further
// loads would wait behind the stores) and a run that streams.  Stores at once and one at a time, one state in a
// loop, 58, 72, 88 and 104 MiB moved: 8 processes, 7 late, bf16 10.3 11.8 14.7 17.6 and 9.0 11.4 12.9 16.0 us, fp32 9.2
// 11.7 14.5 17.8 and 8.8 11.5 14.2 17.2; 8 processes, 5 late, bf16 9.9 11.7 14.7 and 9.0 11.1 13.9, but at 104 MiB (23 tiles
// per CU) 16.8 and 18.1; 10 processes, 4 late, bf16 14.3 and 14.8 at 88; 12 processes, 11 late, 23 slots 11.6 and 13.4
// at 72.
inline bool chunk_paced(const SlotArgs &s, int slots, bool bf16, bool update, int resident)
{
    return slots <= 16 && s.h.n_copy >= (bf16 ? 5 : 6) && s.h.n <= static_cast<long long>(resident) * kCus * 256 &&
           s.h.n * round_bytes(s, update) > kPlainRoundBytes;
}

// Whether a run that the kernel of short lists can take (short_round) is its: where it is ahead of chunk_kernel, which is
// nearly everywhere (eager_short.h has the times).  Not so, short_kernel and chunk_kernel:
//   * where copies are stored one at a time (chunk_paced), which takes the wavefronts that chunk_kernel has registers for: 8
//     processes, 7 late, 1.06 M elements, fp32 fused 15.9 and 14.6 us, bf16 13.8 and 12.1
//   * bf16 in any order, beyond the 128 k elements up to which a lane may have one, from 8 streams on: 12 processes with
//     4 send buffers, 262 k 4.76 and 4.43 us, 8 processes 3.06 and 2.93 (4 processes 2.79 and 2.79)
//   * bf16 in fixed order, one element to a lane, 4 or more send buffers among many streams: 8 processes with 8 send
//     buffers 1024 elements 3.16 and 2.86 us, 131 k 4.52 and 3.70; with 4, 4 late 2.96 and 2.87; with 4, on time, 2.68 and 2.74
inline bool short_pays(const SlotArgs &s, bool bf16, bool fast, bool nt, bool update)
{
    const int terms = sum_terms(s), slots = terms + s.h.n_copy;
    if (nt && chunk_paced(s, slots, bf16, update, 32)) return false;
    if (!bf16) return true;
    if (fast) return s.h.n <= 1 << 17 || slots < 8;
    int fp32 = 0;
    for (int j = 0; j < terms; ++j) fp32 += !(s.slot[j] & kSlotBf16);
    return fp32 < 4 || slots + s.h.n_copy <= 12 || !chunk_narrow(s.h.n, slots, s.h.n_copy, bf16, false, 0);
}

// Resident wavefronts per CU of the burst kernel, -1: no cap.
//   * 14 for fp32 streams (26 KiB in flight), 12 where copies follow.  A wavefront with few slots spends
//     more of its life on its arguments, on w and v and on stores, so short lists with copies take
//     more: 18 up to 5 slots, 14 up to 9 (3 processes, 1 late, 26 M elements: 139 us with 12, 130 with
//     18; into the receive buffer 109 and 94; 4 processes, 2 late 177 and 175 with 14; 8 processes, 4
//     late, 12 slots: 289 with 12, 295 with 16).
//   * Up to 1.75 times as many with bf16 streams, whose bursts are half as large (34 of 34 streams bf16,
//     43 M elements: 585 us with 25, 619 with 21, 780 with 14, 594 without a cap; 27 of 34: 946 with 25,
//     960 with 21), and more still where the wavefront moves little else: into the receive buffer (8
//     processes on time, 40 M elements: 118 us without a cap, 127 with 25; 16 processes 230 and 243), or
//     beside by-products while w and v come from the last-level cache (8 processes, 16 M: 84 and 85; but
//     80 M elements 426 and 410).
//   * With by-products it also computes for a while with nothing in flight: 2 more beside fp32 streams (8
//     processes, 32 M elements: 239 us with 14, 230 with 16; 16 processes 414 and 406), 4 more where copies
//     and the update rule meet (8 processes, 26 M elements, finish included: 298.8 with 16, 309.5 with
//     12); into the receive buffer with copies none (386 us a layer-wise step with 12, 394 with 16).
//   * A run of few generations of wavefronts takes the neighbouring count that fills them best (2 M
//     elements, 32 tiles per CU: 49.3 us with 16, 52.1 with 14); one that fits the chip at once needs no
//     cap (1 M elements, 16 processes: 34.8 us, 42.7 with 14).
inline int burst_waves(const SlotArgs &s, long long tiles, bool stats, bool update, bool state_streamed)
{
    const int n = s.h.n_sum + s.h.n_copy;
    int n_bf = 0;
    for (int k = 0; k < n; ++k)
        n_bf += (s.slot[k] & kSlotBf16) && (s.slot[k] & (kKindMask | kSlotCopy)) != kSkip;
    int w0 = !s.h.n_copy ? 14 : n <= 5 ? 18 : n <= 9 ? 14 : 12;
    if (n > 0) {
        w0 += 3 * 14 * n_bf / (4 * n);
        if (s.h.n_copy) {
            if (stats && update) w0 += 4 * (n - n_bf) / n;
        } else {
            if (!update || (stats && !state_streamed)) w0 += 6 * n_bf / n;
            if (stats) w0 += 2 * (n - n_bf) / n;
        }
    }
    const long long per_cu = (tiles + kCus - 1) / kCus;
    if (per_cu <= w0 + 6) return -1;
    int best = -1;
    double least = 1e9;
    for (int units = 4; units <= 16; ++units) {
        const int w = kLdsUnits / units;
        if (w < w0 - 2 || 3 * w > 4 * w0) continue;
        const long long generations = (per_cu + w - 1) / w;
        const double cost = static_cast<double>(generations * w) / static_cast<double>(per_cu) +
                            0.16 / w0 * (w > w0 ? w - w0 : w0 - w);
        if (cost < least) {
            least = cost;
            best = w;
        }
    }
    return best == 32 ? -1 : best;
}

}  // namespace eager
