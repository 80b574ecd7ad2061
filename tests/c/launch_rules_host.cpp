// The rules that give launches their shape (csrc/eager_rules.h), checked on the CPU: built and run
// by tests/test_launch_rules.py.
#include "../../paper_1908_04207_amd/csrc/eager_rules.h"

#include <cstdio>

#define CHECK(cond)                                                              \
    do {                                                                         \
        if (!(cond)) {                                                           \
            std::printf("line %d: %s\n", __LINE__, #cond);                       \
            return 1;                                                            \
        }                                                                        \
    } while (0)

using namespace eager;

// Every run that a call accepts has a grid: enough wavefronts for its tiles and its ragged tail,
// and a thread count that the launcher takes and 32 bits hold.
static int grids()
{
    const long long top = kMaxRunElements;
    for (int bf16 = 0; bf16 < 2; ++bf16)
        for (int block = 64; block <= 256; block *= 2)
            for (long long base : {1ll, 256ll, 4096ll, 1ll << 20, 1ll << 31, top - 4096, top - 256, top - 8})
                for (long long n = base; n < base + 300 && n <= top; ++n) {
                    const long long g = round_workgroups(n, bf16 != 0, block);
                    const long long nvec = bf16 ? slot_nvec<true>(n) : slot_nvec<false>(n);
                    const long long waves = g * (block / 64), tiles = (nvec + 63) / 64;
                    CHECK(waves >= tiles + (nvec * 4 < n) && waves < tiles + 1 + block / 64);
                    CHECK(g * block <= kMaxRoundThreads && g * block < (1ll << 32));
                }
    return 0;
}

// Every lane of every tile reads inside the run, a SKIP's too: 4 elements of an fp32 stream, an aligned piece of 8 of a
// bf16 stream; the lanes that are in have the run's lane-vectors, each one.
static int lanes()
{
    const unsigned most = static_cast<unsigned>(kMaxRunElements / 4);
    for (unsigned skip = 0; skip < 16; ++skip)
        for (unsigned nvec : {256u, 256u + 15, 300u, 512u, most - 1, most})
            for (unsigned tile = 0; tile * 64 < nvec; tile += tile < 8 ? 1 : tile + 4 < nvec / 64 ? nvec / 64 - tile - 3 : 1) {
                const unsigned tile0 = tile * 64;
                unsigned next = tile == 0 ? skip : tile0;
                for (unsigned lane = 0; lane < 64; ++lane) {
                    const LanePlace p = place_lane(lane, tile, nvec - tile0, skip);
                    CHECK(p.first >= skip && p.first + p.at < nvec);
                    if (skip % 2 == 0 && nvec % 2 == 0)
                        CHECK((p.first + p.at) / 2 == p.first / 2 + p.at / 2 && p.first % 2 == 0);
                    CHECK(p.in == (tile0 + lane >= skip && tile0 + lane < nvec));
                    CHECK(p.held == (tile0 + lane < nvec) && p.first == place_lane(0, tile, nvec - tile0, skip).first);
                    if (p.in) CHECK(p.first + p.at == next++);
                }
                CHECK(next == (nvec < tile0 + 64 ? nvec : tile0 + 64));
            }
    return 0;
}

// How far a launch steps back: to a multiple of 64 elements, runs of 1024 elements or more, and never beyond the largest run.
static int back()
{
    for (long long e0 : {0ll, 4ll, 60ll, 64ll, 68ll, (1ll << 40) + 32}) {
        CHECK(run_back(e0, 1023) == 0 && run_back(e0, 1024) == e0 % 64);
        CHECK(run_back(e0, kMaxRunElements - 64) == e0 % 64 && run_back(e0, kMaxRunElements - 63) == 0 && run_back(e0, kMaxRunElements) == 0);
    }
    return 0;
}

// The finishing kernels: many buckets get small workgroups, and no more threads in all than a
// workgroup of 256 per bucket and slice would take.
static int finishing()
{
    for (int n : {1, 2, 161, 600, 768, 769, 1000, 4096, 65536, 1 << 20, (1 << 24) - 1}) {
        const long long t = finish_threads(n);
        CHECK(t == 256 || t == 1024);
        CHECK(n >= 1000 ? t == 256 : n > 600 || t == 1024);
        CHECK(n * t <= 1024 * 1024ll || t == 256);
        CHECK(n * t < 1ll << 32);
    }
    return 0;
}

static StatsArgs sliced(long long largest, int buckets, long long records, bool grouped = false)
{
    StatsArgs a{};
    a.largest = static_cast<int>(largest);
    a.n_records = records;
    finish_slices(a, buckets, grouped);
    return a;
}

// A bucket's records in slices: whole groups of records, enough of them for the largest bucket, and no more to a slice than
// 4096 or, with all 64 in use, its share of that bucket, whatever stands beside it.
static int slices()
{
    for (long long most : {0ll, 1ll, 4096ll, 4097ll, 12'288ll, 12'289ll, 100'000ll, 258'048ll, 258'049ll, 262'144ll, 273'438ll, 1ll << 25})
        for (int buckets : {1, 2, 3, 8, 64, 161, 768, 769, 5000})
            for (long long others : {0ll, 1ll, 7ll}) {
                const StatsArgs a = sliced(most, buckets, std::min((others + 1) * most + 8, 1ll << 25));
                CHECK(a.slices >= 1 && a.slices <= kStatsMaxSlices && a.per_slice > 0 && a.per_slice % kNormsTiles == 0);
                if (a.slices > 1) CHECK(a.slices * static_cast<long long>(a.per_slice) >= most);
                if (a.slices == kStatsMaxSlices) CHECK(a.per_slice < most / kStatsMaxSlices + 1 + kNormsTiles || a.per_slice <= 4096);
                const StatsArgs alone = sliced(most, buckets, most + 8);
                CHECK(a.slices == alone.slices && a.per_slice == alone.per_slice);
                const StatsArgs group = sliced(most, buckets, most + 8, true), eighth = sliced((most + 7) / 8, buckets, most + 8);
                CHECK(group.slices == eighth.slices && group.per_slice >= 8 * eighth.per_slice - 56);
                CHECK(group.per_slice <= 8 * eighth.per_slice && group.per_slice % kNormsTiles == 0);
                CHECK(group.slices == 1 || group.slices * static_cast<long long>(group.per_slice) >= most);
            }
    // every grid within what a launch takes
    for (int buckets : {1000, 65'536, 131'072, 200'000, 262'144, 1 << 20, 1 << 23})
        for (long long most : {12'289ll, 258'049ll, 1ll << 25})
            for (bool grouped : {false, true}) {
                const StatsArgs a = sliced(most, buckets, 1ll << 25, grouped);
                CHECK(a.slices >= 1 && static_cast<long long>(a.slices) * buckets * finish_threads(buckets) <= kMaxGridThreads);
                CHECK(a.slices == 1 || a.slices * static_cast<long long>(a.per_slice) >= most);
            }
    CHECK(sliced(4096, 161, 100'000).slices == 1 && sliced(9216, 161, 100'000).slices == 3 && sliced(9216, 171, 100'000).slices == 1);
    // two or three only where they pay: not for little more than 4096 records, nor beside too many others
    CHECK(sliced(5632, 1, 5640).slices == 1 && sliced(5633, 1, 5640).slices > 1 && sliced(7168, 65, 9000).slices == 1);
    CHECK(sliced(7169, 65, 9000).slices == 2 && sliced(7169, 255, 9000).slices == 2 && sliced(7169, 256, 9000).slices == 1);
    CHECK(sliced(5633, 769, 9000).slices == 2 && sliced(12'288, 1536, 20'000).slices == 3 && sliced(12'288, 1537, 20'000).slices == 1);
    CHECK(sliced(12'289, 48, 100'000).slices == 4);
    CHECK(sliced(12'288, 1, 12'290).slices == 12 && sliced(12'288, 1, 12'290).per_slice == 1024);
    CHECK(sliced(273'438, 8, 2'187'504).slices == 64 && sliced(273'438, 8, 2'187'504).per_slice == 4280);
    return 0;
}

// The norms pass works in groups of tiles only where nearly all groups lie inside one bucket.
static int norms()
{
    const long long line = 50'331'648 / 256;
    CHECK(norms_grouped(line, 1) && !norms_grouped(line - 1, 1));
    CHECK(norms_grouped(line, static_cast<int>(line / 128)) && !norms_grouped(line, static_cast<int>(line / 128) + 1));
    for (long long elements : {4ll << 20, 16ll << 20, 64ll << 20, 1ll << 30, 1ll << 33})
        for (long long bucket : {64, 512, 3000, 10'000, 30'000})
            CHECK(!norms_grouped(elements / 256, static_cast<int>(elements / bucket)));
    CHECK(!norms_grouped(8, 1) && norms_grouped(1ll << 25, 1 << 18));
    return 0;
}

// A workgroup per bucket: up to 16384 elements, beyond 4096 not where most buckets are tiny, and no more behind a bucket's
// last lane-vector than its workgroup of at least 256 threads has lanes.
static int by_bucket()
{
    for (int n : {1, 512, 513, 1 << 21}) {
        CHECK(rate_by_bucket(0, 0, 0, n) && rate_by_bucket(4096, 256, 4096, n) && !rate_by_bucket(4096, 257, 1ll << 32, n));
        CHECK(rate_by_bucket(4097, 256, 1024ll * n, n) && rate_by_bucket(16384, 0, 1024ll * n, n));
        CHECK(rate_by_bucket(4097, 0, 1024ll * n - 1, n) == (n <= 512) && !rate_by_bucket(16385, 0, 1ll << 32, n));
    }
    CHECK(!rate_by_bucket(4, 0, 1ll << 32, (1 << 21) + 1));
    return 0;
}

// Bytes by the type of each stream; what fills the list up moves nothing.
static int bytes()
{
    SlotArgs s{};
    auto push = [&s](unsigned long long tag) { s.slot[s.h.n_sum + s.h.n_copy] = 0x10000ull * (s.h.n_sum + s.h.n_copy + 1) | tag; };
    for (unsigned tag : {0u + kAdd, 0u + kHold, kPair + 0u + kSlotBf16, kAdd + 0u + kSlotBf16, 0u + kSkip}) {
        push(tag);
        ++s.h.n_sum;
    }
    CHECK(round_bytes(s, true) == 2 * 4 + 2 * 2 + 16 && round_bytes(s, false) == 2 * 4 + 2 * 2 + 4);
    for (unsigned tag : {kSkip + 0u + kSlotCopy, kSkip + 0u + kSlotCopy + kSlotBf16}) {
        push(tag);
        ++s.h.n_copy;
    }
    CHECK(round_bytes(s, true) == 12 + 8 + 6 + 16);
    // the line between the two forms of a round, with and without what shortens its bursts
    s.h.n = (112ll << 20) / 42;
    CHECK(small_round(s, 42));
    ++s.h.n;
    CHECK(!small_round(s, 42));
    SlotArgs f{};
    f.slot[0] = f.slot[1] = 0x10000 | kAdd;
    f.h.n_sum = 2;
    f.h.n = (96ll << 20) / 24;
    CHECK(small_round(f, 24));
    ++f.h.n;
    CHECK(!small_round(f, 24) && small_round(f, 12));
    f.slot[0] |= kSlotBf16;
    f.slot[1] |= kSlotBf16;
    f.h.n = (56ll << 20) / 20;
    CHECK(small_round(f, 20));
    ++f.h.n;
    CHECK(!small_round(f, 20));
    return 0;
}

// The burst kernel's occupancy: a count that the LDS cap can realise, for every list and length, and
// more for short lists with copies and for bf16 streams than for long fp32 ones.
static int occupancy()
{
    auto waves = [](int sums, int copies, bool bf16, long long tiles, bool stats, bool update, bool streamed) {
        SlotArgs s{};
        s.h.n_sum = sums;
        s.h.n_copy = copies;
        for (int k = 0; k < sums + copies; ++k)
            s.slot[k] = 0x10000ull * (k + 1) + (k < sums ? 0u + kAdd : kSkip + 0u + kSlotCopy) + (bf16 ? 0u + kSlotBf16 : 0u);
        return burst_waves(s, tiles, stats, update, streamed);
    };
    for (int sums = 0; sums <= 128; sums += 2)
        for (int copies = 0; copies <= 63 && sums + copies <= 128; copies += copies < 8 ? 1 : 5)
            for (long long tiles : {0ll, 1ll, 4097ll, 8192ll, 19'532ll, 62'500ll, 100'000ll, 262'144ll, 6'000'000ll, 1ll << 25})
                for (int flags = 0; flags < 16; ++flags) {
                    const int w = waves(sums, copies, flags & 1, tiles, flags & 2, flags & 4, flags & 8);
                    CHECK(w == -1 || (w >= 10 && w <= 25 && kLdsUnits / (kLdsUnits / w) == w));
                    CHECK(w == -1 || w * kCus < tiles);
                }
    const long long many = 1ll << 22;
    CHECK(waves(16, 0, false, many, false, true, true) == 14 && waves(12, 4, false, many, false, true, true) == 12);
    CHECK(waves(4, 1, false, many, false, true, true) == 18 && waves(4, 3, false, many, false, true, true) == 14);
    CHECK(waves(16, 0, true, many, false, true, true) == 25 && waves(16, 0, true, many, false, false, true) == -1);
    CHECK(waves(16, 0, false, many, true, true, true) == 16);
    return 0;
}

// One element to a lane: short runs of long lists without by-products, and only where the number of loads in
// flight is the library's to choose.
static int narrow()
{
    for (int bf16 = 0; bf16 < 2; ++bf16) {
        auto is = [bf16](long long n, int slots, int copies, bool stats, int chunk) {
            return chunk_narrow(n, slots, copies, bf16 != 0, stats, chunk);
        };
        CHECK(is(1, 9, 0, false, 0) && is(1 << 17, 128, 40, false, 0) && is(1 << 15, 128, 63, false, 0));
        CHECK(is(1 << 16, 128, 63, false, 0) != bf16 && is(1 << 17, 95, 47, false, 0) != bf16);
        CHECK(!is((1 << 17) + 1, 128, 0, false, 0) && !is(64, 8, 0, false, 0) && !is(64, 9, 0, true, 0));
        for (int chunk : {8, 16}) CHECK(!is(1, 9, 0, false, chunk) && !is(1 << 17, 128, 0, false, chunk));
    }
    return 0;
}

// A copy's store waits for the one before it: one chunk of many copies, a run that streams and is resident at once.
static int paced()
{
    CHECK(resident_waves(99) == 16 && resident_waves(96) == 20 && resident_waves(92) == 20 && resident_waves(50) == 32);
    CHECK(resident_waves(0) == 0 && resident_waves(80) == 24 && resident_waves(72) == 28);
    auto is = [](int sums, int copies, bool bf16, bool update, long long n, int resident = 20) {
        SlotArgs s{};
        s.h.n = n;
        s.h.n_sum = sums;
        s.h.n_copy = copies;
        for (int k = 0; k < sums + copies; ++k)
            s.slot[k] = 0x10000ull * (k + 1) + (k < sums ? 0u + kAdd : kSkip + 0u + kSlotCopy) + (bf16 && k >= sums ? 0u + kSlotBf16 : 0u);
        return chunk_paced(s, sums + copies, bf16, update, resident);
    };
    const long long streams = (56ll << 20) / (32 + 7 * 6 + 16) + 1, resident = 20 * 256 * 256;
    CHECK(is(8, 7, true, true, streams) && !is(8, 7, true, true, streams - 1));
    CHECK(is(8, 7, true, true, resident) && !is(8, 7, true, true, resident + 1) && is(8, 7, false, false, resident));
    CHECK(is(6, 5, true, true, 1 << 20) && !is(6, 5, false, true, 1 << 20) && !is(6, 4, true, true, 1 << 20));
    CHECK(is(9, 7, true, true, 1 << 20) && !is(10, 7, true, true, 1 << 20));
    CHECK(is(8, 7, true, true, 1 << 20, 16) && !is(8, 7, true, true, (1 << 20) + 1, 16) && !is(8, 7, true, true, 1 << 20, 0));
    return 0;
}

// Weight views: a cap from 6 tiles per CU on (updates of more than 24 views:
// always), and an average of few views or of views that the caches just hold past them.
static int views()
{
    const long long line = 6ll * 256 * 256;
    for (int n_views = 1; n_views <= 64; ++n_views)
        for (long long n : {1ll, 255ll, line, line + 4, 1ll << 20, 1ll << 33}) {
            const int update = views_sgd_waves(n_views, n), average = views_average_waves(n_views, n);
            CHECK((update == -1) == (n <= line && n_views <= 24) && (average == -1) == (n <= line || n_views == 1));
            for (int w : {update, average}) CHECK(w == -1 || (w >= 2 && w <= 16));
        }
    CHECK(views_tiles(1) == 1 && views_tiles(256) == 1 && views_tiles(260) == 2);
    for (int n_views : {17, 23, 24, 64}) {
        CHECK(views_average_waves(n_views, (1 << 20) - 1) == 4 && views_average_waves(n_views, 1 << 20) == (n_views < 24 ? 4 : 3));
        CHECK(views_sgd_waves(n_views, 1 << 20) == 2);
    }
    CHECK(views_average_waves(12, 1 << 25) == 3 && views_average_waves(16, 1 << 25) == 3 && views_average_waves(11, 1 << 25) == 4);
    CHECK(views_sgd_waves(8, 1 << 25) == 2 && views_sgd_waves(9, 1 << 25) == 3 && views_sgd_waves(12, 1 << 25) == 3 && views_sgd_waves(13, 1 << 25) == 2);
    for (int n_views : {1, 3, 4, 8, 9, 64}) {
        const long long most = kPlainRoundBytes / 8 / n_views, held = (((n_views == 4 ? 32ll : 28ll) << 20) - 1) / 8 / n_views;
        CHECK(views_average_streamed(n_views, most + 1) && views_average_streamed(n_views, most) == (n_views < 4));
        CHECK(views_average_streamed(n_views, held) == (n_views <= 8) && views_average_streamed(n_views, held + 1) == (n_views < 4));
    }
    return 0;
}

// Short lists that chunk_kernel keeps: copies stored one at a time, bf16 in any order with 8 streams and four elements to a lane,
// bf16 in fixed order with 4 send buffers among many streams and one element to a lane.
static int short_lists()
{
    auto is = [](int pending, int grads, int copies, bool bf16, bool fast, long long n, bool nt = false, bool update = true) {
        SlotArgs s{};
        s.h.n = n;
        int k = 0;
        auto push = [&](unsigned long long tag) {
            s.slot[k] = 0x10000ull * (k + 1) | tag;
            ++k;
        };
        const unsigned long long type = bf16 ? kSlotBf16 + 0ull : 0ull;
        for (int j = 0; j < pending; ++j) push(kAdd);
        for (int j = 0; j < grads; ++j) push(kAdd | type);
        if (k % kBurst) push(kSkip);
        s.h.n_sum = k;
        s.h.n_copy = copies;
        for (int j = 0; j < copies; ++j) push(kSkip | kSlotCopy | type);
        return short_round(s) && short_pays(s, bf16, fast, nt, update);
    };
    const long long wide = (1 << 17) + 1;
    for (bool fast : {false, true}) {
        CHECK(is(8, 8, 0, false, fast, 64) && is(8, 8, 0, false, fast, wide) && is(0, 1, 7, false, fast, 1 << 20));
        CHECK(!is(0, 1, 7, false, fast, 1'060'000, true) && is(0, 3, 5, false, fast, 1'060'000, true));
        CHECK(!is(0, 1, 7, true, fast, 1'300'000, true) && is(0, 1, 8, true, fast, 64) && !is(0, 1, 9, true, fast, 64));
        CHECK(is(2, 4, 5, true, fast, 64) && is(4, 4, 0, true, fast, 64) && is(4, 8, 0, true, fast, 64));
    }
    CHECK(!is(8, 8, 0, true, false, 64) && !is(4, 12, 0, true, false, 1 << 17) && !is(4, 4, 4, true, false, 64) && !is(4, 1, 8, true, false, 64));
    CHECK(is(3, 13, 0, true, false, 64) && is(8, 8, 0, true, false, wide) && is(8, 8, 0, true, true, 64));
    CHECK(!is(0, 8, 0, true, true, wide) && is(0, 7, 0, true, true, wide) && is(0, 8, 0, true, false, wide));
    return 0;
}

int main()
{
    if (short_lists() || views() || lanes() || back() || paced() || narrow() || grids() || finishing() || slices() || norms() || by_bucket() || bytes() || occupancy()) return 1;
    std::printf("ok\n");
    return 0;
}
