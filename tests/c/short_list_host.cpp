// The list of short_kernel (fill_short of csrc/eager_rules.h) on the CPU: random rounds of up to 16 streams, worked through
// slot by slot and, from the list, as the kernel does; built and run by tests/test_launch_rules.py.
#include "../../paper_1908_04207_amd/csrc/eager_rules.h"

#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

using namespace eager;

static float at(unsigned long long address, bool bf)      // some number that belongs to an address
{
    return static_cast<float>(static_cast<int>(address * 2654435761u >> 7 & 0xffffff) - 0x800000) * (bf ? 1e-3f : 1e-6f);
}
typedef std::vector<std::pair<float *, float>> Copies;

template <int SLOTS>
static bool same(const SlotArgs &s, bool fast, float want, const Copies &copies)
{
    ShortArgs<SLOTS> a;
    std::memset(static_cast<void *>(&a), 0xff, sizeof a);
    fill_short(s, fast, kPaced, a);
    std::vector<float> x(SLOTS, 1e30f);
    const int n_sum = a.shape & 255, n_last = a.shape >> 8 & 255;
    auto load = [&](int j) { x[j] = at(a.slot[j], a.bits >> (16 + j) & 1); };
    if (SLOTS == 16)
        for (int j = 0; j < 8 && j < n_sum; ++j) load(j);
    for (int j = 0; j < n_last; ++j) load(a.kHalf + j);
    Copies got;
    for (int j = 0; j < SLOTS; ++j)
        if (a.copies >> j & 1) {
            if (j < a.kHalf || j < n_sum) return false;
            got.push_back({a.dst[j - a.kHalf], x[j]});
        }
    float s1 = 0.0f, part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int j = 0; j < n_sum; ++j) part[(a.bits >> (16 + j) & 1 ? 2 : 0) + (j & 1)] += x[j];
    for (int j = 1; j < SLOTS; ++j)
        if (a.bits >> j & 1) {
            if (j >= n_sum) return false;
            x[j] = x[j - 1] + x[j];
            x[j - 1] = 0.0f;
        }
    for (int j = 0; j < n_sum; ++j) s1 = s1 + x[j];
    const float sum = fast ? (part[0] + part[1]) + (part[2] + part[3]) : s1;
    const bool w = a.w == (s.h.w ? s.h.w + s.h.e0 : nullptr);
    return w && a.n == s.h.n && !std::memcmp(&sum, &want, 4) && got == copies && (a.shape >> kShortForm & 3) == kPaced &&
           (a.shape >> 16 & 1) == (s.h.nesterov ? 1u : 0u) && a.shape >> kShortSkip == static_cast<unsigned>(s.h.skip) * 4;
}

int main()
{
    std::mt19937_64 rng(7);
    int seen = 0;
    for (int trial = 0; trial < 40000; ++trial) {
        const int P = 1 + static_cast<int>(rng() % 18);
        const bool bf16 = rng() & 1, fast = rng() & 1, stores = rng() & 1;
        const unsigned long long active = rng(), valid = rng() & (rng() % 3 ? ~0ull : rng());
        SlotArgs s;
        std::memset(static_cast<void *>(&s), 0, sizeof s);
        s.h.e0 = static_cast<long long>(rng() % 1000) * 64;
        s.h.n = 1 + static_cast<long long>(rng() % 100000);
        s.h.skip = static_cast<int>(rng() % 16);
        s.h.nesterov = rng() & 1;
        s.h.w = rng() & 1 ? reinterpret_cast<float *>(0x7000000ull) : nullptr;
        auto base = [](int p, bool r) { return 0x10000000ull * (p + 1) + (r ? 0x8000000ull : 0); };
        auto value = [&](int p, bool r) {
            const bool bf = !r && bf16;
            return at(base(p, r) + s.h.e0 * (bf ? 2 : 4), bf);
        };
        int n = 0;
        float sum = 0.0f, part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int p = 0; p < P; ++p) {
            const bool on = active >> p & 1, r = valid >> p & 1;
            if (r) s.slot[n++] = base(p, true) | (on ? kHold : kAdd);
            if (on) s.slot[n++] = base(p, false) | (r ? kPair : kAdd) | (bf16 ? kSlotBf16 : 0u);
            if (r && on) sum = sum + (value(p, true) + value(p, false));
            else if (r || on) sum = sum + value(p, r);
        }
        int m = 0;
        for (int type = 0; type < 2; ++type)
            for (int k = 0; k < n; ++k)
                if (((s.slot[k] & kSlotBf16) != 0) == (type != 0))
                    part[2 * type + (m++ & 1)] += at((s.slot[k] & ~static_cast<unsigned long long>(kSlotTag)) + s.h.e0 * (type ? 2 : 4), type != 0);
        while (n % kBurst) s.slot[n++] = 0x10000000ull | kSkip;
        s.h.n_sum = n;
        Copies copies;
        for (int p = 0; stores && p < P; ++p)
            if (!(active >> p & 1)) {
                s.dst[n] = reinterpret_cast<float *>(base(p, true));
                s.slot[n++] = base(p, false) | kSkip | kSlotCopy | (bf16 ? kSlotBf16 : 0u);
                ++s.h.n_copy;
                copies.push_back({s.dst[n - 1] + s.h.e0, value(p, false)});
            }
        if (!short_round(s)) continue;
        ++seen;
        const float want = fast ? (part[0] + part[1]) + (part[2] + part[3]) : sum;
        const bool eight = sum_terms(s) + s.h.n_copy <= 8;
        if ((eight && !same<8>(s, fast, want, copies)) || !same<16>(s, fast, want, copies)) {
            std::printf("trial %d: P %d\n", trial, P);
            return 1;
        }
    }
    std::printf(seen > 10000 ? "ok\n" : "too few\n");
    return 0;
}
