// The list of chunk_kernel (fill_chunk of csrc/eager_rules.h) on the CPU: random rounds are worked through
// slot by slot and, from the list, in chunks as the kernel takes them; built and run by
// tests/test_launch_rules.py.
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

// in chunks of CH, pairs across them by the held value, or in any order two sums of fp32 streams in
// turn and two of bf16 streams; the copies as (destination, source)
template <typename A>
static float by_chunks(const A &a, int CH, bool fast, std::vector<std::pair<float *, float>> &copies)
{
    float s = 0.0f, s2 = 0.0f, s3 = 0.0f, s4 = 0.0f, held = 0.0f;
    for (int k0 = 0; k0 < a.h.n_slots; k0 += CH) {
        std::vector<float> x(CH, 1e30f);
        auto bit = [&](unsigned ChunkBits::*m, int j) { return a.bits[(k0 + j) / kChunkWord].*m >> (k0 + j) % kChunkWord & 1u; };
        for (int j = 0; j < CH && k0 + j < a.h.n_slots; ++j) x[j] = at(a.slot[k0 + j], bit(&ChunkBits::bf, j));
        const int sums = a.h.n_sum - k0;
        for (int j = 0; !fast && j < CH && k0 + j < A::kSlots; ++j)
            if (bit(&ChunkBits::pair, j)) {
                float &before = j ? x[j - 1] : held;
                x[j] = before + x[j];
                before = 0.0f;
            }
        if (!fast && sums > CH && bit(&ChunkBits::hold, CH - 1)) {
            held = x[CH - 1];
            x[CH - 1] = 0.0f;
        }
        for (int j = 0; j < CH && j < sums; ++j) {
            float &part = !fast ? s : bit(&ChunkBits::bf, j) ? (j & 1 ? s4 : s3) : j & 1 ? s2 : s;
            part = part + x[j];
        }
        for (int j = 0; j < CH && k0 + j < A::kSlots; ++j)
            if (bit(&ChunkBits::copy, j)) {
                const int d = k0 + j - a.h.dst_first;
                if (d < 0 || d >= A::kCopies + 8) return 1e38f;
                copies.push_back({a.dst[d], x[j]});
            }
    }
    return fast ? (s + s2) + (s3 + s4) : s;
}

template <int SLOTS, int COPIES>
static bool same(const SlotArgs &s, bool fast, float sum, float in_turn, const std::vector<std::pair<float *, float>> &copies)
{
    ChunkArgs<SLOTS, COPIES, false> a;
    std::memset(static_cast<void *>(&a), 0xff, sizeof a);
    fill_chunk(s, fast, 512, 99, a);
    for (int CH : {8, 16, 32}) {
        std::vector<std::pair<float *, float>> got;
        const float t = by_chunks(a, CH, fast, got);
        if (std::memcmp(&t, fast ? &in_turn : &sum, 4) || got != copies) return false;
    }
    const bool w = a.h.w == (s.h.w ? s.h.w + s.h.e0 + 512 : nullptr);
    return w && a.h.n == 99 && !std::memcmp(&a.h.first, &a.bits[0], sizeof a.h.first);
}

int main()
{
    std::mt19937_64 rng(5);
    for (int trial = 0; trial < 4000; ++trial) {
        const int P = 1 + static_cast<int>(rng() % (trial % 2 ? 64 : 18));
        const bool bf16 = rng() & 1, fast = rng() & 1, stores = rng() & 1;
        const unsigned long long active = rng(), valid = rng() & (rng() % 3 ? ~0ull : rng());
        SlotArgs s;
        std::memset(static_cast<void *>(&s), 0, sizeof s);
        s.h.e0 = static_cast<long long>(rng() % 1000) * 8;
        s.h.w = rng() & 1 ? reinterpret_cast<float *>(0x7000000ull) : nullptr;
        auto base = [](int p, bool r) { return 0x10000000ull * (p + 1) + (r ? 0x8000000ull : 0); };
        int n = 0;
        float sum = 0.0f, term = 0.0f;
        auto value = [&](int p, bool r) {
            const bool bf = !r && bf16;
            return at(base(p, r) + (s.h.e0 + 512) * (bf ? 2 : 4), bf);
        };
        for (int p = 0; p < P; ++p) {
            const bool on = active >> p & 1, r = valid >> p & 1;
            if (r) s.slot[n++] = base(p, true) | (on ? kHold : kAdd);
            if (on) s.slot[n++] = base(p, false) | (r ? kPair : kAdd) | (bf16 ? kSlotBf16 : 0u);
            if (r && on) term = value(p, true) + value(p, false);
            else if (r || on) term = value(p, r);
            if (r || on) sum = sum + term;
        }
        float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};     // in any order: the fp32 streams in turn, then the bf16 streams
        int m = 0;
        for (int type = 0; type < 2; ++type) for (int k = 0; k < n; ++k) {
            const bool bf = (s.slot[k] & kSlotBf16) != 0;
            if (bf == (type != 0)) part[2 * type + (m++ & 1)] += at((s.slot[k] & ~static_cast<unsigned long long>(kSlotTag)) + (s.h.e0 + 512) * (bf ? 2 : 4), bf);
        }
        const float in_turn = (part[0] + part[1]) + (part[2] + part[3]);
        while (n % kBurst) s.slot[n++] = 0x10000000ull | kSkip;
        s.h.n_sum = n;
        std::vector<std::pair<float *, float>> copies;
        for (int p = 0; stores && p < P; ++p)
            if (!(active >> p & 1)) {
                s.dst[n] = reinterpret_cast<float *>(base(p, true));
                s.slot[n++] = base(p, false) | kSkip | kSlotCopy | (bf16 ? kSlotBf16 : 0u);
                ++s.h.n_copy;
                copies.push_back({s.dst[n - 1] + s.h.e0 + 512, value(p, false)});
            }
        const bool few = chunk_fits(s, kChunkFewSlots, kChunkFewCopies);
        if (!chunk_fits(s, kMaxSlots, kMaxP) && s.h.n_sum + s.h.n_copy > kMaxSlots + 1) return 1;
        if ((few && !same<kChunkFewSlots, kChunkFewCopies>(s, fast, sum, in_turn, copies)) ||
            !same<kMaxSlots, kMaxP>(s, fast, sum, in_turn, copies)) {
            std::printf("trial %d: P %d\n", trial, P);
            return 1;
        }
    }
    std::printf("ok\n");
    return 0;
}
