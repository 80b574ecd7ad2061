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

int main()
{
    if (grids()) return 1;
    std::printf("ok\n");
    return 0;
}
