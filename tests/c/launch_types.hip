// The launch helpers of csrc/eager_device.h take a kernel with arguments of its own types only: compiled (host pass, no
// code) by tests/test_launch_rules.py, as it stands and with each WRONG, which must not compile.
#include "../../paper_1908_04207_amd/csrc/eager_device.h"

namespace eager {

__global__ void takes_sgd(const SgdArgs) {}
__global__ void takes_two(const SgdArgs, const StatsArgs) {}
__global__ void takes_long(const ChunkArgs<kMaxSlots, kMaxP, false>) {}

hipError_t launches(const SgdArgs &a, const StatsArgs &st, const ChunkArgs<kMaxSlots, kMaxP, false> &chunk,
                    const ChunkArgs<kChunkFewSlots, kChunkFewCopies, false> &few, hipStream_t stream)
{
    Launch cfg;
    (void)few;
#if WRONG == 1        // a second argument that the kernel would read past the array of addresses
    return launch_capped(takes_two, a, -1, cfg, dim3(1), stream);
#elif WRONG == 2      // a block of another size
    return launch_capped(takes_long, few, -1, cfg, dim3(1), stream);
#elif WRONG == 3
    return launch(takes_two, dim3(1), dim3(64), 0, stream, st, a);
#else
    hipError_t e = launch_capped(takes_sgd, a, -1, cfg, dim3(1), stream);
    if (e == hipSuccess) e = launch_capped(takes_long, chunk, -1, cfg, dim3(1), stream);
    return e == hipSuccess ? launch(takes_two, dim3(1), dim3(64), 0, stream, a, st) : e;
#endif
}

}  // namespace eager
