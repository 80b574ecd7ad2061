// short_kernel with bf16 gradients, the sum in any order.
#include "eager_short.h"

namespace eager {

hipError_t launch_short_bf16_fast(const SlotArgs &s, bool nt, hipStream_t st)
{
    return launch_short<true, true>(s, nt, st);
}

}  // namespace eager
