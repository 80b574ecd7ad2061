// short_kernel with fp32 gradients, the sum in any order.
#include "eager_short.h"

namespace eager {

hipError_t launch_short_f32_fast(const SlotArgs &s, bool nt, hipStream_t st)
{
    return launch_short<false, true>(s, nt, st);
}

}  // namespace eager
