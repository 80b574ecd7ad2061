// short_kernel with fp32 gradients.
#include "eager_short.h"

namespace eager {

hipError_t launch_short_f32(const SlotArgs &s, bool nt, hipStream_t st)
{
    return launch_short<false, false>(s, nt, st);
}

}  // namespace eager
