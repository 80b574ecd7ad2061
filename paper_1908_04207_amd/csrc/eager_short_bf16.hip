// short_kernel with bf16 gradients.
#include "eager_short.h"

namespace eager {

hipError_t launch_short_bf16(const SlotArgs &s, bool nt, hipStream_t st)
{
    return launch_short<true, false>(s, nt, st);
}

}  // namespace eager
