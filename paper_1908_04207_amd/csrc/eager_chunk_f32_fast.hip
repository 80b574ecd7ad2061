// chunk_kernel with fp32 gradients in any order.
#include "eager_chunk.h"

namespace eager {

hipError_t launch_chunk_f32_fast(const SlotArgs &s, bool nt, bool nts, bool eight, int bpc, const Launch &cfg, hipStream_t st)
{
    return launch_kind<false, true, false>(s, nt, nts, eight, bpc, cfg, st);
}

}  // namespace eager
