// chunk_kernel with fp32 gradients.
#include "eager_chunk.h"

namespace eager {

hipError_t launch_chunk_f32(const SlotArgs &s, bool nt, bool nts, bool eight, int bpc, const Launch &cfg, hipStream_t st)
{
    return launch_kind<false, false, false>(s, nt, nts, eight, bpc, cfg, st);
}

}  // namespace eager
