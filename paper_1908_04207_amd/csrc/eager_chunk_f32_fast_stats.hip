// chunk_kernel with fp32 gradients in any order and by-products.
#include "eager_chunk.h"

namespace eager {

hipError_t launch_chunk_f32_fast_stats(const SlotArgs &s, bool nt, bool nts, bool eight, int bpc, const Launch &cfg, hipStream_t st)
{
    return launch_kind<false, true, true>(s, nt, nts, eight, bpc, cfg, st);
}

}  // namespace eager
