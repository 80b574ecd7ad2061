// chunk_kernel with bf16 gradients.
#include "eager_chunk.h"

namespace eager {

hipError_t launch_chunk_bf16(const SlotArgs &s, bool nt, bool nts, bool eight, int bpc, const Launch &cfg, hipStream_t st)
{
    return launch_kind<true, false, false>(s, nt, nts, eight, bpc, cfg, st);
}

}  // namespace eager
