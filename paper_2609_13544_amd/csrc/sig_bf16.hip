// Pass 1 of the error signature for bf16 pairs.
#include "sig_chunk.h"

namespace peat {

hipError_t launch_sig_bf16(const SigParams &p, int64_t n, const InjDesc *inj, hipStream_t s) {
    return inj ? launch_kind_inject<PEAT_BF16>(p, n, inj, s) : launch_kind<PEAT_BF16, PEAT_BF16>(p, n, s);
}

}  // namespace peat
