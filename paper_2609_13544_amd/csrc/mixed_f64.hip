// Pass 1 of the error signature for mixed-precision pairs with a binary64 test
// side (Section III-C: the FP32-FP64 error unit).
#include "sig_chunk.h"

namespace peat {

hipError_t launch_sig_mixed_f64(const SigParams &p, int kind, int64_t n, hipStream_t s) {
    static_assert(kKindTypes[3][1] == PEAT_F64 && kKindTypes[9][0] == PEAT_BF16, "kind table order");
    switch (kind) {
        case 3: return launch_kind<PEAT_F32, PEAT_F64>(p, n, s);
        case 8: return launch_kind<PEAT_F16, PEAT_F64>(p, n, s);
        case 9: return launch_kind<PEAT_BF16, PEAT_F64>(p, n, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace peat
