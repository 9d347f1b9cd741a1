// Int8-weight forms of the register-resident streaming kernel.
#include "stream_direct.hpp"

namespace quasar {

int launch_direct_int8(int epi, int pre, bool resid, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) {
    if (epi == EPI_ARGMAX) return launch_direct_as<false, EPI_ARGMAX, PRE_NONE, false>(p, MP, d, stream);
    if (epi == EPI_LOGITS) return launch_direct_as<false, EPI_LOGITS, PRE_NONE, false>(p, MP, d, stream);
    if (epi == EPI_SWIGLU)
        return pre == PRE_RMSNORM ? launch_direct_as<false, EPI_SWIGLU, PRE_RMSNORM, false>(p, MP, d, stream)
                                  : launch_direct_as<false, EPI_SWIGLU, PRE_NONE, false>(p, MP, d, stream);
    if (pre == PRE_RMSNORM)
        return resid ? launch_direct_as<false, EPI_LINEAR, PRE_RMSNORM, true>(p, MP, d, stream)
                     : launch_direct_as<false, EPI_LINEAR, PRE_RMSNORM, false>(p, MP, d, stream);
    return resid ? launch_direct_as<false, EPI_LINEAR, PRE_NONE, true>(p, MP, d, stream)
                 : launch_direct_as<false, EPI_LINEAR, PRE_NONE, false>(p, MP, d, stream);
}

}  // namespace quasar
