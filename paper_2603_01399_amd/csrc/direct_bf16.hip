// Bf16-weight forms of the register-resident streaming kernel.
#include "stream_direct.hpp"

namespace quasar {

int launch_direct_bf16(int epi, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) {
    if (epi == EPI_ARGMAX) return launch_direct_as<true, EPI_ARGMAX, PRE_NONE, false>(p, MP, d, stream);
    return launch_direct_as<true, EPI_LINEAR, PRE_NONE, false>(p, MP, d, stream);
}

}  // namespace quasar
