// 4-bit forms of the register-resident streaming kernel.
#include "stream_direct_w4.hpp"

namespace quasar {

int launch_direct_w4(int epi, const GemmParams &base, int MP, const DirectPlan &d, hipStream_t stream) {
    GemmParams p = base;
    p.S = p.K / kStepK4;
    p.ksplit = 1;
    share_tiles(p, d.groups, 1, 1);
    return epi == EPI_ARGMAX ? launch_w4_as<EPI_ARGMAX>(p, MP, d, stream) : launch_w4_as<EPI_LINEAR>(p, MP, d, stream);
}

}  // namespace quasar
