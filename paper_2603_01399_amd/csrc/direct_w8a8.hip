// W8A8 forms of the register-resident streaming kernel.
#include "stream_direct_a8.hpp"

namespace quasar {

int launch_direct_w8a8(int epi, const GemmParams &base, int MP, const DirectPlan &d, hipStream_t stream) {
    GemmParams p = base;
    p.S = p.K / 64;
    p.sc_bytes = d.sc_bytes;
    share_tiles(p, d.groups, 1, 1);
    if (epi == EPI_ARGMAX && p.dx) return launch_a8_codes<1, 2, 3, 4, 5, 6>(d.XS, d.groups, d.lds_bytes, stream, p);
    if (epi == EPI_ARGMAX)
        return p.smooth ? launch_a8_as<EPI_ARGMAX, true>(p, MP, d, stream) : launch_a8_as<EPI_ARGMAX, false>(p, MP, d, stream);
    return p.smooth ? launch_a8_as<EPI_LINEAR, true>(p, MP, d, stream) : launch_a8_as<EPI_LINEAR, false>(p, MP, d, stream);
}

}  // namespace quasar
