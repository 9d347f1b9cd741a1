// w4 forms of the streaming kernel with K outermost.
#include "stream_outer.hpp"

namespace quasar {

int launch_outer_w4(const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) { return launch_outer_as<FMT_W4>(p, MP, d, stream); }

}  // namespace quasar
