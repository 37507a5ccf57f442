// Network tangent pass, F32 network, embedding width 128 (also the BF16-operand form).
#include "k_tangent_impl.h"

namespace pn {
template void launch_net_tangent_w<float, 128>(const pn_ctx*, hipStream_t, int64_t, const double*, const float*,
                                            char*, const WsLayout&, bool, float*);
}  // namespace pn
