// Tangent-pass adjoint, F32 network, embedding width 128.
#include "k_tangent_adj_impl.h"

namespace pn {
template void launch_net_tangent_adj_w<float, 128>(const pn_ctx*, hipStream_t, int64_t, const double*,
                                                const float*, char*, const WsLayout&);
}  // namespace pn
