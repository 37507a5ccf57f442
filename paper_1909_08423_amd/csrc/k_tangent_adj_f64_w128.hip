// Tangent-pass adjoint, F64 network, embedding width 128.
#include "k_tangent_adj_impl.h"

namespace pn {
template void launch_net_tangent_adj_w<double, 128>(const pn_ctx*, hipStream_t, int64_t, const double*,
                                                const double*, char*, const WsLayout&);
}  // namespace pn
