// Tangent-pass adjoint, FP32 network (also the BF16-operand form, whose
// adjoint products run in FP32), general widths.
#include "k_tangent_adj_impl.h"

namespace pn {
template size_t tangent_adj_ops_bytes<float>(const Dims&, int, int64_t);
template size_t tangent_adj_lds_bytes<float>(const Dims&, int, bool);
template void launch_net_tangent_adj_w<float, 0>(const pn_ctx*, hipStream_t, int64_t, const double*, const float*,
                                                 char*, const WsLayout&);
}  // namespace pn
