// Tangent-pass adjoint, FP64 network, general widths; also the choice of the
// width's form.
#include "k_tangent_adj_impl.h"

namespace pn {
template size_t tangent_adj_ops_bytes<double>(const Dims&, int, int64_t);
template size_t tangent_adj_lds_bytes<double>(const Dims&, int, bool);
template void launch_net_tangent_adj_w<double, 0>(const pn_ctx*, hipStream_t, int64_t, const double*, const double*,
                                                  char*, const WsLayout&);

// Widths with a form of their own (instantiated in their translation units).
#define PN_WIDTH(TN, SX)                                                                                         \
  extern template void launch_net_tangent_adj_w<TN, SX>(const pn_ctx*, hipStream_t, int64_t, const double*, const TN*, \
                                                        char*, const WsLayout&)
PN_WIDTH(float, 0);
PN_WIDTH(float, 64);
PN_WIDTH(float, 128);
PN_WIDTH(double, 64);
PN_WIDTH(double, 128);
#undef PN_WIDTH

template <typename TN>
void launch_net_tangent_adj(const pn_ctx* c, hipStream_t s, int64_t nw, const double* r, const TN* P, char* ws,
                            const WsLayout& L) {
  const int sx = 2 * c->d.DZ == c->d.DX ? c->d.DX : 0;
  if (sx == 64)
    launch_net_tangent_adj_w<TN, 64>(c, s, nw, r, P, ws, L);
  else if (sx == 128)
    launch_net_tangent_adj_w<TN, 128>(c, s, nw, r, P, ws, L);
  else
    launch_net_tangent_adj_w<TN, 0>(c, s, nw, r, P, ws, L);
}
template void launch_net_tangent_adj<float>(const pn_ctx*, hipStream_t, int64_t, const double*, const float*, char*,
                                            const WsLayout&);
template void launch_net_tangent_adj<double>(const pn_ctx*, hipStream_t, int64_t, const double*, const double*, char*,
                                             const WsLayout&);
}  // namespace pn
