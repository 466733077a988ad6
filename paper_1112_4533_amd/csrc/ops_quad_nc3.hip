// The four-lanes-per-link phase kernels of SU(3).
#include "sun_quad.hpp"

namespace sun {
template <>
void launch_update_quad<3, float, 3>(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1,
                                     uint32_t step) {
    quad::launch<3, float, 3>(c, kind, mu, par, beta, k0, k1, step);
}
template <>
void launch_update_quad<3, double, 3>(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1,
                                      uint32_t step) {
    quad::launch<3, double, 3>(c, kind, mu, par, beta, k0, k1, step);
}
}  // namespace sun
