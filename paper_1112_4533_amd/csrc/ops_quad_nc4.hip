// The four-lanes-per-link phase kernels of SU(4).
#include "sun_quad.hpp"

namespace sun {
template <>
void launch_update_quad<4, float, 4>(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1,
                                     uint32_t step) {
    quad::launch<4, float, 4>(c, kind, mu, par, beta, k0, k1, step);
}
template <>
void launch_update_quad<4, double, 4>(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1,
                                      uint32_t step) {
    quad::launch<4, double, 4>(c, kind, mu, par, beta, k0, k1, step);
}
}  // namespace sun
