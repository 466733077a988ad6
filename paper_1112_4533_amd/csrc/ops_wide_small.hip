// ops_wide_small.hip -- launchers of the four-links-per-wavefront update
// (4 <= Nc <= 8 of the large-Nc path), one kernel per Nc and precision.
#include "sun_ops.hpp"
#include "sun_wide_small.hpp"

namespace sun {
namespace {

template <typename T, int N>
void launch(const Ctx& c, int hb, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step) {
    wide::k_update_small<T, N><<<wide_update_tiles(c.nc, c.g.Vh), wide::kLanes, wide::small_lds<T, N>(), c.stream>>>(
        (T2<T>*)c.links, c.g, mu, par, hb, (T)beta, k0, k1, step);
}
template <typename T, int N>
void launch_batch(const ChainDesc* d, int n, int tiles, int hb, int mu, int par, uint32_t off, hipStream_t s) {
    wide::k_update_small_batch<T, N><<<tiles, wide::kLanes, wide::small_lds<T, N>(), s>>>(d, n, mu, par, hb, off);
}

}  // namespace

template <typename T>
void launch_update_small(const Ctx& c, int hb, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step) {
    switch (c.nc) {
        case 4: launch<T, 4>(c, hb, mu, par, beta, k0, k1, step); break;
        case 5: launch<T, 5>(c, hb, mu, par, beta, k0, k1, step); break;
        case 6: launch<T, 6>(c, hb, mu, par, beta, k0, k1, step); break;
        case 7: launch<T, 7>(c, hb, mu, par, beta, k0, k1, step); break;
        default: launch<T, 8>(c, hb, mu, par, beta, k0, k1, step); break;
    }
}
template <typename T>
void launch_update_small_batch(const ChainDesc* d, int n, int tiles, int hb, int mu, int par, uint32_t off, int nc,
                               hipStream_t s) {
    switch (nc) {
        case 4: launch_batch<T, 4>(d, n, tiles, hb, mu, par, off, s); break;
        case 5: launch_batch<T, 5>(d, n, tiles, hb, mu, par, off, s); break;
        case 6: launch_batch<T, 6>(d, n, tiles, hb, mu, par, off, s); break;
        case 7: launch_batch<T, 7>(d, n, tiles, hb, mu, par, off, s); break;
        default: launch_batch<T, 8>(d, n, tiles, hb, mu, par, off, s); break;
    }
}

template void launch_update_small<float>(const Ctx&, int, int, int, double, uint32_t, uint32_t, uint32_t);
template void launch_update_small<double>(const Ctx&, int, int, int, double, uint32_t, uint32_t, uint32_t);
template void launch_update_small_batch<float>(const ChainDesc*, int, int, int, int, int, uint32_t, int, hipStream_t);
template void launch_update_small_batch<double>(const ChainDesc*, int, int, int, int, int, uint32_t, int, hipStream_t);

static_assert(wide::kSmallMax == kWideSmallMax && wide::kSmallLinks == kWideSmallLinks, "host and device agree");

}  // namespace sun
