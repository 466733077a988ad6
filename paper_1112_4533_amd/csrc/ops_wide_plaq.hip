// ops_wide_plaq.hip -- launchers of the large-Nc plaquette.
#include "sun_ops.hpp"
#include "sun_wide_plaq.hpp"

namespace sun {
namespace {

// f(Nc) with Nc <= kWideSmallMax as a compile-time constant
template <typename F>
void with_small(int nc, F f) {
    switch (nc) {
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
        default: f(std::integral_constant<int, 8>{}); break;
    }
}

// f(form) for Nc > kWideSmallMax
template <typename F>
void with_form(int nc, F f) {
    if (nc <= wide::kTile)
        f(std::integral_constant<int, wide::PLAQ_ONE>{});
    else if (nc <= wide::kEdgeMax)
        f(std::integral_constant<int, wide::PLAQ_EDGES>{});
    else
        f(std::integral_constant<int, wide::PLAQ_FOUR>{});
}

}  // namespace

template <typename T>
void launch_plaquette_wide(const Ctx& c, double* partial) {
    const T2<T>* u = (const T2<T>*)c.links;
    const int tiles = wide_plaquette_tiles(c.nc, c.g.V);
    if (c.nc <= kWideSmallMax)
        with_small(c.nc, [&](auto n) {
            constexpr int N = decltype(n)::value;
            wide::k_plaquette_small<T, N><<<tiles, wide::kLanes, wide::plaq_small_lds<T, N>(), c.stream>>>(u, c.g,
                                                                                                           partial);
        });
    else
        with_form(c.nc, [&](auto form) {
            constexpr int F = decltype(form)::value;
            wide::k_plaquette_large<T, F><<<tiles, wide::plaq_threads(F), wide::plaq_large_lds<T>(c.nc), c.stream>>>(
                u, c.g, c.nc, partial);
        });
}
template <typename T>
void launch_plaquette_wide_batch(const ChainDesc* d, int n, int tiles, int nc, hipStream_t s) {
    if (nc <= kWideSmallMax)
        with_small(nc, [&](auto k) {
            constexpr int N = decltype(k)::value;
            wide::k_plaquette_small_batch<T, N><<<tiles, wide::kLanes, wide::plaq_small_lds<T, N>(), s>>>(d, n);
        });
    else
        with_form(nc, [&](auto form) {
            constexpr int F = decltype(form)::value;
            wide::k_plaquette_large_batch<T, F><<<tiles, wide::plaq_threads(F), wide::plaq_large_lds<T>(nc), s>>>(d, n,
                                                                                                                  nc);
        });
}

template void launch_plaquette_wide<float>(const Ctx&, double*);
template void launch_plaquette_wide<double>(const Ctx&, double*);
template void launch_plaquette_wide_batch<float>(const ChainDesc*, int, int, int, hipStream_t);
template void launch_plaquette_wide_batch<double>(const ChainDesc*, int, int, int, hipStream_t);

}  // namespace sun
