// ops_wide_plaq.hip -- launchers of the large-Nc plaquette.
#include <climits>

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

// The sites of a lattice from which Nc = 17 to 20 take the one tile and its
// edges: below four sites per CU (ten for Nc = 20) the four tiles' lower latency
// counts; edges against four tiles, us: SU(17) FP32 4 4 4 8 35.8 / 33.6, 4 4 8 8
// 36.7 / 52.3; SU(19) FP64 4 4 4 8 45 / 36, 4 4 8 8 48 / 56; SU(20) FP64 4 4 8 8
// 58 / 56, 6 6 8 8 116 / 111, 8^4 141 / 187.  By the lattice, in a batch too: a
// chain's plaquette has the same bits alone and in a batch.
int edge_sites(int nc) { return 256 * (nc < wide::kEdgeMax ? 4 : 10); }

// f(form, from, to) for Nc > kWideSmallMax: the form for lattices of from .. to - 1
// sites.
template <typename F>
void with_forms(int nc, F f) {
    if (nc <= wide::kTile) {
        f(std::integral_constant<int, wide::PLAQ_ONE>{}, 0, INT_MAX);
    } else if (nc <= wide::kEdgeMax) {
        f(std::integral_constant<int, wide::PLAQ_EDGES>{}, edge_sites(nc), INT_MAX);
        f(std::integral_constant<int, wide::PLAQ_FOUR>{}, 0, edge_sites(nc));
    } else {
        f(std::integral_constant<int, wide::PLAQ_FOUR>{}, 0, INT_MAX);
    }
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
        with_forms(c.nc, [&](auto form, int from, int to) {
            constexpr int F = decltype(form)::value;
            if (c.g.V < from || c.g.V >= to) return;
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
        with_forms(nc, [&](auto form, int from, int to) {
            constexpr int F = decltype(form)::value;
            wide::k_plaquette_large_batch<T, F><<<tiles, wide::plaq_threads(F), wide::plaq_large_lds<T>(nc), s>>>(
                d, n, nc, from, to);
        });
}

template void launch_plaquette_wide<float>(const Ctx&, double*);
template void launch_plaquette_wide<double>(const Ctx&, double*);
template void launch_plaquette_wide_batch<float>(const ChainDesc*, int, int, int, hipStream_t);
template void launch_plaquette_wide_batch<double>(const ChainDesc*, int, int, int, hipStream_t);

}  // namespace sun
