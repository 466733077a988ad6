// ops_wide_reunit.hip -- launchers of the large-Nc re-unitarization and
// unitarity report.
#include <type_traits>

#include "sun_ops.hpp"
#include "sun_wide_reunit.hpp"

namespace sun {
namespace {

// f(ROWS, NC): rows of a link's half-wave share and columns per lane for Nc.
// Nine columns up to Nc = 18: with twelve the unitarity report of SU(17) on 8^4
// takes 129 us instead of 105, the re-unitarization 207 instead of 185 (one
// wavefront per link with the LU in LDS 119 and 210).
template <typename F>
void with_rows(int nc, F f) {
    auto call = [&](auto rows, auto cols) { f(rows, cols); };
#define SUN_ROWS(R, C) call(std::integral_constant<int, R>{}, std::integral_constant<int, C>{})
    if (nc <= 6)
        SUN_ROWS(8, 3);
    else if (nc <= 8)
        SUN_ROWS(8, 4);
    else if (nc <= 12)
        SUN_ROWS(16, 6);
    else if (nc <= 16)
        SUN_ROWS(16, 8);
    else if (nc <= 18)
        SUN_ROWS(32, 9);
    else if (nc <= 24)
        SUN_ROWS(32, 12);
    else
        SUN_ROWS(32, 16);
#undef SUN_ROWS
}

template <typename T, int MODE>
int launch(const Ctx& c, double* partial) {
    const int tiles = wide_reunit_tiles(c.nc, c.g.V);
    with_rows(c.nc, [&](auto rows, auto cols) {
        constexpr int R = decltype(rows)::value, C = decltype(cols)::value;
        wide::k_reunit_rows<T, R, C, MODE><<<tiles, wide::kLanes, wide::rows_lds<R, C>(c.nc), c.stream>>>(
            (T2<T>*)c.links, c.g, c.nc, partial);
    });
    return tiles;
}

}  // namespace

template <typename T>
int launch_reunit_wide(const Ctx& c, double* partial) {
    return partial ? launch<T, wide::REUNIT_REPORT>(c, partial) : launch<T, wide::REUNIT_PLAIN>(c, nullptr);
}
template <typename T>
int launch_unitarity_wide(const Ctx& c, double* partial) {
    return launch<T, wide::UNITARITY_ONLY>(c, partial);
}
template <typename T>
void launch_reunit_wide_batch(const ChainDesc* d, int n, int tiles, int nc, hipStream_t s) {
    with_rows(nc, [&](auto rows, auto cols) {
        constexpr int R = decltype(rows)::value, C = decltype(cols)::value;
        wide::k_reunit_rows_batch<T, R, C><<<tiles, wide::kLanes, wide::rows_lds<R, C>(nc), s>>>(
            d, n, nc);
    });
}

template int launch_reunit_wide<float>(const Ctx&, double*);
template int launch_reunit_wide<double>(const Ctx&, double*);
template int launch_unitarity_wide<float>(const Ctx&, double*);
template int launch_unitarity_wide<double>(const Ctx&, double*);
template void launch_reunit_wide_batch<float>(const ChainDesc*, int, int, int, hipStream_t);
template void launch_reunit_wide_batch<double>(const ChainDesc*, int, int, int, hipStream_t);

}  // namespace sun
