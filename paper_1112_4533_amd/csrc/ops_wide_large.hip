// ops_wide_large.hip -- launchers of the two-wavefront update (Nc >= 9), one
// workgroup per link; Nc is a run-time argument, the LDS size follows it.
#include "sun_ops.hpp"
#include "sun_wide_large.hpp"

namespace sun {
namespace {

template <typename T, int RANGE, bool HB>
void launch(const Ctx& c, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step) {
    wide::k_update_large<T, RANGE, HB><<<wide_update_tiles(c.nc, c.g.Vh), wide::kLargeThreads,
                                         wide::large_lds<T, RANGE>(c.nc, HB), c.stream>>>((T2<T>*)c.links, c.g, c.nc, mu, par,
                                                                                   (T)beta, k0, k1, step);
}
template <typename T, int RANGE, bool HB>
void launch_batch(const ChainDesc* d, int n, int tiles, int mu, int par, uint32_t off, int nc, hipStream_t s) {
    wide::k_update_large_batch<T, RANGE, HB><<<tiles, wide::kLargeThreads, wide::large_lds<T, RANGE>(nc, HB), s>>>(
        d, n, nc, mu, par, off);
}

// f(range, kind) with both as compile-time constants.  The FP64 heatbath takes
// the last form from Nc = 23, where the LDS holds fewer than 8 links per CU
// in any case and the form's larger register budget spares it spills (8^4:
// SU(24) 381 -> 320 us, at beta 6.2, most draws in the Creutz range, 655 -> 491).
template <typename T, typename F>
void with_range(int nc, int hb, F f) {
    auto kind = [&](auto range) {
        if (hb)
            f(range, std::true_type{});
        else
            f(range, std::false_type{});
    };
    if (nc <= wide::kLargeMax[0])
        kind(std::integral_constant<int, 0>{});
    else if (nc <= wide::kLargeMax[1])
        kind(std::integral_constant<int, 1>{});
    else if (nc <= (hb && sizeof(T) == 8 ? 22 : wide::kLargeMax[2]))
        kind(std::integral_constant<int, 2>{});
    else
        kind(std::integral_constant<int, 3>{});
}

}  // namespace

template <typename T>
void launch_update_large(const Ctx& c, int hb, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step) {
    with_range<T>(c.nc, hb, [&](auto range, auto kind) {
        launch<T, decltype(range)::value, decltype(kind)::value>(c, mu, par, beta, k0, k1, step);
    });
}
template <typename T>
void launch_update_large_batch(const ChainDesc* d, int n, int tiles, int hb, int mu, int par, uint32_t off, int nc,
                               hipStream_t s) {
    with_range<T>(nc, hb, [&](auto range, auto kind) {
        launch_batch<T, decltype(range)::value, decltype(kind)::value>(d, n, tiles, mu, par, off, nc, s);
    });
}

template void launch_update_large<float>(const Ctx&, int, int, int, double, uint32_t, uint32_t, uint32_t);
template void launch_update_large<double>(const Ctx&, int, int, int, double, uint32_t, uint32_t, uint32_t);
template void launch_update_large_batch<float>(const ChainDesc*, int, int, int, int, int, uint32_t, int, hipStream_t);
template void launch_update_large_batch<double>(const ChainDesc*, int, int, int, int, int, uint32_t, int, hipStream_t);

}  // namespace sun
