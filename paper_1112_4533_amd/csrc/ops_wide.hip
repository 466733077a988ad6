// ops_wide.hip -- the large-Nc table of launchers: the kernels of sun_wide.hpp
// (one wavefront per link or spatial site, Nc a run-time argument, the LDS size
// following it) are launched here, the others in their own units.
#include "sun_ops.hpp"
#include "sun_wide.hpp"

namespace sun {

template <typename T>
struct OpsWide {
    using P = T2<T>;

    // The launch shape does not apply to the update: its workgroups follow
    // from Nc.
    static void update(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step) {
        const int hb = kind == 0 ? 1 : 0;
        if (c.nc <= kWideSmallMax)
            launch_update_small<T>(c, hb, mu, par, beta, k0, k1, step);
        else
            launch_update_large<T>(c, hb, mu, par, beta, k0, k1, step);
    }
    static void init(const Ctx& c, int hot, uint32_t k0, uint32_t k1) {
        wide::k_init<T><<<4 * c.g.V, wide::kLanes, wide::fp64_lds(c.nc, 2), c.stream>>>((P*)c.links, c.g, c.nc, hot, k0,
                                                                                        k1);
    }
    static int reunit(const Ctx& c, double* partial) { return launch_reunit_wide<T>(c, partial); }
    static int unitarity(const Ctx& c, double* partial) { return launch_unitarity_wide<T>(c, partial); }
    static int plaquette(const Ctx& c, double* partial) {
        launch_plaquette_wide<T>(c, partial);
        return c.g.V;
    }
    static int polyakov(const Ctx& c, double* partial) {
        const int Vs = c.g.V / c.g.L[3];
        wide::k_polyakov<T><<<Vs, wide::kLanes, wide::fp64_lds(c.nc, 3), c.stream>>>((const P*)c.links, c.g, c.nc,
                                                                                     partial);
        return Vs;
    }
    static int entry_blocks(const Ctx& c) {
        return (int)((4LL * c.g.V * c.nc * c.nc + 255) / 256);
    }
    static void export_field(const Ctx& c, double* out) {
        wide::k_export<T><<<entry_blocks(c), 256, 0, c.stream>>>((const P*)c.links, c.g, c.nc, out);
    }
    static void import_field(const Ctx& c, const double* in) {
        wide::k_import<T><<<entry_blocks(c), 256, 0, c.stream>>>((P*)c.links, c.g, c.nc, in);
    }

    // Batches: one launch per phase covers every chain of the group (same
    // Nc and precision).
    static void update_batch(const ChainDesc* d, int n, int tiles, int kind, int mu, int par, uint32_t off,
                             const Shape& /*shape*/, int nc, hipStream_t s) {
        const int hb = kind == 0 ? 1 : 0;
        if (nc <= kWideSmallMax)
            launch_update_small_batch<T>(d, n, tiles, hb, mu, par, off, nc, s);
        else
            launch_update_large_batch<T>(d, n, tiles, hb, mu, par, off, nc, s);
    }
    static void reunit_batch(const ChainDesc* d, int n, int tiles, int nc, hipStream_t s) {
        launch_reunit_wide_batch<T>(d, n, tiles, nc, s);
    }
    static void plaquette_batch(const ChainDesc* d, int n, int tiles, double* out, int nc, hipStream_t s) {
        launch_plaquette_wide_batch<T>(d, n, tiles, nc, s);
        wide::k_plaquette_final_batch_wide<><<<n, kBlock, 0, s>>>(d, n, nc, out);
    }

    static const Ops* table() {
        static const Ops ops = {&update, &init, &reunit, &unitarity, &plaquette, &polyakov, &export_field,
                                &import_field, &update_batch, &reunit_batch, &plaquette_batch};
        return &ops;
    }
};

const Ops* ops_wide(int f64) { return f64 ? OpsWide<double>::table() : OpsWide<float>::table(); }

void launch_sample_su2_batched(int f64, const double* alpha, int n, uint32_t k0, uint32_t k1, uint32_t step,
                               uint32_t mu_sg, double* x, int* attempts, hipStream_t s) {
    const int sites = (n + wide::kSampleSteps - 1) / wide::kSampleSteps;
    if (f64)
        wide::k_sample_su2_batched<double><<<sites, wide::kLanes, 0, s>>>(alpha, n, k0, k1, step, mu_sg, x, attempts);
    else
        wide::k_sample_su2_batched<float><<<sites, wide::kLanes, 0, s>>>(alpha, n, k0, k1, step, mu_sg, x, attempts);
}

}  // namespace sun
