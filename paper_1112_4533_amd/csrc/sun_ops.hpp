// sun_ops.hpp -- host-side launchers, one table per (Nc, storage type).
// Each ops_nc*.hip translation unit instantiates the kernels of one Nc.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sun_device.hpp"

namespace sun {

// Launch shape of a phase kernel.
struct Shape {
    int block = 256;  // work-items per workgroup (64, 128 or 256)
    int xcd = 1;      // XCD-aware workgroup order
    int waves = 0;    // resident waves per CU (0 = no cap)
    int tblock = 0;   // time slices per block of the tile walk (0: linear)
    int spt = 1;      // sites per work-item (1, 2 or 4): tiles a workgroup takes in turn
    // 64-item workgroups issue the staple's loads ahead (SU(3); fixed by the
    // lattice, whatever shape is set)
    bool ahead = false;
};
inline bool valid_spt(int s) { return s == 1 || s == 2 || s == 4; }
inline int grid_for(int nblk, int spt) { return (nblk + spt - 1) / spt; }

// The walk of a single lattice's phase for a shape; falls back to the linear
// walk where the t-blocked one is not a permutation of the tiles.
inline Walk walk_for(const Geom& g, const Shape& sh) {
    Walk w{sh.xcd, 0, 1, 1, 0, sh.spt};
    const long long plane_h = (long long)g.L[0] * g.L[1] / 2;
    if (sh.tblock > 1 && plane_h % sh.block == 0 && g.L[3] % sh.tblock == 0) {
        w.tb = sh.tblock;
        w.tpp = (int)(plane_h / sh.block);
        w.lz = g.L[2];
    }
    return w;
}
inline bool valid_tblock(int t) { return t == 0 || t == 1 || t == 2 || t == 4 || t == 8; }

struct Ctx {
    void* links;
    Geom g;
    hipStream_t stream;
    Shape shape[2];   // per update kind: heatbath, overrelaxation
    int nc;
    int nt;           // nontemporal access to updated links (field well above the Infinity Cache)
    int rev;          // this phase walks its tiles in reverse order
    uint64_t order = 0;  // nonzero: a random tile order drawn from this value (race check)
};

// The affine permutation q -> (pa q + pc) mod n of a random tile order,
// drawn from `order` (splitmix64 steps); pa is coprime to n.
inline void random_tile_order(uint64_t order, int n, Walk& w) {
    auto mix = [](uint64_t& x) {
        uint64_t z = (x += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    auto gcd = [](uint64_t a, uint64_t b) {
        while (b) {
            const uint64_t t = a % b;
            a = b;
            b = t;
        }
        return a;
    };
    if (n <= 1) return;
    uint64_t x = order;
    uint64_t a = 1 + mix(x) % (uint64_t)(n - 1);
    while (gcd(a, (uint64_t)n) != 1) a = a % (uint64_t)(n - 1) + 1;
    w.pa = (uint32_t)a;
    w.pc = (uint32_t)(mix(x) % (uint64_t)n);
}

// Infinity Cache (MALL) of an MI355X is 256 MB.  Updated links keep plain
// (cached) access up to 1.25 x that size: measured on 32^4 SU(3), a 302 MB
// field ran 3.6% faster with plain access, 402 and 604 MB fields 1-2% faster
// with nontemporal access (with alternating walk directions).
constexpr size_t kPlainAccessMaxBytes = 320ull << 20;

// Dynamic LDS per workgroup that limits a CU to `waves` resident waves of
// `block`-item workgroups (0 = no cap).  LDS per CU: 160 KiB on gfx950; the
// size is kLdsPerCu / (blocks + 1/2) rounded down to 512 bytes, so that
// `blocks` workgroups fit with room to spare and one more does not.
constexpr int kLdsPerCu = 160 * 1024;
inline int lds_for_wave_cap(int waves, int block) {
    if (waves <= 0) return 0;
    const int per_block = block / 64;
    const int blocks = waves / per_block < 1 ? 1 : waves / per_block;
    return (int)(2.0 * kLdsPerCu / (2 * blocks + 1)) & ~511;
}
inline bool valid_wave_cap(int w) { return w == 0 || w == 8 || w == 12 || w == 16; }

// The plaquette kernel re-reads each link from up to six sites; with its
// register use alone a CU holds 16 of its waves, and their combined working
// set can thrash the L2.  The best cap depends on whether the field stays in
// the Infinity Cache (measured on SU(3) 32^4): the 201 MB two-row FP32 field
// runs best uncapped at 16 waves per CU (8 / 12 / 16: 115.7 / 107.3 /
// 104.6 us), the 302 MB 18-real field at 8 (150 / 152 / 165.5 us), and the
// 604 MB FP64 field at 12 (358 us against 369 uncapped).
constexpr size_t kInfinityCacheBytes = 256ull << 20;
inline int plaquette_wave_cap(size_t field_bytes) {
    if (field_bytes <= kInfinityCacheBytes) return 16;
    if (field_bytes <= kPlainAccessMaxBytes) return 8;
    return 12;
}

// Launch shapes the phase kernels are instantiated for.
constexpr int kPhaseBlocks[3] = {64, 128, 256};
inline bool valid_phase_block(int b) { return b == 64 || b == 128 || b == 256; }

// What a phase's default launch shape follows from besides the link type.
struct PhaseGrid {
    long long links;  // links a phase updates
    int dirs;         // directions present
    bool far;         // 64-item workgroups would walk linearly over large planes
};
inline PhaseGrid phase_grid(const Geom& g, bool linear) {  // linear: the walk is never t-blocked (a batch's)
    const int plane = g.L[0] * g.L[1] / 2;
    return PhaseGrid{g.Vh, __builtin_popcount(g.present), plane > 12 * 64 && (linear || plane % 64 != 0 || g.L[3] % 4 != 0)};
}

// Workgroup, wave cap and walk that a phase starts with; a tuner or the caller
// may replace them, but not whether 64-item workgroups of SU(3) issue the loads
// ahead: they do where they are the default, but for two stretches of the
// overrelaxation in which they are faster with the loads by direction (FP32
// 72-byte links from five quarters of a wavefront per SIMD to one and a half,
// 20 20 20 24 16.1 -> 15.5; FP64 from one to one and a half, 20^4 24.7 -> 23.4,
// 18 20 22 24 28.2 -> 27.4).  Where they are not the default, a 64-item shape that
// is asked for has the loads by direction too (24^4 FP32 overrelaxation 28.0 ->
// 26.9, FP64 heatbath 64.4 -> 60.6).  block 256 unless 64-item workgroups do
// better, which spread a small grid over all CUs and, for SU(3), issue the
// staple's loads ahead at half the resident wavefronts.  Overrelaxation /
// heatbath phase, 256 -> 64, in microseconds:
//   SU(2), SU(4), up to two wavefronts per SIMD: SU(2) FP32 20^4 6.0/7.3 ->
//     5.3/7.0, SU(4) 16^4 FP32 18.6/23.0 -> 16.4/21.6, FP64 24.7/61.8 -> 23.4/53.9;
//     past it equal (SU(4) 24^4 54.3/60.7, 55.0/59.9) or slower (SU(2) 32^4
//     15.1/16.9 -> 15.5/17.3)
//   SU(3) FP32, up to one and a half: 16^4 10.9/13.7 -> 8.5/11.7, 20^4 16.3/19.6 ->
//     13.6/17.6; slower past it (16 32 16 32 20.1/23.4 -> 21.1/24.0, 24^4
//     26.9/29.9 -> 28.0/31.1), until the caches no longer hold the field and fewer
//     wavefronts re-read more from L2: overrelaxation of 72-byte links from eight
//     per SIMD on (28^4 45.4 -> 47.2, 24 24 40 38 62.7 -> 64.9, 24 24 40 44 74.4 ->
//     76.0, 32^4 73.5 -> 71.7, 16 32 48 48 97.2 -> 88.2, 48^4 531 -> 436), of
//     48-byte ones from six (24 24 40 36 45.9 -> 46.0, 20 20 48 48 45.2 -> 44.0,
//     32^4 48.2 -> 46.8, 36^4 89.6 -> 84.8, 48^4 310 -> 289); heatbath of
//     72-byte links from four on (16 32 32 32 44.4 -> 40.1, 32^4 88.0 -> 78.0), of
//     48-byte ones not (32^4 54.2 -> 59.1)
//   SU(3) FP64, up to one (144-byte links below it: 16 16 16 32 18.7/26.7 ->
//     19.2/27.1, two-row 14.9/22.5 -> 14.2/22.4): 16^4 12.2/20.5 -> 10.5/19.0;
//     overrelaxation at any size (24^4 51.3 -> 46.1, 32^4 151 -> 137, two-row 32^4 101 -> 92) unless it
//     walks linearly over planes of more than twelve wavefronts (40^4 445 -> 458,
//     44^4 696 -> 702; 36^4, of ten, 263 -> 261; 48^4, t-blocked, 936 -> 789); the
//     heatbath not (20^4 36.3 -> 38.3)
//   SU(3) with a direction absent: only in three, up to half a wavefront per SIMD
//     (40^3 FP32 8.8/11.6 -> 8.3/11.0, FP64 32 32 64 9.6/19.6 -> 9.2/18.9).  The loads
//     ahead are issued for the absent direction too, and a wavefront of fewer
//     staples does better with others beside it (48 48 40 FP32 9.1/12.3 -> 9.5/12.9,
//     48^3 9.4/12.6 -> 10.8/14.4, 256 512 7.6/12.8 -> 10.7/16.1; FP64
//     overrelaxation 512^2 17.4 -> 22.3, 56^3 19.5 -> 21.7).
// Wave caps of larger grids, from sweeps on SU(3) 32^4: the heatbath 16
// resident waves per CU whatever the storage, the overrelaxation 12 for
// 48-byte links (FP32 two-row) and 8 for larger ones (18-real FP32 70.0 -> 67.3
// us, FP64 161 -> 152); a grid of two wavefronts per SIMD needs none, nor a
// t-blocked walk (16^4 8.5 -> 8.8 with one).
inline Shape default_shape(int nc, bool f64, size_t link_bytes, const PhaseGrid& grid, bool heatbath) {
    const long long per_simd = 1024 * 64;  // links of one wavefront on every SIMD
    const long long few = nc != 3 ? 2 * per_simd : !f64 ? per_simd * 3 / 2 : link_bytes > 96 ? per_simd - 1 : per_simd;
    const long long few3 = grid.dirs == 4 ? few : grid.dirs == 3 ? per_simd / 2 : 0;
    if (grid.links <= (nc == 3 ? few3 : few)) {
        const bool late = !f64 && !heatbath && link_bytes > 48 && grid.links > per_simd * 5 / 4;
        return Shape{64, 1, 0, 0, 1, nc == 3 && !late};
    }
    if (nc == 3 && grid.dirs == 4) {
        if (f64 && !heatbath && !grid.far) return Shape{64, 1, 8, 4, 1, grid.links >= per_simd * 3 / 2};
        const bool many = heatbath ? link_bytes > 48 && grid.links >= 4 * per_simd
                                   : grid.links >= (link_bytes > 48 ? 8 : 6) * per_simd;
        if (!f64 && many) return Shape{64, 1, 8, 4, 1, true};
    }
    return Shape{256, 1, heatbath ? 16 : link_bytes > 48 ? 8 : 12, 4};
}

struct Ops {
    // one checkerboard phase; kind 0 heatbath, 1 overrelaxation
    void (*update)(const Ctx&, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step);
    void (*init)(const Ctx&, int hot, uint32_t k0, uint32_t k1);
    // reductions write 2 doubles per workgroup into partial and return the
    // workgroup count (reunit: partial may be null, then nothing is reported)
    int (*reunit)(const Ctx&, double* partial);
    int (*unitarity)(const Ctx&, double* partial);
    int (*plaquette)(const Ctx&, double* partial);
    // partial: 2 doubles per block; returns the block count
    int (*polyakov)(const Ctx&, double* partial);
    void (*export_field)(const Ctx&, double* out);
    void (*import_field)(const Ctx&, const double* in);
    // batches: d is a device table of n chains of this Nc (nc) and storage
    // type; tiles is the total tile count of the grid kind the call uses (on
    // the workgroup-per-link path: wide_*_tiles)
    void (*update_batch)(const ChainDesc* d, int n, int tiles, int kind, int mu, int par, uint32_t step_offset,
                         const Shape& shape, int nc, hipStream_t s);
    void (*reunit_batch)(const ChainDesc* d, int n, int tiles, int nc, hipStream_t s);
    void (*plaquette_batch)(const ChainDesc* d, int n, int tiles, double* out, int nc, hipStream_t s);
};

constexpr int kLaunchBlock = 256;
inline int blocks_for(long long n) { return (int)((n + kLaunchBlock - 1) / kLaunchBlock); }
inline int link_blocks(const Geom& g) { return blocks_for(4LL * g.V); }
inline int half_blocks(const Geom& g) { return blocks_for(g.Vh); }
inline int half_blocks(const Geom& g, int bs) { return (g.Vh + bs - 1) / bs; }
inline int spatial_blocks(const Geom& g) { return blocks_for(g.V / g.L[3]); }

// f64 = 0: float storage, 1: double storage
const Ops* ops_nc2(int f64);
const Ops* ops_nc3(int f64);
const Ops* ops_nc4(int f64);
const Ops* ops_nc3_two_row(int f64);  // SU(3), rows 0 and 1 stored
const Ops* ops_wide(int f64);         // 4 <= Nc <= 32: link-major storage

// Phases of small lattices take four lanes to a link, kQuadLinks links to a
// wavefront (sun_quad.hpp).  They win while a phase is about one wavefront per
// SIMD (1024 of them): beyond it the quad's shared work is issued in turn with
// other links' and costs more than it shortens.  Overrelaxation / heatbath
// phase, one lane to a link -> four, in microseconds:
//   SU(2), two wavefronts per SIMD: FP64 8^4 4.6/9.2 -> 2.9/4.7, 16^4 (at the
//     limit) 5.2/9.4 -> 4.8/7.6, FP32 16^4 4.7/6.3 -> 4.2/5.1
//   SU(3), one: FP32 8^4 9.0/11.6 -> 4.5/6.4, 12^4 9.8/12.4 -> 6.6/8.4;
//     FP64 12 12 14 16 (at the limit) 11.0/19.3 -> 9.2/14.8, 14^4 (past it)
//     11.4/19.6 -> 12.4/19.8
//   SU(4), five quarters: 12^4 FP32 17.8/21.9 -> 10.9/14.7, FP64 20.9/58.1 ->
//     12.1/24.5; 14^4 18.4/22.7 -> 13.9/18.6; 14^3 16 (past it) FP32 18.3/22.7 ->
//     17.8/22.1, FP64 22.4/60.2 -> 23.9/48.1
// With fewer directions a link has fewer staples, a one-lane work-item is
// sooner done and the overrelaxation's line lies lower:
//   three directions: SU(2) 32 32 64 (two per SIMD) 4.1/6.2 -> 4.3/5.6, 48 48 20
//     4.2/6.2 -> 3.9/5.2; SU(3) FP32 32^3 (one) 7.7/10.8 -> 7.6/9.6; SU(4) FP64
//     32 32 40 (five quarters) 15.5/55 -> 18.8/44, 32^3 15.1/54 -> 13.1/28
//   two: SU(2) FP64 256^2 (two) 4.1/10.4 -> 4.5/9.2, 192 256 4.0/10.3 -> 4.0/8.6;
//     SU(3) FP64 128 256 (one) 6.7/18.6 -> 7.9/15.4, 128 160 6.2 -> 6.6, 128^2
//     (half) 6.1/19.7 -> 5.6/12.9; SU(4) FP32 160 256 (five quarters) 10.1/17.4 ->
//     13.9/19.1, 128 256 (one) 9.8/17.1 -> 11.6/16.6, 128 192 9.5/17.1 -> 9.6/14.3
//   one (no staples): SU(3) 16384 4.9/8.2 -> 5.1/7.7, 65536 4.9/8.4 -> 6.1/10.6
constexpr int kQuadLinks = 16;
// wavefronts: [directions - 1][Nc - 2][heatbath, overrelaxation]
constexpr int kQuadWaves[4][3][2] = {{{1024, 0}, {512, 0}, {640, 0}},
                                     {{2048, 1536}, {1024, 512}, {1024, 768}},
                                     {{2048, 1536}, {1024, 1024}, {1280, 1024}},
                                     {{2048, 2048}, {1024, 1024}, {1280, 1280}}};
inline bool quad_applies(int nc, const Geom& g, int kind) {
    return g.Vh <= kQuadLinks * kQuadWaves[__builtin_popcount(g.present) - 1][nc - 2][kind];
}
template <int N, typename T, int R>
void launch_update_quad(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step);

// Up to Nc = kWideSmallMax an update workgroup (one wavefront) takes
// kWideSmallLinks links, above it (two wavefronts) one.
constexpr int kWideSmallMax = 8, kWideSmallLinks = 4;
inline int wide_update_tiles(int nc, int Vh) {
    return nc <= kWideSmallMax ? (Vh + kWideSmallLinks - 1) / kWideSmallLinks : Vh;
}
// Likewise the plaquette takes kWideSmallLinks sites, or one.
inline int wide_plaquette_tiles(int nc, int V) {
    return nc <= kWideSmallMax ? (V + kWideSmallLinks - 1) / kWideSmallLinks : V;
}
// Re-unitarization: a wavefront takes four links up to Nc = 8, two up to 16.
inline int wide_reunit_tiles(int nc, int V) {
    const int links = nc <= 8 ? 4 : nc <= 16 ? 2 : 1;
    return (4 * V + links - 1) / links;
}
template <typename T>
int launch_reunit_wide(const Ctx& c, double* partial);
template <typename T>
int launch_unitarity_wide(const Ctx& c, double* partial);
template <typename T>
void launch_reunit_wide_batch(const ChainDesc* d, int n, int tiles, int nc, hipStream_t s);
template <typename T>
void launch_plaquette_wide(const Ctx& c, double* partial);
template <typename T>
void launch_plaquette_wide_batch(const ChainDesc* d, int n, int tiles, int nc, hipStream_t s);
template <typename T>
void launch_update_small(const Ctx& c, int hb, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step);
template <typename T>
void launch_update_small_batch(const ChainDesc* d, int n, int tiles, int hb, int mu, int par, uint32_t off, int nc,
                               hipStream_t s);
template <typename T>
void launch_update_large(const Ctx& c, int hb, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step);
template <typename T>
void launch_update_large_batch(const ChainDesc* d, int n, int tiles, int hb, int mu, int par, uint32_t off, int nc,
                               hipStream_t s);

void launch_finalize_max2(const double* partial, int nblk, double* out, hipStream_t s);
void launch_finalize_sum2(const double* partial, int nblk, double* out, double scale, hipStream_t s);
void launch_plaquette_final(const double* partial, int nblk, double* out, double norm_sp, double norm_tm,
                            double norm_all, hipStream_t s);
void launch_advance_steps(ChainDesc* d, int n, int n_hb, hipStream_t s);
void launch_sample_su2(int f64, const double* alpha, int n, uint32_t k0, uint32_t k1, uint32_t step,
                       uint32_t mu_sg, double* x, int* attempts, hipStream_t s);
// the large-Nc path's batched draw (element i: subgroup mu_sg + i mod 8 of site i / 8)
void launch_sample_su2_batched(int f64, const double* alpha, int n, uint32_t k0, uint32_t k1, uint32_t step,
                               uint32_t mu_sg, double* x, int* attempts, hipStream_t s);

}  // namespace sun
