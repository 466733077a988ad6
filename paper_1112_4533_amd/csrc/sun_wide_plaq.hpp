// sun_wide_plaq.hpp -- the plaquette of the large-Nc path, FP64:
// ReTr(U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag) = Re sum_ij H_ij conj(K_ij)
// with H = U_mu(x) U_nu(x+mu) and K = U_nu(x) U_mu(x+nu), both kept in the
// registers that formed them: twelve products per site and no matrix stored.
//
// Up to Nc = 8 a wavefront takes four sites, sixteen lanes each (row r and
// column half of H and K per lane, as in the update); above, the products
// are 16 x 16 FP64 matrix-core tiles: one on one wavefront to Nc = 20, with what
// lies past it from Nc = 17 on the vector units, then four on four wavefronts.
// The links of the next product load while this one runs.
//
// Bound by the FP64 rate (Nc >= 21: the tiles' padding included) and the
// links' re-reads through L2.  Against one wavefront per site, products and
// one factor through LDS: SU(6) FP32 12^4 106 -> 37 us, SU(8) FP64 12^4 130 -> 64,
// SU(16) FP64 8^4 116 -> 48, SU(17) FP32 8^4 151 -> 82, SU(24) FP64 8^4 510 -> 214,
// SU(32) FP32 8^4 1357 -> 269.
#pragma once

#include "sun_wide_large.hpp"
#include "sun_wide_small.hpp"

namespace sun {
namespace wide {

// Site s in logical order.
__device__ __forceinline__ Site site_at(const Geom& g, int s) {
    Site x;
    const int r1 = s / g.L[0], r2 = r1 / g.L[1], r3 = r2 / g.L[2];
    x.x[0] = s - r1 * g.L[0];
    x.x[1] = r1 - r2 * g.L[1];
    x.x[2] = r2 - r3 * g.L[2];
    x.x[3] = r3;
    x.s = s;
    return x;
}

// The planes of a site in order: next(mu, nu) steps to the next plane whose
// directions are both present, mu = 4 past the last.
struct Plane {
    int mu = 0, nu = 0;
    __device__ __forceinline__ void next(int present) {
        do {
            if (++nu == 4) {
                ++mu;
                nu = mu + 1;
            }
        } while (mu < 3 && !((present >> mu) & (present >> nu) & 1));
    }
    __device__ __forceinline__ bool done() const { return mu >= 3; }
};

// -- Nc <= 8 -----------------------------------------------------------------

// Sums of sites s0 .. s0 + 3 (those below V): partial[2 s] over the planes
// without direction 3, partial[2 s + 1] with.
template <typename T, int N>
__device__ __forceinline__ void plaquette_sites_small(const T2<T>* __restrict__ U, const Geom& g, int s0,
                                                      double* __restrict__ partial) {
    using S = SmallShape<T, N>;
    constexpr int kHalf = S::kHalf, kRow = S::kRow, n2 = N * N;
    extern __shared__ double4 smem_plaq[];
    const int lane = threadIdx.x;
    const int p = lane / kPlaceLanes, q = lane % kPlaceLanes;
    const int r8 = q & 7, r = r8 < N ? r8 : N - 1, j0 = (q >> 3) * kHalf;
    const bool live = s0 + p < g.V;
    T2<T>* const A = reinterpret_cast<T2<T>*>(smem_plaq) + 2 * p * S::kMat;
    T2<T>* const B = A + S::kMat;
    const Site x = site_at(g, live ? s0 + p : g.V - 1);
    const int u0 = step_shift(g, x, true, 0), u1 = step_shift(g, x, true, 1);
    const int u2 = step_shift(g, x, true, 2), u3 = step_shift(g, x, true, 3);
    const int par = parity_of(x), op = par ^ 1, h = x.s >> 1, Vh = g.Vh;
    LinkRegs<T, N> fa, fb;
    auto load = [&](int m, int k) {  // the factors of U_m(x) U_k(x + m)
        fa.load(link_at<T>(U, n2, m, par, h, Vh), q);
        fb.load(link_at<T>(U, n2, k, op, (x.s + pick_dir(u0, u1, u2, u3, m)) >> 1, Vh), q);
    };
    // the lane's entries of the staged product
    auto product = [&](double(&re)[kHalf], double(&im)[kHalf]) {
        double ar[N], ai[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const T2<T> v = A[r * kRow + k];
            ar[k] = v.x;
            ai[k] = v.y;
        }
#pragma unroll
        for (int j = 0; j < kHalf; ++j) {
            re[j] = im[j] = 0.0;
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const T2<T> b = B[k * kRow + j0 + j];
                cmac(re[j], im[j], ar[k], ai[k], (double)b.x, (double)b.y);
            }
        }
    };
    double space = 0.0, time = 0.0;  // planes without and with direction 3
    Plane pl;
    pl.next(g.present);
    if (!pl.done()) load(pl.mu, pl.nu);
    while (!pl.done()) {
        double hr[kHalf], hi[kHalf], kr[kHalf], ki[kHalf];
        fa.store(A, q);
        fb.store(B, q);
        load(pl.nu, pl.mu);
        wave_lds_order();
        product(hr, hi);
        wave_lds_order();
        fa.store(A, q);
        fb.store(B, q);
        const bool with_time = pl.nu == 3;
        pl.next(g.present);
        if (!pl.done()) load(pl.mu, pl.nu);
        wave_lds_order();
        product(kr, ki);
        wave_lds_order();
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
            if (j0 + j < N) t = fmadd(hi[j], ki[j], fmadd(hr[j], kr[j], t));
        (with_time ? time : space) += t;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {  // over the site's sixteen lanes
        double v = r8 >= N ? 0.0 : c ? time : space;
        v += partner<0>(v);
        v += partner<1>(v);
        v += partner<2>(v);
        v += partner<3>(v);
        if (live && q == 0) partial[2 * (size_t)x.s + c] = v;
    }
}
template <typename T, int N>
constexpr size_t plaq_small_lds() {
    return (size_t)kSmallLinks * 2 * SmallShape<T, N>::kMat * sizeof(T2<T>);
}

template <typename T, int N>
__global__ __launch_bounds__(kLanes, 2) void k_plaquette_small(const T2<T>* __restrict__ U, Geom g,
                                                               double* __restrict__ partial) {
    plaquette_sites_small<T, N>(U, g, kSmallLinks * xcd_tile((int)blockIdx.x, (int)gridDim.x), partial);
}
template <typename T, int N>
__global__ __launch_bounds__(kLanes, 2) void k_plaquette_small_batch(const ChainDesc* __restrict__ d, int nchains) {
    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int c = find_chain<TILE_SITE>(d, nchains, tile);
    plaquette_sites_small<T, N>((const T2<T>*)d[c].links, d[c].g, kSmallLinks * (tile - d[c].tile0[TILE_SITE]),
                                d[c].scratch);
}

// -- Nc >= 9 -----------------------------------------------------------------

// One 16 x 16 tile of A B in FP64: rows row0 .., columns col0 .., A and B in
// LDS as stored (T).  Lane l holds row (column) l mod 16 and term l / 16 of
// the four that an instruction sums (Re A, then Im A terms of two k).
struct PlaqTile {
    f64x4 re, im;
    template <typename T>
    __device__ __forceinline__ void product(const T2<T>* A, const T2<T>* B, int n, int ns, int row0, int col0) {
        re = im = f64x4{0, 0, 0, 0};
        const int l = fresh_lane();
        const int part = (l >> 4) & 1, kk = l >> 5;
        const T* a = reinterpret_cast<const T*>(A + min(row0 + (l & 15), n - 1) * ns + kk) + part;
        const T* b = reinterpret_cast<const T*>(B + kk * ns + min(col0 + (l & 15), n - 1));
        struct Ops {
            T a, same, other;  // the lane's part of A, that part of B, the other part of B
        };
        for_steps<4>((n + 1) >> 1,
                     [&](int s) { return Ops{a[4 * s], b[4 * s * ns + part], b[4 * s * ns + 1 - part]}; },
                     [&](const Ops& o) {
                         const double av = o.a;
                         re = mma16(part ? -av : av, (double)o.same, re);
                         im = mma16(av, (double)o.other, im);
                     });
    }
};

// Forms: one wavefront and one tile to Nc = 16; the same up to kEdgeMax with the
// rows and columns past 15 on the vector units; four wavefronts and tiles above.
enum PlaqForm { PLAQ_ONE, PLAQ_EDGES, PLAQ_FOUR };
constexpr int kEdgeMax = kTile + 4;
constexpr int plaq_threads(int form) { return form == PLAQ_FOUR ? 4 * kLanes : kLanes; }
constexpr int plaq_loads(int form) {  // entries of a link per work-item
    const int n = form == PLAQ_ONE ? kTile : form == PLAQ_EDGES ? kEdgeMax : kNcMax;
    return (n * n + plaq_threads(form) - 1) / plaq_threads(form);
}
template <typename T>
constexpr size_t plaq_large_lds(int n) {
    return (size_t)2 * mat_entries(n) * sizeof(T2<T>);
}

// The entries of A B in rows or columns past 15, kTile < n <= kEdgeMax: lane l
// sums entries l, l + 64, ... of the rows past 15 and then of the columns past
// 15 in the rows above them.  Four tiles would spend three quarters of the
// matrix cores' time on them: SU(17) on 8^4 FP32 169 us against 82, FP64 177
// against 88 (one wavefront per site with products through LDS: 151 and 157),
// SU(20) 181 against 137 and 188 against 141.
struct PlaqEdges {
    static constexpr int kMost = (kEdgeMax * kEdgeMax - kTile * kTile + kLanes - 1) / kLanes;
    double re[kMost], im[kMost];
    static __device__ __forceinline__ int count(int n) { return n * n - kTile * kTile; }
    template <typename T>
    __device__ __forceinline__ void product(const T2<T>* A, const T2<T>* B, int n, int ns) {
        const int l = fresh_lane(), past = n - kTile, in_rows = past * n;
#pragma unroll
        for (int q = 0; q < kMost; ++q) {
            re[q] = im[q] = 0.0;
            if (q * kLanes >= count(n)) continue;  // the same on all lanes
            const int e = min(l + q * kLanes, count(n) - 1), c = e - in_rows;
            const int i = c < 0 ? kTile + e / n : c / past, j = c < 0 ? e % n : kTile + c % past;
            const T2<T>* a = A + i * ns;
            const T2<T>* b = B + j;
#pragma unroll 4
            for (int k = 0; k < n; ++k) {
                const T2<T> x = a[k], y = b[k * ns];
                cmac(re[q], im[q], (double)x.x, (double)x.y, (double)y.x, (double)y.y);
            }
        }
    }
    // Re sum over the lane's entries of this conj(o)
    __device__ __forceinline__ double dot(const PlaqEdges& o, int n) const {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kMost; ++q)
            if ((int)threadIdx.x + q * kLanes < count(n)) t = fmadd(im[q], o.im[q], fmadd(re[q], o.re[q], t));
        return t;
    }
};

// Sums of site s (as above), one wavefront per tile.
template <typename T, int FORM>
__device__ __forceinline__ void plaquette_site_large(const T2<T>* __restrict__ U, const Geom& g, int n, int s,
                                                     double* __restrict__ partial) {
    constexpr bool BIG = FORM == PLAQ_FOUR;
    constexpr int kThreads = plaq_threads(FORM), kLoads = plaq_loads(FORM);
    extern __shared__ double4 smem_plaq[];
    __shared__ double wave_acc[2 * kThreads / kLanes];
    const int n2 = n * n, ns = row_stride(n);
    T2<T>* const A = reinterpret_cast<T2<T>*>(smem_plaq);
    T2<T>* const B = A + mat_entries(n);
    const Places<kLoads, kThreads> place(n, n2);
    const Site x = site_at(g, s);
    const int u0 = step_shift(g, x, true, 0), u1 = step_shift(g, x, true, 1);
    const int u2 = step_shift(g, x, true, 2), u3 = step_shift(g, x, true, 3);
    const int par = parity_of(x), op = par ^ 1, h = x.s >> 1, Vh = g.Vh;
    LinkPart<T, kLoads, kThreads> fa, fb;
    auto load = [&](int m, int k) {
        fa.load(link_at<T>(U, n2, m, par, h, Vh), n2);
        fb.load(link_at<T>(U, n2, k, op, (x.s + pick_dir(u0, u1, u2, u3, m)) >> 1, Vh), n2);
    };
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLanes);
    const int row0 = BIG ? kTile * (w >> 1) : 0, col0 = BIG ? kTile * (w & 1) : 0;
    if ((n & 1) && (int)threadIdx.x <= n) {  // row and column n of an odd Nc
        const int t = (int)threadIdx.x;
        A[t * ns + n] = A[n * ns + t] = B[t * ns + n] = B[n * ns + t] = cpx<T>(T(0), T(0));
    }
    double space = 0.0, time = 0.0;  // planes without and with direction 3
    Plane pl;
    pl.next(g.present);
    if (!pl.done()) load(pl.mu, pl.nu);
    while (!pl.done()) {
        PlaqTile H, K;
        PlaqEdges he, ke;
        fa.store(A, place);
        fb.store(B, place);
        load(pl.nu, pl.mu);
        __syncthreads();
        H.product<T>(A, B, n, ns, row0, col0);
        if constexpr (FORM == PLAQ_EDGES) he.product<T>(A, B, n, ns);
        __syncthreads();
        fa.store(A, place);
        fb.store(B, place);
        const bool with_time = pl.nu == 3;
        pl.next(g.present);
        if (!pl.done()) load(pl.mu, pl.nu);
        __syncthreads();
        K.product<T>(A, B, n, ns, row0, col0);
        if constexpr (FORM == PLAQ_EDGES) ke.product<T>(A, B, n, ns);
        __syncthreads();
        double t = 0.0;
        const int l = fresh_lane();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (row0 + tile_row<double>(l, r) < n) t = fmadd(H.im[r], K.im[r], fmadd(H.re[r], K.re[r], t));
        if (col0 + (l & 15) >= n) t = 0.0;
        if constexpr (FORM == PLAQ_EDGES) t += he.dot(ke, n);
        (with_time ? time : space) += t;
    }
    const double sums[2] = {wave_sum(space), wave_sum(time)};
    if constexpr (BIG) {
        if ((threadIdx.x & (kLanes - 1)) == 0) {
            wave_acc[2 * w] = sums[0];
            wave_acc[2 * w + 1] = sums[1];
        }
        __syncthreads();
        if (threadIdx.x < 2)
            partial[2 * (size_t)s + threadIdx.x] = (wave_acc[threadIdx.x] + wave_acc[2 + threadIdx.x]) +
                                                   (wave_acc[4 + threadIdx.x] + wave_acc[6 + threadIdx.x]);
    } else if (threadIdx.x == 0) {
        partial[2 * (size_t)s] = sums[0];
        partial[2 * (size_t)s + 1] = sums[1];
    }
}

template <typename T, int FORM>
__global__ __launch_bounds__(plaq_threads(FORM)) void k_plaquette_large(const T2<T>* __restrict__ U, Geom g, int n,
                                                                         double* __restrict__ partial) {
    plaquette_site_large<T, FORM>(U, g, n, xcd_tile((int)blockIdx.x, (int)gridDim.x), partial);
}
// The chains of a batch group that have from .. to - 1 sites.
template <typename T, int FORM>
__global__ __launch_bounds__(plaq_threads(FORM)) void k_plaquette_large_batch(const ChainDesc* __restrict__ d,
                                                                              int nchains, int n, int from, int to) {
    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int c = find_chain<TILE_SITE>(d, nchains, tile);
    if (d[c].g.V < from || d[c].g.V >= to) return;
    plaquette_site_large<T, FORM>((const T2<T>*)d[c].links, d[c].g, n, tile - d[c].tile0[TILE_SITE], d[c].scratch);
}

}  // namespace wide
}  // namespace sun
