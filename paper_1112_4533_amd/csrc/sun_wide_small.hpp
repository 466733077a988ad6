// sun_wide_small.hpp -- the large-Nc phase update for 4 <= Nc <= 8: four
// links to a wavefront, sixteen lanes to a link.
//
// A link of this size leaves most of a wavefront idle when it has one to
// itself: its products have Nc rows and its subgroup steps Nc columns.  Here
// lane 8 h + r of a link's sixteen takes, in the products, row r and column
// half h (the left factor's row in registers, the right factor read from LDS
// by broadcast), and in the subgroup steps column r of W = U A (h = 0) or of
// U (h = 1), so that one instruction serves four links and every product
// entry stays the sum over k in increasing k that one lane forms.  Nc is a
// template argument: the rows live in registers.
//
// Bound by vector issue and, in FP64, by LDS reads of the broadcast factors
// (each read serves four fused multiply-adds).  Against one wavefront per
// link, 12^4: SU(6) FP32 overrelaxation 65 -> 17 us a phase, heatbath
// 93 -> 23 us; SU(8) FP64 145 -> 49 and 266 -> 81 us; on 8^4, where the phase
// is one link's latency, SU(6) FP32 20 -> 11.5 and 28 -> 15.6 us.
#pragma once

#include <type_traits>

#include "sun_wide.hpp"

namespace sun {
namespace wide {

constexpr int kSmallMax = 8;    // largest Nc of this form
constexpr int kSmallLinks = 4;  // links per wavefront
static_assert(kSmallLinks * kPlaceLanes == kLanes, "sixteen lanes per link");

template <typename T, int N>
struct SmallShape {
    static_assert(N >= kNcMin && N <= kSmallMax, "Nc of the four-link form");
    static constexpr int kHalf = (N + 1) / 2;  // columns of half 0 (half 1 has N - kHalf)
    static constexpr int kSteps = N * (N - 1) / 2;
    static constexpr int kChunk = kSteps < kPlaceLanes ? kSteps : kPlaceLanes;  // steps whose draws are in hand
    static constexpr int kLoads = (N * N + kPlaceLanes - 1) / kPlaceLanes;  // entries of a link per lane
    // Row stride: even in FP32, so that a row is read two entries (16 bytes)
    // at a time, and such that the rows the two halves read together, kHalf
    // apart, start in different banks.
    static constexpr int kRow = sizeof(T) == 4 ? (N <= 6 ? N + N % 2 : 10) : (N == 4 || N == 8 ? N + 1 : N);
    // Matrix stride: N rows and the columns read past a row's end, 8 mod 16
    // entries, so that W and U (and the links) spread over the banks.
    static constexpr int kMat = ((N * kRow + N + 7) / 16) * 16 + 8;
    static_assert(kMat >= N * kRow + N, "odd Nc reads one row past the matrix");
};

// LDS of one link: the three factors of a staple term; after the staples W
// = U A, U, and (heatbath) the draw records of the next subgroup steps.  Its
// size is half of the banks past their multiple, so that neighbouring links'
// matrices start in different banks (SU(8) FP64 12^4 sweep step 1239 us at a
// multiple, 1196 like this).
template <typename T, int N>
struct alignas(16) SmallLds {
    static constexpr int kMatBytes = SmallShape<T, N>::kMat * sizeof(T2<T>);
    static constexpr int kDrawBytes = SmallShape<T, N>::kChunk * sizeof(DrawRec<T, kQuickHits>);
    static constexpr int kUsed = 2 * kMatBytes + (kMatBytes > kDrawBytes ? kMatBytes : kDrawBytes);
    static constexpr int kTail = (kUsed + 127) / 256 * 256 + 128 - 2 * kMatBytes;
    T2<T> q[SmallShape<T, N>::kMat], r[SmallShape<T, N>::kMat];
    union {
        T2<T> left[SmallShape<T, N>::kMat];
        DrawRec<T, kQuickHits> draw[SmallShape<T, N>::kChunk];
        char fill[kTail];
    };
};
template <typename T, int N>
constexpr size_t small_lds() {
    return kSmallLinks * sizeof(SmallLds<T, N>);
}

// A link's entries e = lane mod 16 + 16 c, from memory to registers and from
// there to an LDS matrix.
template <typename T, int N>
struct LinkRegs {
    T re[SmallShape<T, N>::kLoads], im[SmallShape<T, N>::kLoads];
    __device__ __forceinline__ void load(const T2<T>* __restrict__ src, int q) {
#pragma unroll
        for (int c = 0; c < SmallShape<T, N>::kLoads; ++c) {
            const int e = q + kPlaceLanes * c;
            const T2<T> v = src[e < N * N ? e : N * N - 1];
            re[c] = v.x;
            im[c] = v.y;
        }
    }
    __device__ __forceinline__ void store(T2<T>* dst, int q) const {
        constexpr int kRow = SmallShape<T, N>::kRow;
#pragma unroll
        for (int c = 0; c < SmallShape<T, N>::kLoads; ++c) {
            const int e = q + kPlaceLanes * c;
            if (e < N * N) dst[(e / N) * kRow + e % N] = cpx<T>(re[c], im[c]);
        }
    }
};

// Value of v's partner half: lanes 0 .. 7 of a link's sixteen hold half 0 of
// a row, lanes 8 .. 15 half 1.  from_half<0> gives every lane half 0's value,
// from_half<1> half 1's.
template <int H>
__device__ __forceinline__ int from_half(int v) {
    // row_shr:8 / row_shl:8; lanes without a source keep their own
    return __builtin_amdgcn_update_dpp(v, v, H == 0 ? 0x118 : 0x108, 0xF, 0xF, false);
}
template <int H>
__device__ __forceinline__ float from_half(float v) {
    return __builtin_bit_cast(float, from_half<H>(__builtin_bit_cast(int, v)));
}
template <int H>
__device__ __forceinline__ double from_half(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)from_half<H>((int)(u & 0xffffffffu));
    const unsigned hi = (unsigned)from_half<H>((int)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// acc[j] += sum_k left[k] B_kj over the lane's columns j = j0 .. j0 + kHalf - 1
// (columns past N - 1 give values nobody reads), B the LDS matrix m:
// DAG: B = m^dag (its row k is column k of m, conjugated), else B = m.
// CONJ: left holds the conjugates of the left factor's row.
template <bool DAG, typename T, int N, bool CONJ, typename V, int H>
__device__ __forceinline__ void row_times(V (&acc)[H], const V (&left)[N], const V* m, int j0) {
    constexpr int kRow = SmallShape<T, N>::kRow;
#pragma unroll
    for (int j = 0; j < H; ++j) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const V b = DAG ? m[(j0 + j) * kRow + k] : m[k * kRow + j0 + j];
            cmac(acc[j].x, acc[j].y, left[k].x, CONJ ? -left[k].y : left[k].y, b.x, DAG ? -b.y : b.y);
        }
    }
}

// One phase of four links h0 .. h0 + 3 (those below Vh) of one lattice.
template <typename T, int N>
__device__ __forceinline__ void update_links_small(T2<T>* __restrict__ U, const Geom& g, int mu, int par, int hb,
                                                   T beta, uint32_t k0, uint32_t k1, uint32_t step, int h0) {
    using S = SmallShape<T, N>;
    constexpr int kHalf = S::kHalf, kRow = S::kRow, n2 = N * N;
    extern __shared__ double4 smem_small[];
    const int lane = threadIdx.x;
    const int p = lane / kPlaceLanes, q = lane % kPlaceLanes;  // link of the four, lane of the sixteen
    const int half = q >> 3, r8 = q & 7;
    const int r = r8 < N ? r8 : N - 1;  // idle lanes repeat the last row
    const int j0 = half * kHalf;
    const bool live = h0 + p < g.Vh;
    const int h = live ? h0 + p : g.Vh - 1;
    SmallLds<T, N>& lds = reinterpret_cast<SmallLds<T, N>*>(smem_small)[p];
    T2<T>* const Q = lds.q;
    T2<T>* const R = lds.r;
    T2<T>* const F = lds.left;
    const int Vh = g.Vh;
    const Site x = site_of(g, par, h);
    const int op = par ^ 1;
    const int u0 = step_shift(g, x, true, 0), u1 = step_shift(g, x, true, 1);
    const int u2 = step_shift(g, x, true, 2), u3 = step_shift(g, x, true, 3);
    const int d0 = step_shift(g, x, false, 0), d1 = step_shift(g, x, false, 1);
    const int d2 = step_shift(g, x, false, 2), d3 = step_shift(g, x, false, 3);
    const int sp = x.s + pick_dir(u0, u1, u2, u3, mu);  // x + mu

    // Loads run one staple term ahead of the arithmetic, in the registers of
    // the sixteen lanes.
    LinkRegs<T, N> fl, fq, fr;
    auto load_upper = [&](int nu) {
        const int spn = x.s + pick_dir(u0, u1, u2, u3, nu);
        fl.load(link_at<T>(U, n2, nu, op, sp >> 1, Vh), q);
        fq.load(link_at<T>(U, n2, mu, op, spn >> 1, Vh), q);
        fr.load(link_at<T>(U, n2, nu, par, h, Vh), q);
    };
    auto load_lower = [&](int nu) {
        const int sh = pick_dir(d0, d1, d2, d3, nu);  // the same from x + mu: nu is another direction
        const int smn = x.s + sh;
        fl.load(link_at<T>(U, n2, nu, par, (sp + sh) >> 1, Vh), q);
        fq.load(link_at<T>(U, n2, mu, op, smn >> 1, Vh), q);
        fr.load(link_at<T>(U, n2, nu, op, smn >> 1, Vh), q);
    };
    auto stage = [&] {
        fl.store(F, q);
        fq.store(Q, q);
        fr.store(R, q);
    };
    auto next_dir = [&](int nu) {
        do ++nu;
        while (nu < 4 && (nu == mu || !((g.present >> nu) & 1)));
        return nu;
    };

    int nu = next_dir(-1);
    if (nu < 4)
        load_upper(nu);
    else
        fr.load(link_at<T>(U, n2, mu, par, h, Vh), q);
    T2<T> acc[kHalf];  // row r of the staple sum, the half's columns
#pragma unroll
    for (int j = 0; j < kHalf; ++j) acc[j] = cpx<T>(T(0), T(0));
    // the lane's columns of row r of F Q^dag (dag: F^dag Q^dag), then the
    // whole row from both halves
    auto first_product = [&](auto dag, T2<T>(&row)[N]) {
        constexpr bool kDag = decltype(dag)::value;
        T2<T> m[kHalf], left[N];
#pragma unroll
        for (int k = 0; k < N; ++k) left[k] = kDag ? F[k * kRow + r] : F[r * kRow + k];
#pragma unroll
        for (int j = 0; j < kHalf; ++j) m[j] = cpx<T>(T(0), T(0));
        row_times<true, T, N, kDag>(m, left, Q, j0);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const T2<T> v = m[k < kHalf ? k : k - kHalf];
            row[k] = k < kHalf ? cpx<T>(from_half<0>(v.x), from_half<0>(v.y))
                               : cpx<T>(from_half<1>(v.x), from_half<1>(v.y));
        }
    };
    while (nu < 4) {
        T2<T> row[N];
        // upper staple U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
        stage();
        load_lower(nu);
        wave_lds_order();
        first_product(std::false_type{}, row);
        row_times<true, T, N, false>(acc, row, R, j0);
        wave_lds_order();
        // lower staple U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
        stage();
        nu = next_dir(nu);
        if (nu < 4)
            load_upper(nu);
        else
            fr.load(link_at<T>(U, n2, mu, par, h, Vh), q);  // the link itself
        wave_lds_order();
        first_product(std::true_type{}, row);
        row_times<false, T, N, false>(acc, row, R, j0);
        wave_lds_order();
    }
    // W = U A: A through Q, U into R; lane (half, r) forms column r, rows
    // half * kHalf ..., each entry the sum over k of U_ik A_kr
    fr.store(R, q);
    if (r8 < N)
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
            if (j0 + j < N) Q[r * kRow + j0 + j] = acc[j];
    wave_lds_order();
    {
        T2<T> a[N], w[kHalf];
#pragma unroll
        for (int k = 0; k < N; ++k) a[k] = Q[k * kRow + r];
#pragma unroll
        for (int i = 0; i < kHalf; ++i) {
            w[i] = cpx<T>(T(0), T(0));
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const T2<T> u = R[(j0 + i) * kRow + k];
                cmac(w[i].x, w[i].y, u.x, u.y, a[k].x, a[k].y);
            }
        }
        wave_lds_order();
        if (r8 < N)
#pragma unroll
            for (int i = 0; i < kHalf; ++i)
                if (j0 + i < N) Q[(j0 + i) * kRow + r] = w[i];
    }
    wave_lds_order();

    // The subgroup steps in their fixed order, one per link at a time: lane
    // (half, r) owns column r of W (half 0) or U (half 1).
    const T cb = T(2) * beta / T(N);  // alpha = 2 beta k / n
    T2<T>* const col = (half ? R : Q) + r;
    const uint32_t mu_hi = (uint32_t)mu << 16;
    int t = 0;
    for (int i = 0; i < N - 1; ++i)
        for (int j = i + 1; j < N; ++j, ++t) {
            const T2<T> wii = Q[i * kRow + i], wij = Q[i * kRow + j], wji = Q[j * kRow + i], wjj = Q[j * kRow + j];
            const T2<T> ci = col[i * kRow], cj = col[j * kRow];
            Quat<T> pq, v, a;
            pq.q[0] = T(0.5) * (wii.x + wjj.x);
            pq.q[3] = T(0.5) * (wii.y - wjj.y);
            pq.q[2] = T(0.5) * (wij.x - wji.x);
            pq.q[1] = T(0.5) * (wij.y + wji.y);
            const T k = chain_unit_quat(pq, v);
            bool apply = true;
            if (hb) {
                // the draws' terms that need no alpha, sixteen steps at a time
                if (t % kPlaceLanes == 0) {
                    fill_draws<T>(lds.draw, min(kPlaceLanes, S::kSteps - t), (uint32_t)t, k0, k1, (uint32_t)x.s, step,
                                  mu_hi);
                    wave_lds_order();
                }
                Quat<T> xs;
                apply = place_draw<T>(cb * k, true, lds.draw[t % kPlaceLanes], k0, k1, (uint32_t)x.s, step, mu_hi | (uint32_t)t,
                                      xs) != 0;
                a = qmul(xs, qconj(v));
            } else {
                const Quat<T> vc = qconj(v);
                a = qmul(vc, vc);
            }
            if (apply && r8 < N) rows_left_mul_at<T>(col + i * kRow, col + j * kRow, a, ci, cj);
            wave_lds_order();
        }
    if (live) {
        T2<T>* dst = const_cast<T2<T>*>(link_at<T>(U, n2, mu, par, h, Vh));
#pragma unroll
        for (int c = 0; c < S::kLoads; ++c) {
            const int e = q + kPlaceLanes * c;
            if (e < n2) dst[e] = R[(e / N) * kRow + e % N];
        }
    }
}

// One phase of one lattice, workgroups in the XCD-aware order: neighbouring
// links are read by neighbouring workgroups, so each XCD takes one contiguous
// share of them.
template <typename T, int N>
__global__ __launch_bounds__(kLanes, 2) void k_update_small(T2<T>* __restrict__ U, Geom g, int mu, int par, int hb,
                                                         T beta, uint32_t k0, uint32_t k1, uint32_t step) {
    update_links_small<T, N>(U, g, mu, par, hb, beta, k0, k1, step,
                             kSmallLinks * xcd_tile((int)blockIdx.x, (int)gridDim.x));
}

// One phase of every chain of a batch group (TILE_HALF_HB counts workgroups
// of kSmallLinks links here).
template <typename T, int N>
__global__ __launch_bounds__(kLanes, 2) void k_update_small_batch(const ChainDesc* __restrict__ d, int nchains, int mu,
                                                               int par, int hb, uint32_t step_offset) {
    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int c = find_chain<TILE_HALF_HB>(d, nchains, tile);
    const Geom g = d[c].g;
    if (!((g.present >> mu) & 1)) return;
    update_links_small<T, N>((T2<T>*)d[c].links, g, mu, par, hb, (T)d[c].beta, d[c].k0, d[c].k1,
                             (uint32_t)(d[c].step + step_offset), kSmallLinks * (tile - d[c].tile0[TILE_HALF_HB]));
}

}  // namespace wide
}  // namespace sun
