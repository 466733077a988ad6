// sun_wide_reunit.hpp -- re-unitarization and the unitarity report of the
// large-Nc path, FP64, one wavefront to four links (Nc <= 8), two (Nc <= 16)
// or one.
//
// The links are in LDS.  The determinant is an LU elimination of a copy in
// registers: lane (link, half, row) keeps the columns 2 j + half of its row,
// the pivot row goes through LDS to the others and is not moved, its row
// number goes into the permutation's sign.  Row Gram-Schmidt writes M = L Q
// with L lower triangular and real positive on its diagonal, so det Q has the
// phase of det M.  Every entry sees the operations of one link per wavefront,
// in their order: the results, and the report's rounding-level deviations,
// are the same bits.
//
// Bound by vector issue and, above Nc = 16, by the LDS that a link's matrix
// takes (nine wavefronts on a CU at Nc = 32).  Against one wavefront per link
// with LU and Gram-Schmidt both in LDS: SU(6) FP32 12^4 234 -> 63 us, SU(8) FP64
// 12^4 356 -> 87, SU(16) 8^4 192 -> 107, SU(24) 8^4 472 -> 360, SU(32) 8^4
// 945 -> 677.  (Gram-Schmidt from the normalized row to the rows below it, all
// in registers, ran SU(8) in 57 and SU(32) in 515 us with other roundings,
// which an FP64 report of deviations at the rounding level shows.)
#pragma once

#include <climits>
#include <utility>

#include "sun_wide.hpp"

namespace sun {
namespace wide {

// ROWS lanes per half of a link, NC columns per lane.
template <int ROWS, int NC>
struct RowLanes {
    static constexpr int kLinks = kLanes / (2 * ROWS);  // links per wavefront
    int link, half, row;
    __device__ __forceinline__ RowLanes() {
        const int l = (int)threadIdx.x;
        row = l % ROWS;
        half = (l / ROWS) & 1;
        link = l / (2 * ROWS);
    }
};

// The value of the lane's partner in the other half.
template <int ROWS>
__device__ __forceinline__ int other_half(int v) {
    if constexpr (ROWS == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false);  // rotate 16 lanes by 8
    if constexpr (ROWS == 16) return partner<4>(v);
    return partner<5>(v);
}
template <int ROWS>
__device__ __forceinline__ double other_half(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)other_half<ROWS>((int)(u & 0xffffffffu));
    const unsigned hi = (unsigned)other_half<ROWS>((int)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// The largest value over the lanes of a link.
template <int ROWS, typename V, typename F>
__device__ __forceinline__ V link_reduce(V v, F op) {
    v = op(v, partner<0>(v));
    v = op(v, partner<1>(v));
    v = op(v, partner<2>(v));
    if constexpr (ROWS >= 16) v = op(v, partner<3>(v));
    if constexpr (ROWS == 32) v = op(v, partner<4>(v));
    return op(v, other_half<ROWS>(v));
}

// One lane's part of a link: entries (row, 2 j + half), zero outside n x n.
template <int NC>
struct RowPart {
    double re[NC], im[NC];
    __device__ __forceinline__ void load(const double2* M, int n, int ns, int row, int half) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = 2 * j + half;
            const bool in = row < n && c < n;
            const double2 v = M[in ? row * ns + c : 0];
            re[j] = in ? v.x : 0.0;
            im[j] = in ? v.y : 0.0;
        }
    }
};

// The row that is passed on: entry j of half h of each link of the wavefront.
template <int ROWS, int NC>
struct PassedRow {
    double2 v[RowLanes<ROWS, NC>::kLinks][2][NC];
};

// det of the link in m (destroyed), the same on all its lanes.  The columns
// are compile-time constants, so that m stays in registers.  A column without
// a pivot makes det 0 for good; its elimination subtracts nothing (1 / 0 in
// place of inv = 0 would put NaN into the rows).  A flag that skipped the
// elimination instead cost SU(16) 8^4 a tenth (107 -> 118 us).
template <int ROWS, int NC, int... COL>
__device__ __forceinline__ void rows_det(RowPart<NC>& m, const RowLanes<ROWS, NC>& ln, PassedRow<ROWS, NC>& pass,
                                         int n, double& dr, double& di, std::integer_sequence<int, COL...>) {
    dr = 1.0;
    di = 0.0;
    uint32_t unused = n == 32 ? 0xFFFFFFFFu : (1u << n) - 1u;  // rows that were no pivot yet
    double2* const mine = pass.v[ln.link][ln.half];
    auto eliminate = [&](auto col) {
        constexpr int j0 = decltype(col)::value >> 1, hc = decltype(col)::value & 1;
        if (decltype(col)::value >= n) return false;
        // the pivot: the largest |m|^2 of the column, the lowest row among
        // equals; non-negative doubles compare as their two words
        const double a = fmadd(m.re[j0], m.re[j0], m.im[j0] * m.im[j0]);
        const unsigned long long bits = __builtin_bit_cast(unsigned long long, a);
        const bool can = ln.half == hc && ((unused >> ln.row) & 1);
        const int hi = can ? (int)(bits >> 32) & 0x7FFFFFFF : -1;
        const int best_hi = link_reduce<ROWS>(hi, [](int x, int y) { return max(x, y); });
        const int lo = hi == best_hi ? (int)((uint32_t)bits ^ 0x80000000u) : INT_MIN;  // unsigned order
        const int best_lo = link_reduce<ROWS>(lo, [](int x, int y) { return max(x, y); });
        const unsigned long long hits = __ballot(hi == best_hi && lo == best_lo) >> (2 * ROWS * ln.link + ROWS * hc);
        const int piv = __ffsll(hits & (ROWS == 32 ? 0xFFFFFFFFull : (1ull << (ROWS & 31)) - 1ull)) - 1;
        if (ln.row == piv)
#pragma unroll
            for (int j = j0; j < NC; ++j) mine[j] = make_double2(m.re[j], m.im[j]);
        // the lane's entry of the column, in both halves
        const double orr = other_half<ROWS>(m.re[j0]), oi = other_half<ROWS>(m.im[j0]);
        const double er = ln.half == hc ? m.re[j0] : orr, ei = ln.half == hc ? m.im[j0] : oi;
        wave_lds_order();
        const double2 p = pass.v[ln.link][hc][j0];
        const double pm = fmadd(p.x, p.x, p.y * p.y);
        const double inv = pm >= DBL_MIN ? newton_rcp(pm) : pm > 0.0 ? 1.0 / pm : 0.0;
        const double fr = fmadd(ei, p.y, er * p.x) * inv, fi = fmadd(ei, p.x, -(er * p.y)) * inv;
        if (ln.row != piv)
#pragma unroll
            for (int j = j0; j < NC; ++j) {
                const double2 u = mine[j];
                m.re[j] -= fmadd(fr, u.x, -(fi * u.y));
                m.im[j] -= fmadd(fr, u.y, fi * u.x);
            }
        wave_lds_order();
        const double nr = fmadd(dr, p.x, -(di * p.y)), ni = fmadd(di, p.x, dr * p.y);
        const bool odd = __popc(unused & ((1u << piv) - 1u)) & 1;
        dr = odd ? -nr : nr;
        di = odd ? -ni : ni;
        if (best_hi <= 0 && best_lo == INT_MIN) dr = di = 0.0;  // no pivot left in the column
        unused &= ~(1u << piv);
        return true;
    };
    (void)(eliminate(std::integral_constant<int, COL>{}) && ...);
}

// Gram-Schmidt on all rows of M (LDS, row stride ns), then the last row times
// conj(det) / |det| (paper Sec. 2, re-unitarization; Nc > 3).  Each row is
// orthogonalized against the earlier ones by classical Gram-Schmidt, with a
// second pass where the first removed more than half the row's squared norm
// (Daniel, Gragg, Kaufman and Stewart, Math. Comp. 30 (1976): twice is enough,
// as stable as the modified form): lane k forms <r_k, r_i>, then lane c
// subtracts every projection from column c of r_i, so a row costs two LDS
// hand-offs per pass.  P (n entries per link) holds the projections.  Above
// Nc = 8 the halves share each sum; below, both form all of it.
template <int ROWS, int NC>
__device__ __forceinline__ void rows_reunit(double2* M, double2* P, const RowLanes<ROWS, NC>& ln, int n, int ns,
                                            double dr, double di) {
    constexpr bool kSplit = ROWS > 8;
    const int q = ln.row;
    const bool own = q < n;
    const int m0 = kSplit ? n / 2 : n;  // columns of the lower half
    const int upper = kSplit ? ln.half : 0;
    const int cbeg = upper ? m0 : 0, clen = upper ? n - m0 : m0;
    // |r|^2 of the row whose column q the lane holds
    auto norm2 = [&](const double2& r) {
        double v = own ? fmadd(r.y, r.y, r.x * r.x) : 0.0;
        v = v + partner<0>(v);
        v = v + partner<1>(v);
        v = v + partner<2>(v);
        if constexpr (ROWS >= 16) v = v + partner<3>(v);
        if constexpr (ROWS == 32) v = v + partner<4>(v);
        return v;
    };
    // one classical pass: r_i -= sum_{k < i} <r_k, r_i> r_k
    auto project = [&](int i, const double2& b) {
        // p_q = <r_q, r_i> for q < i; columns taken from a lane-dependent
        // start within the half's range, so lanes hit different banks
        double pr = 0.0, pi = 0.0;
        if (q < i && clen > 0) {
            int t = q % clen;
#pragma unroll 4
            for (int u = 0; u < clen; ++u) {
                const int c = cbeg + t;
                const double2 a = M[q * ns + c], r = M[i * ns + c];
                cmac(pr, pi, a.x, -a.y, r.x, r.y);
                t = (t + 1 == clen) ? 0 : t + 1;
            }
        }
        if constexpr (kSplit) {
            pr += other_half<ROWS>(pr);
            pi += other_half<ROWS>(pi);
        }
        if (q < i && ln.half == 0) P[q] = make_double2(pr, pi);
        wave_lds_order();
        // r_i -= sum_{k < i} p_k r_k, the k range split between the halves
        double sr = 0.0, si = 0.0;
        if (own) {
            const int kmid = kSplit ? i / 2 : i;
            const int kb = upper ? kmid : 0, ke = upper ? i : kmid;
#pragma unroll 4
            for (int k = kb; k < ke; ++k) {
                const double2 p = P[k], a = M[k * ns + q];
                cmac(sr, si, p.x, p.y, a.x, a.y);
            }
        }
        if constexpr (kSplit) {
            sr += other_half<ROWS>(sr);
            si += other_half<ROWS>(si);
        }
        return make_double2(b.x - sr, b.y - si);
    };
    for (int i = 0; i < n; ++i) {
        double2 r = M[i * ns + (own ? q : 0)];
        const double s0 = norm2(r);
        double s2 = s0;
        if (i > 0) {
            // a second pass only where the first removed more than half of
            // the row's squared norm (the DGKS criterion): a row of a nearly
            // unitary link keeps almost all of it
            r = project(i, r);
            s2 = norm2(r);
            const bool twice = s2 < 0.5 * s0;  // the same on all lanes of a link
            if (__any(twice)) {
                if (own && ln.half == 0) M[i * ns + q] = r;
                wave_lds_order();
                const double2 r2 = project(i, r);
                if (twice) {
                    r = r2;
                    s2 = norm2(r2);
                }
            }
        }
        const double inv = s2 >= DBL_MIN ? newton_rsqrt(s2) : rsqrt(s2);
        r.x *= inv;
        r.y *= inv;
        if (i == n - 1) {
            const double mod = sqrt(fmadd(dr, dr, di * di));
            const double cr = dr / mod, ci = -di / mod;
            r = make_double2(fmadd(cr, r.x, -(ci * r.y)), fmadd(ci, r.x, cr * r.y));
        }
        if (own && ln.half == 0) M[i * ns + q] = r;
        wave_lds_order();
    }
}

// max_ij |(M^dag M - 1)_ij| of the lane's link, M (n x n) in LDS: entries
// (i, i + d mod n) for d = 0 .. n / 2, one i per lane, the halves taking
// alternate d (the matrix is Hermitian; each is formed in the upper triangle).
template <int ROWS, int NC>
__device__ __forceinline__ double rows_unitarity_dev(const double2* M, const RowLanes<ROWS, NC>& ln, int n, int ns) {
    double du2 = 0.0;
    const int i = ln.row;
    if (i < n)
        for (int d = ln.half; 2 * d <= n; d += 2) {
            const int j = i + d < n ? i + d : i + d - n;
            const int c0 = min(i, j), c1 = max(i, j);
            double r = d == 0 ? -1.0 : 0.0, m = 0.0;
            for (int k = 0; k < n; ++k) {
                const double2 a = M[k * ns + c0], b = M[k * ns + c1];
                cmac(r, m, a.x, -a.y, b.x, b.y);
            }
            du2 = fmax(du2, nan_to_inf(fmadd(m, m, r * r)));  // a NaN entry counts as infinite
        }
    return sqrt(link_reduce<ROWS>(du2, [](double x, double y) { return fmax(x, y); }));
}

// What a launch does with its links.
enum ReunitMode { REUNIT_PLAIN, REUNIT_REPORT, UNITARITY_ONLY };

// LDS: the row that is passed on, then each link's projections and matrix
// (odd row stride: rows start in different banks).
__host__ __device__ constexpr int rows_stride(int n) { return n | 1; }
template <int ROWS, int NC>
constexpr size_t rows_lds(int n) {
    return sizeof(PassedRow<ROWS, NC>) +
           (size_t)RowLanes<ROWS, NC>::kLinks * (ROWS + n * rows_stride(n)) * sizeof(double2);
}

// Links kLinks wg .. of one lattice (ids in [0, 4V)); with a report partial[2 wg
// ..] gets the largest deviations {|U^dag U - 1|, |det U - 1|} found before the
// projection.
template <typename T, int ROWS, int NC, int MODE>
__device__ __forceinline__ void reunit_links(T2<T>* __restrict__ U, const Geom& g, int n, int wg,
                                             double* __restrict__ partial) {
    using Lanes = RowLanes<ROWS, NC>;
    extern __shared__ double4 smem_rows[];
    PassedRow<ROWS, NC>& pass = *reinterpret_cast<PassedRow<ROWS, NC>*>(smem_rows);
    const Lanes ln;
    const int n2 = n * n, ns = rows_stride(n), first = wg * Lanes::kLinks, most = 4 * g.V - 1;
    const int inv = ((1 << 16) + n - 1) / n;  // e / n = (e inv) >> 16 for e < 1024
    double2* const proj = reinterpret_cast<double2*>(&pass + 1);
    double2* const mats = proj + Lanes::kLinks * ROWS;
    double2* const P = proj + ln.link * ROWS;
    double2* const M = mats + ln.link * n * ns;
    // link k of the wavefront (the last one past the end), and whether it is to
    // be touched
    auto link_of_wave = [&](int k, bool& live) {
        const int id = min(first + k, most);
        int mu, par, h;
        link_id(g, id, mu, par, h);
        live = first + k <= most && ((g.present >> mu) & 1);
        return const_cast<T2<T>*>(link_at<T>(U, n2, mu, par, h, g.Vh));
    };
    bool live = false;
#pragma unroll
    for (int k = 0; k < Lanes::kLinks; ++k) {
        bool touch;
        const T2<T>* src = link_of_wave(k, touch);
        if (k == ln.link) live = touch;
#pragma unroll 8
        for (int e = threadIdx.x; e < n2; e += kLanes) {
            const T2<T> v = src[e];
            mats[k * n * ns + e + (ns - n) * ((e * inv) >> 16)] = make_double2(v.x, v.y);
        }
    }
    wave_lds_order();
    double du = 0.0;
    if constexpr (MODE != REUNIT_PLAIN) du = rows_unitarity_dev<ROWS, NC>(M, ln, n, ns);
    double dr, di;
    {
        RowPart<NC> m;
        m.load(M, n, ns, ln.row, ln.half);
        rows_det(m, ln, pass, n, dr, di, std::make_integer_sequence<int, 2 * NC>{});
    }
    if constexpr (MODE != UNITARITY_ONLY) {
        rows_reunit<ROWS, NC>(M, P, ln, n, ns, dr, di);
#pragma unroll
        for (int k = 0; k < Lanes::kLinks; ++k) {
            bool touch;
            T2<T>* dst = link_of_wave(k, touch);
            if (touch)
                for (int e = threadIdx.x; e < n2; e += kLanes) {
                    const double2 v = mats[k * n * ns + e + (ns - n) * ((e * inv) >> 16)];
                    dst[e] = cpx<T>((T)v.x, (T)v.y);
                }
        }
    }
    if constexpr (MODE != REUNIT_PLAIN) {
        const double dd = nan_to_inf(sqrt(fmadd(di, di, (dr - 1.0) * (dr - 1.0))));
        const double u = wave_max(live ? du : 0.0), d = wave_max(live ? dd : 0.0);
        if (threadIdx.x == 0) {
            partial[2 * (size_t)wg] = u;
            partial[2 * (size_t)wg + 1] = d;
        }
    }
}

template <typename T, int ROWS, int NC, int MODE>
__global__ __launch_bounds__(kLanes, NC > 12 ? 3 : 4) void k_reunit_rows(T2<T>* __restrict__ U, Geom g, int n,
                                                           double* __restrict__ partial) {
    reunit_links<T, ROWS, NC, MODE>(U, g, n, (int)blockIdx.x, partial);
}

// Re-unitarization of every chain of a batch group (TILE_LINK counts
// workgroups here).
template <typename T, int ROWS, int NC>
__global__ __launch_bounds__(kLanes, NC > 12 ? 3 : 4) void k_reunit_rows_batch(const ChainDesc* __restrict__ d, int nchains, int n) {
    const int c = find_chain<TILE_LINK>(d, nchains, (int)blockIdx.x);
    reunit_links<T, ROWS, NC, REUNIT_PLAIN>((T2<T>*)d[c].links, d[c].g, n, (int)blockIdx.x - d[c].tile0[TILE_LINK],
                                            nullptr);
}

}  // namespace wide
}  // namespace sun
