// sun_quad.hpp -- the phase update of small lattices (Nc <= 4): four lanes to a
// link.
//
// With one link per work-item a phase of a small lattice is a wavefront or
// less per SIMD, and its time is that of one work-item: all the staple's
// loads, the products and the subgroup steps one after another.  Here the
// four lanes of a quad share a link.  SU(3), SU(4): lane r forms row r of the
// staple sum -- its row (column) of the left factor in registers, the entries
// of the others from the lanes that loaded them, by quad broadcasts -- and then
// owns column r of U and of W = U A, so that a lane loads Nc entries of a
// neighbour instead of Nc^2, all nineteen links' loads are issued at once and
// every entry is still formed by one lane in the order of the one-lane form.
// SU(2): lane l forms the two staples of the l-th direction, which every lane
// then adds in the fixed order.  Heatbath: lanes 0 .. 2 try the first three
// attempts, lane 3 draws the direction; rejected quads try four more at a
// time.  The lowest accepting attempt wins, as in the sequential draw: the
// link has the same bits.
//
// What bounds it: the dependent instructions of one wavefront (FP32 SU(3)
// overrelaxation: 1300 vector instructions, 2.2 us if nothing waits) behind
// two memory latencies; 8^4 SU(3) 9.0 -> 4.5 us a phase, SU(2) 4.6 -> 2.9 (a
// launch alone takes about 2).  A fifth of the instructions are quad broadcasts:
// a multiply-add takes no lane-permuted operand here.
#pragma once

#include <type_traits>

#include "sun_kernels.hpp"
#include "sun_ops.hpp"

namespace sun {
namespace quad {

constexpr int kBlockItems = 64;                // one wavefront per workgroup
constexpr int kLinks = kBlockItems / 4;        // links per workgroup
static_assert(kLinks == kQuadLinks, "host and device agree");

// v of lane PA, PB, PC, PD of the quad in its lanes 0 .. 3.
template <int PA, int PB, int PC, int PD>
__device__ __forceinline__ int perm(int v) {
    return __builtin_amdgcn_mov_dpp(v, PA | PB << 2 | PC << 4 | PD << 6, 0xF, 0xF, true);
}
template <int PA, int PB, int PC, int PD>
__device__ __forceinline__ uint32_t perm(uint32_t v) {
    return (uint32_t)perm<PA, PB, PC, PD>((int)v);
}
template <int PA, int PB, int PC, int PD>
__device__ __forceinline__ float perm(float v) {
    return __builtin_bit_cast(float, perm<PA, PB, PC, PD>(__builtin_bit_cast(int, v)));
}
template <int PA, int PB, int PC, int PD>
__device__ __forceinline__ double perm(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)perm<PA, PB, PC, PD>((int)(u & 0xffffffffu));
    const unsigned hi = (unsigned)perm<PA, PB, PC, PD>((int)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// v of lane SRC in the whole quad
template <int SRC, typename V>
__device__ __forceinline__ V from(V v) {
    return perm<SRC, SRC, SRC, SRC>(v);
}
// v of lane src of the quad (the same src on its four lanes)
template <typename V>
__device__ __forceinline__ V from_first(V v, int src) {
    const V a = from<0>(v), b = from<1>(v), c = from<2>(v), d = from<3>(v);
    return src == 0 ? a : src == 1 ? b : src == 2 ? c : d;
}

// N complex numbers of a lane: its row or its column of a matrix.
template <int N, typename T>
struct Vec {
    T re[N], im[N];
};
template <int SRC, int N, typename T>
__device__ __forceinline__ Vec<N, T> from(const Vec<N, T>& v) {
    Vec<N, T> r;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        r.re[k] = from<SRC>(v.re[k]);
        r.im[k] = from<SRC>(v.im[k]);
    }
    return r;
}

// conj(p x q) component from p_a, p_b, q_a, q_b: the operations of
// third_row_entry.
template <typename T>
__device__ __forceinline__ void cross_entry(T par, T pai, T pbr, T pbi, T qar, T qai, T qbr, T qbi, T& re, T& im) {
    T xr = par * qbr, xi = par * qbi;
    xr = fmadd(-pai, qbi, xr);
    xi = fmadd(pai, qbr, xi);
    xr = fmadd(-pbr, qar, xr);
    xi = fmadd(-pbr, qai, xi);
    xr = fmadd(pbi, qai, xr);
    xi = fmadd(-pbi, qar, xi);
    re = xr;
    im = -xi;
}

// The field, addressed by 32-bit byte offsets (the host checks that they fit).
template <int N, typename T, int R>
struct Field {
    static constexpr uint32_t kEntry = sizeof(T2<T>);
    static constexpr uint32_t E = Planes<N, R>::E;
    const char* base;
    uint32_t Vh;
    __device__ __forceinline__ uint32_t plane(uint32_t mu, uint32_t par, uint32_t e) const {
        return (mu * 2 + par) * E + e;
    }
    __device__ __forceinline__ T2<T> entry(uint32_t pl, uint32_t h) const {
        return *reinterpret_cast<const T2<T>*>(base + (pl * Vh + h) * kEntry);
    }
    // column r of link (mu, par, h): entries (k, r), the stored rows only
    __device__ __forceinline__ Vec<N, T> col(int mu, int par, int h, int r) const {
        Vec<N, T> v;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if (k >= R) {
                v.re[k] = v.im[k] = T(0);
                continue;
            }
            const T2<T> e = entry(plane(mu, par, k * N + r), h);
            v.re[k] = e.x;
            v.im[k] = e.y;
        }
        return v;
    }
    // row r (lanes past the stored rows repeat the last one)
    __device__ __forceinline__ Vec<N, T> row(int mu, int par, int h, int r) const {
        Vec<N, T> v;
        const uint32_t rs = r < R ? r : R - 1;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const T2<T> e = entry(plane(mu, par, rs * N + k), h);
            v.re[k] = e.x;
            v.im[k] = e.y;
        }
        return v;
    }
};

// Row 2 of a two-row link from the columns the quad holds (lane c: column c).
template <int N, typename T, int R>
__device__ __forceinline__ void complete_col(Vec<N, T>& v) {
    if constexpr (R < N) {
        // entry c = conj(row0 x row1)_c, from columns a = c + 1, b = c + 2 mod 3
        cross_entry(perm<1, 2, 0, 0>(v.re[0]), perm<1, 2, 0, 0>(v.im[0]), perm<2, 0, 1, 1>(v.re[0]),
                    perm<2, 0, 1, 1>(v.im[0]), perm<1, 2, 0, 0>(v.re[1]), perm<1, 2, 0, 0>(v.im[1]),
                    perm<2, 0, 1, 1>(v.re[1]), perm<2, 0, 1, 1>(v.im[1]), v.re[2], v.im[2]);
    }
}
// Row 2, in lanes 2 and 3, from rows 0 and 1 of lanes 0 and 1 (SU(3)).
template <typename T>
__device__ __forceinline__ void complete_row(Vec<3, T>& v, int r) {
    const Vec<3, T> p = from<0>(v), q = from<1>(v);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int a = (c + 1) % 3, b = (c + 2) % 3;
        T re, im;
        cross_entry(p.re[a], p.im[a], p.re[b], p.im[b], q.re[a], q.im[a], q.re[b], q.im[b], re, im);
        v.re[c] = r >= 2 ? re : v.re[c];
        v.im[c] = r >= 2 ? im : v.im[c];
    }
}

// acc[j] += sum_k left[k] B_kj with B the matrix the quad holds by columns
// (lane c: column c): DAG: B = m^dag, entries conj(m_jk) of lane k; else B = m,
// entries m_kj of lane j.  CONJ: left holds the conjugates.
template <bool DAG, bool CONJ, int N, typename T, int K = 0>
__device__ __forceinline__ void row_times(Vec<N, T>& acc, const Vec<N, T>& left, const Vec<N, T>& m) {
    if constexpr (K < N) {
        // the k-th term of every entry; the terms of one entry stay in order
        if constexpr (DAG) {
            const Vec<N, T> b = from<K>(m);  // b[j] = m_jK
#pragma unroll
            for (int j = 0; j < N; ++j)
                cmac(acc.re[j], acc.im[j], left.re[K], CONJ ? -left.im[K] : left.im[K], b.re[j], -b.im[j]);
        } else {
            const T ar = left.re[K], ai = CONJ ? -left.im[K] : left.im[K];
            auto term = [&](auto col) {
                constexpr int j = decltype(col)::value;
                cmac(acc.re[j], acc.im[j], ar, ai, from<j>(m.re[K]), from<j>(m.im[K]));
            };
            term(std::integral_constant<int, 0>{});
            term(std::integral_constant<int, 1>{});
            if constexpr (N > 2) term(std::integral_constant<int, 2>{});
            if constexpr (N > 3) term(std::integral_constant<int, 3>{});
        }
        row_times<DAG, CONJ, N, T, K + 1>(acc, left, m);
    }
}
// out[k] = sum_m D_km col[m]: the lane's column of D E from its column of E, D
// held by columns.
template <int N, typename T, int M = 0>
__device__ __forceinline__ void times_col(Vec<N, T>& out, const Vec<N, T>& D, const Vec<N, T>& col) {
    if constexpr (M < N) {
        const Vec<N, T> d = from<M>(D);  // d[k] = D_kM
#pragma unroll
        for (int k = 0; k < N; ++k) cmac(out.re[k], out.im[k], d.re[k], d.im[k], col.re[M], col.im[M]);
        times_col<N, T, M + 1>(out, D, col);
    }
}
template <int N, typename T>
__device__ __forceinline__ Vec<N, T> zero_vec() {
    Vec<N, T> v;
#pragma unroll
    for (int k = 0; k < N; ++k) v.re[k] = v.im[k] = T(0);
    return v;
}

// The neighbours of one direction: rows or columns as the products take them.
template <int N, typename T>
struct Nbrs {
    Vec<N, T> a, b, c;  // upper: U_nu(x+mu) by rows, U_mu(x+nu), U_nu(x) by columns
    Vec<N, T> d, e, f;  // lower: U_mu(x-nu), U_nu(x+mu-nu), U_nu(x-nu) by columns
};
template <int N, typename T, int R, int MU, int NU>
__device__ __forceinline__ void load_dir(Nbrs<N, T>& n, const Field<N, T, R>& F, const Geom& g, const Site& x,
                                         const Site& xp, int par, int h, int r) {
    const int op = par ^ 1;
    const Site xpn = step_up(g, x, NU), xmn = step_down(g, x, NU), xpmn = step_down(g, xp, NU);
    n.a = F.row(NU, op, xp.s >> 1, r);
    n.b = F.col(MU, op, xpn.s >> 1, r);
    n.c = F.col(NU, par, h, r);
    n.d = F.col(MU, op, xmn.s >> 1, r);
    n.e = F.col(NU, par, xpmn.s >> 1, r);
    n.f = F.col(NU, op, xmn.s >> 1, r);
}
// Row r of the direction's two staples added to A.  SU(3) in FP64 forms rows 0
// and 1 of a staple and rebuilds row 2, as staple_dir does.
template <int N, typename T, int R>
__device__ __forceinline__ void add_dir(Vec<N, T>& A, Nbrs<N, T>& n, int r) {
    constexpr bool kRebuild = N == 3 && sizeof(T) == 8;
    complete_col<N, T, R>(n.b);
    complete_col<N, T, R>(n.c);
    complete_col<N, T, R>(n.d);
    complete_col<N, T, R>(n.e);
    complete_col<N, T, R>(n.f);
    if constexpr (R < N && !kRebuild) complete_row(n.a, r);
    Vec<N, T> m = zero_vec<N, T>(), l = zero_vec<N, T>();
    row_times<true, false>(m, n.a, n.b);
    if constexpr (kRebuild) {
        Vec<N, T> su = zero_vec<N, T>(), sd = zero_vec<N, T>();
        row_times<true, false>(su, m, n.c);
        complete_row(su, r);
        times_col(l, n.d, n.e);
        row_times<false, true>(sd, l, n.f);
        complete_row(sd, r);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            A.re[k] += su.re[k];
            A.im[k] += su.im[k];
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            A.re[k] += sd.re[k];
            A.im[k] += sd.im[k];
        }
    } else {
        row_times<true, false>(A, m, n.c);
        times_col(l, n.d, n.e);
        row_times<false, true>(A, l, n.f);
    }
}

// The heatbath draw of the quad's step (alpha the same on its lanes): 0 when
// every attempt was rejected, else its number, with the element in x.
template <typename T>
__device__ __forceinline__ int draw(T alpha, uint32_t k0, uint32_t k1, uint32_t site, uint32_t step, uint32_t mu_sg,
                                    Quat<T>& x) {
    const int q = threadIdx.x & 3;
    const bool creutz = alpha < Const<T>::switch_alpha;
    const T em = creutz ? d_expm1(T(-2) * alpha) : T(0);
    const T ia = fast_inverse(alpha);
    // attempts 0 .. 2 and the direction share the Philox call and a cosine
    const U4 w = philox(site, step, mu_sg, q == 3 ? RNG_DIRECTION << 24 : (RNG_ATTEMPT << 24) | (uint32_t)q, k0, k1);
    const T r0 = uniform<T>(w.w[0]), r1 = uniform<T>(w.w[1]);
    const T r2 = uniform<T>(w.w[2]), r3 = uniform<T>(w.w[3]);
    const T angle = Const<T>::two_pi * r1;
    const T c = draw_cos(angle);
    T x0 = T(1), rad = T(0);
    bool ok = false;
    if (creutz) {
        x0 = (alpha == T(0)) ? T(2) * r0 - T(1) : T(1) + d_log1p((T(1) - r0) * em) * ia;
        const T rhs = T(1) - x0 * x0;
        if (r1 * r1 <= rhs) {
            rad = fast_sqrt(rhs);
            ok = true;
        }
    } else {
        const T lam2 = -(draw_log(r0) + c * c * draw_log(r2)) * (T(0.5) * ia);
        const T rhs = T(1) - lam2;
        if (r3 * r3 <= rhs) {
            x0 = T(1) - T(2) * lam2;
            rad = T(2) * fast_sqrt(lam2) * fast_sqrt(rhs);
            ok = true;
        }
    }
    const T ct = T(1) - T(2) * r0;
    const T st = from<3>(fast_sqrt(T(1) - ct * ct));
    const T cp = from<3>(c), sp = from<3>(draw_sin(angle));
    const int sh = threadIdx.x & 60;
    uint32_t hits = (uint32_t)(__ballot(ok && q < 3) >> sh) & 7u;
    int first = hits ? __ffs((int)hits) - 1 : 0;
    int hit = hits ? first + 1 : 0;
    T ox0 = from_first(x0, first), orad = from_first(rad, first);
    for (int h0 = 3; h0 < kMaxAttempts && __any(hit == 0); h0 += 4) {
        const U4 v = philox(site, step, mu_sg, (RNG_ATTEMPT << 24) | (uint32_t)(h0 + q), k0, k1);
        T ax0 = T(1), arad = T(0);
        ok = h0 + q < kMaxAttempts && su2_attempt(alpha, ia, creutz, em, v, ax0, arad);
        hits = (uint32_t)(__ballot(ok) >> sh) & 15u;
        first = hits ? __ffs((int)hits) - 1 : 0;
        ax0 = from_first(ax0, first);
        arad = from_first(arad, first);
        if (hit == 0 && hits != 0) {
            hit = h0 + first + 1;
            ox0 = ax0;
            orad = arad;
        }
    }
    x.q[0] = ox0;
    x.q[1] = orad * st * cp;
    x.q[2] = orad * st * sp;
    x.q[3] = orad * from<3>(ct);
    return hit;
}

// Column c of the matrix whose rows the quad holds (lane k: row k).
template <int N, typename T>
__device__ __forceinline__ Vec<N, T> transposed(const Vec<N, T>& row, int c) {
    Vec<N, T> v;
    auto entry = [&](auto src) {
        constexpr int k = decltype(src)::value;
        const Vec<N, T> b = from<k>(row);
        v.re[k] = b.re[0];
        v.im[k] = b.im[0];
#pragma unroll
        for (int j = 1; j < N; ++j) {
            v.re[k] = c == j ? b.re[j] : v.re[k];
            v.im[k] = c == j ? b.im[j] : v.im[k];
        }
    };
    entry(std::integral_constant<int, 0>{});
    entry(std::integral_constant<int, 1>{});
    if constexpr (N > 2) entry(std::integral_constant<int, 2>{});
    if constexpr (N > 3) entry(std::integral_constant<int, 3>{});
    return v;
}

// Subgroup step (I, J), number SG, on the quad's columns of U and W; then the
// steps after it in the fixed order.
template <int N, typename T, bool HB, int MU, int I, int J, int SG>
__device__ __forceinline__ void steps(Vec<N, T>& U, Vec<N, T>& W, T cb, uint32_t k0, uint32_t k1, uint32_t site,
                                      uint32_t step) {
    Quat<T> p, v, a;
    p.q[0] = T(0.5) * (from<I>(W.re[I]) + from<J>(W.re[J]));
    p.q[3] = T(0.5) * (from<I>(W.im[I]) - from<J>(W.im[J]));
    p.q[2] = T(0.5) * (from<J>(W.re[I]) - from<I>(W.re[J]));
    p.q[1] = T(0.5) * (from<J>(W.im[I]) + from<I>(W.im[J]));
    const T k = unit_quat(p, norm2(p, first_alone<N, T, HB>(SG)), v);
    bool apply = true;
    if constexpr (HB) {
        Quat<T> xs;
        apply = draw<T>(cb * k, k0, k1, site, step, ((uint32_t)MU << 16) | (uint32_t)SG, xs) != 0;
        a = qmul(xs, qconj(v));
    } else {
        const Quat<T> vc = qconj(v);
        a = qmul(vc, vc);
    }
    auto rotate = [&](Vec<N, T>& M) {
        const T xr = M.re[I], xi = M.im[I], yr = M.re[J], yi = M.im[J];
        const T ir = fmadd(-a.q[1], yi, fmadd(a.q[2], yr, fmadd(-a.q[3], xi, a.q[0] * xr)));
        const T ii = fmadd(a.q[1], yr, fmadd(a.q[2], yi, fmadd(a.q[3], xr, a.q[0] * xi)));
        const T jr = fmadd(a.q[3], yi, fmadd(a.q[0], yr, fmadd(-a.q[1], xi, -a.q[2] * xr)));
        const T ji = fmadd(-a.q[3], yr, fmadd(a.q[0], yi, fmadd(a.q[1], xr, -a.q[2] * xi)));
        M.re[I] = apply ? ir : xr;
        M.im[I] = apply ? ii : xi;
        M.re[J] = apply ? jr : yr;
        M.im[J] = apply ? ji : yi;
    };
    rotate(U);
    rotate(W);
    if constexpr (J + 1 < N)
        steps<N, T, HB, MU, I, J + 1, SG + 1>(U, W, cb, k0, k1, site, step);
    else if constexpr (I + 2 < N)
        steps<N, T, HB, MU, I + 1, I + 2, SG + 1>(U, W, cb, k0, k1, site, step);
}

// U_mu(x), x = site h of parity par, Nc >= 3; live: the link is to be stored.
template <int N, typename T, int R, bool HB, int MU>
__device__ __forceinline__ void update_link(T2<T>* __restrict__ Up, const Geom& g, int par, int h, bool live, T beta,
                                            uint32_t k0, uint32_t k1, uint32_t step) {
    const Field<N, T, R> F{reinterpret_cast<const char*>(Up), (uint32_t)g.Vh};
    const int q = threadIdx.x & 3, r = q < N ? q : N - 1;
    const Site x = site_of(g, par, h);
    const Site xp = step_up(g, x, MU);
    constexpr int D0 = MU == 0 ? 1 : 0, D1 = MU <= 1 ? 2 : 1, D2 = MU == 3 ? 2 : 3;
    Vec<N, T> A = zero_vec<N, T>(), U;
    {
        // three directions' loads in flight before the first product where
        // the registers hold them, else one direction ahead
        constexpr bool kAll = N * sizeof(T) <= 16;
        Nbrs<N, T> n0, n1, n2;
        const bool p0 = (g.present >> D0) & 1, p1 = (g.present >> D1) & 1, p2 = (g.present >> D2) & 1;
        load_dir<N, T, R, MU, D0>(n0, F, g, x, xp, par, h, r);
        load_dir<N, T, R, MU, D1>(n1, F, g, x, xp, par, h, r);
        if constexpr (kAll) {
            load_dir<N, T, R, MU, D2>(n2, F, g, x, xp, par, h, r);
            U = F.col(MU, par, h, r);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (p0) add_dir<N, T, R>(A, n0, r);
        if constexpr (!kAll) {
            load_dir<N, T, R, MU, D2>(n2, F, g, x, xp, par, h, r);
            U = F.col(MU, par, h, r);
        }
        if (p1) add_dir<N, T, R>(A, n1, r);
        if (p2) add_dir<N, T, R>(A, n2, r);
    }
    complete_col<N, T, R>(U);
    // column r of W = U A
    const Vec<N, T> At = transposed(A, r);
    Vec<N, T> W = zero_vec<N, T>();
    times_col(W, U, At);
    const T cb = T(2) * beta / T(N);  // alpha = 2 beta k / N
    steps<N, T, HB, MU, 0, 1, 0>(U, W, cb, k0, k1, (uint32_t)x.s, step);
    if (live && q < N) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            T2<T> v;
            v.x = U.re[k];
            v.y = U.im[k];
            *reinterpret_cast<T2<T>*>(reinterpret_cast<char*>(Up) + (F.plane(MU, par, k * N + q) * F.Vh + (uint32_t)h) *
                                                                        Field<N, T, R>::kEntry) = v;
        }
    }
}

// The same for SU(2): lane l forms the staples of the l-th direction other
// than MU.
template <typename T, bool HB, int MU>
__device__ __forceinline__ void update_link_su2(T2<T>* __restrict__ Up, const Geom& g, int par, int h, bool live,
                                                T beta, uint32_t k0, uint32_t k1, uint32_t step) {
    const Field<2, T, 2> F{reinterpret_cast<const char*>(Up), (uint32_t)g.Vh};
    const int q = threadIdx.x & 3;
    const Site x = site_of(g, par, h);
    const Site xp = step_up(g, x, MU);
    constexpr int D0 = MU == 0 ? 1 : 0, D1 = MU <= 1 ? 2 : 1, D2 = MU == 3 ? 2 : 3;
    auto pick = [&](int a, int b, int c) { return q == 0 ? a : q == 1 ? b : c; };
    const int nu = pick(D0, D1, D2);
    const int up = pick(step_up(g, x, D0).s, step_up(g, x, D1).s, step_up(g, x, D2).s);
    const int dn = pick(step_down(g, x, D0).s, step_down(g, x, D1).s, step_down(g, x, D2).s);
    const int pdn = pick(step_down(g, xp, D0).s, step_down(g, xp, D1).s, step_down(g, xp, D2).s);
    const int op = par ^ 1;
    auto load = [&](int mu, int parity, int hh) {
        const T2<T> a = F.entry(F.plane(mu, parity, 0), hh), b = F.entry(F.plane(mu, parity, 1), hh);
        return Quat<T>{{a.x, a.y, b.x, b.y}};
    };
    const Quat<T> a = load(nu, op, xp.s >> 1), b = load(MU, op, up >> 1), c = load(nu, par, h);
    const Quat<T> d = load(MU, op, dn >> 1), e = load(nu, par, pdn >> 1), f = load(nu, op, dn >> 1);
    const Quat<T> u = load(MU, par, h);
    const Quat<T> su = qmul(qmul(a, qconj(b)), qconj(c));
    const Quat<T> sd = qmul(qconj(qmul(d, e)), f);
    Quat<T> A{{T(0), T(0), T(0), T(0)}};
    auto add = [&](auto lane, int dir) {
        constexpr int l = decltype(lane)::value;
        const bool p = (g.present >> dir) & 1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const T s = from<l>(su.q[k]);
            A.q[k] = p ? A.q[k] + s : A.q[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const T s = from<l>(sd.q[k]);
            A.q[k] = p ? A.q[k] + s : A.q[k];
        }
    };
    add(std::integral_constant<int, 0>{}, D0);
    add(std::integral_constant<int, 1>{}, D1);
    add(std::integral_constant<int, 2>{}, D2);
    Quat<T> v, el;
    const Quat<T> p = qmul(u, A);
    const T k = unit_quat(p, norm2(p, first_alone<2, T, HB>(0)), v);
    bool apply = true;
    if constexpr (HB) {
        Quat<T> xs;
        apply = draw<T>(beta * k, k0, k1, (uint32_t)x.s, step, (uint32_t)MU << 16, xs) != 0;
        el = qmul(xs, qconj(v));
    } else {
        const Quat<T> vc = qconj(v);
        el = qmul(vc, vc);
    }
    const Quat<T> n = qmul(el, u);
    if (live && apply && q < 2) {  // a pair each
        T2<T> o;
        o.x = q == 0 ? n.q[0] : n.q[2];
        o.y = q == 0 ? n.q[1] : n.q[3];
        *reinterpret_cast<T2<T>*>(reinterpret_cast<char*>(Up) +
                                  (F.plane(MU, par, q) * F.Vh + (uint32_t)h) * Field<2, T, 2>::kEntry) = o;
    }
}

// One phase of one lattice: workgroup b takes links 16 w .. 16 w + 15 of walk
// position w.
template <int N, typename T, int R, bool HB, int MU>
__global__ __launch_bounds__(kBlockItems) void k_update_quad(T2<T>* __restrict__ U, Geom g, int par, T beta,
                                                             uint32_t k0, uint32_t k1, uint32_t step, Walk walk) {
    const int h = walk_tile((int)blockIdx.x, (int)gridDim.x, walk) * kLinks + (int)(threadIdx.x >> 2);
    const bool live = h < g.Vh;
    const int hc = live ? h : g.Vh - 1;  // lanes past the end repeat the last link
    if constexpr (N == 2)
        update_link_su2<T, HB, MU>(U, g, par, hc, live, beta, k0, k1, step);
    else
        update_link<N, T, R, HB, MU>(U, g, par, hc, live, beta, k0, k1, step);
}

template <int N, typename T, int R>
void launch(const Ctx& c, int kind, int mu, int par, double beta, uint32_t k0, uint32_t k1, uint32_t step) {
    const int grid = (c.g.Vh + kLinks - 1) / kLinks;
    Walk w{1, 0, 1, 1, 0};
    if (c.order) random_tile_order(c.order, grid, w);
    auto run = [&](auto hb, auto dir) {
        k_update_quad<N, T, R, decltype(hb)::value, decltype(dir)::value>
            <<<grid, kBlockItems, 0, c.stream>>>((T2<T>*)c.links, c.g, par, (T)beta, k0, k1, step, w);
    };
    auto with_dir = [&](auto hb) {
        switch (mu) {
            case 0: run(hb, std::integral_constant<int, 0>{}); break;
            case 1: run(hb, std::integral_constant<int, 1>{}); break;
            case 2: run(hb, std::integral_constant<int, 2>{}); break;
            default: run(hb, std::integral_constant<int, 3>{}); break;
        }
    };
    if (kind == 0)
        with_dir(std::true_type{});
    else
        with_dir(std::false_type{});
}

}  // namespace quad
}  // namespace sun
