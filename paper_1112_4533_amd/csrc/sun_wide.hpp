// sun_wide.hpp -- SU(Nc) for large Nc (4 <= Nc <= 32; paper Sec. 3, generic
// SU(Nc) code; Sec. 4, the large-Nc runs at 8^4): the SU(2) draw of the
// subgroup steps, start configuration, Polyakov loop and field transfer.  The
// phase update is in sun_wide_small.hpp (Nc <= 8, four links to a wavefront)
// and sun_wide_large.hpp (two wavefronts to a link), the plaquette in
// sun_wide_plaq.hpp, the re-unitarization in sun_wide_reunit.hpp.
//
// At large Nc a link no longer fits in one work-item's registers (Nc = 32 is
// 2048 reals): its matrices live in LDS, spread over the lanes.  Links are
// stored link-major (the Nc^2 complex entries of one link are contiguous), so
// a workgroup reads a link with unit stride.
//
// The arithmetic is that of the register kernels: the same closing staple,
// W = U A, the lexicographic subgroup order (run several steps at a time
// where they share no index, which gives the same bits: sun_pairs.hpp), the
// quaternion projection, the same Philox counters, and an SU(2) draw that
// takes the lowest accepting attempt, the sequential draw's result.
// Reductions and re-unitarization are FP64.
#pragma once

#include <cfloat>

#include "sun_kernels.hpp"
#include "sun_pairs.hpp"

namespace sun {
namespace wide {

constexpr int kLanes = 64;
static_assert(kMaxAttempts == kLanes, "one SU(2) attempt per lane");
constexpr int kNcMin = 4, kNcMax = 32;

__host__ __device__ inline size_t fp64_lds(int n, int buffers) { return (size_t)buffers * n * n * sizeof(double2); }

template <typename T>
__device__ __forceinline__ T2<T> cpx(T re, T im) {
    T2<T> v;
    v.x = re;
    v.y = im;
    return v;
}

// Link-major storage: link (mu, parity, h) is n^2 consecutive entries.
template <typename T>
__device__ __forceinline__ const T2<T>* link_at(const T2<T>* U, int n2, int mu, int par, int h, int Vh) {
    return U + ((size_t)(mu * 2 + par) * Vh + h) * n2;
}

// dst (LDS, type D) = src (global, type S), converted.  Each
// lane issues the global loads of kLoadBatch entries before it stores any,
// so a link costs a few load latencies instead of one per entry.
constexpr int kLoadBatch = 8;

template <typename D, typename S>
__device__ __forceinline__ void lds_load(T2<D>* dst, const T2<S>* src, int n) {
    const int n2 = n * n;
    if (n2 <= kLanes) {  // one entry per lane
        const int e = threadIdx.x;
        if (e < n2) {
            const T2<S> v = src[e];
            dst[e] = cpx<D>((D)v.x, (D)v.y);
        }
        return;
    }
    for (int e0 = threadIdx.x; e0 < n2; e0 += kLoadBatch * kLanes) {
        T2<S> v[kLoadBatch];
#pragma unroll
        for (int c = 0; c < kLoadBatch; ++c) {
            const int e = e0 + c * kLanes;
            if (e < n2) v[c] = src[e];
        }
#pragma unroll
        for (int c = 0; c < kLoadBatch; ++c) {
            const int e = e0 + c * kLanes;
            if (e >= n2) break;
            dst[e] = cpx<D>((D)v[c].x, (D)v[c].y);
        }
    }
}

// C = A B (n <= 32; C distinct from B; it may be A itself, because a lane reads
// its block of rows completely in the k loop before it stores any of it, the
// lanes of a row group run that loop together in the one wavefront of the
// workgroup, and no other lane touches those rows).  With g = 64 / n
// row groups, lane l < g n owns column j = l mod n and rows i0, i0 + g, ...
// (i0 = l / n), which it takes R at a time: each B_kj it reads serves R rows,
// and the n lanes of a row group read the same A_ik (an LDS broadcast).  A
// block that runs past the lane's last row repeats that row and does not
// store it, so the k loop has no lane-dependent branch.  Every entry is the
// sum over k = 0 .. n-1 in increasing k, with the same complex multiply-add
// as the plain triple loop.
template <typename T, int R>
__device__ __forceinline__ void lds_mm_rows(T2<T>* C, const T2<T>* A, const T2<T>* B, int n, int g, int j, int i0,
                                            int cnt) {
    for (int t0 = 0; t0 < cnt; t0 += R) {
        int row[R];
        T r[R], m[R];
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int tt = t0 + t < cnt ? t0 + t : cnt - 1;
            row[t] = (i0 + g * tt) * n;
            r[t] = T(0);
            m[t] = T(0);
        }
        // four k per pass, their LDS reads issued together
        int k = 0;
        for (; k + 4 <= n; k += 4) {
            T2<T> y[4], x[4][R];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                y[q] = B[(k + q) * n + j];
#pragma unroll
                for (int t = 0; t < R; ++t) x[q][t] = A[row[t] + k + q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int t = 0; t < R; ++t) cmac(r[t], m[t], x[q][t].x, x[q][t].y, y[q].x, y[q].y);
        }
        for (; k < n; ++k) {
            const T2<T> y = B[k * n + j];
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const T2<T> x = A[row[t] + k];
                cmac(r[t], m[t], x.x, x.y, y.x, y.y);
            }
        }
#pragma unroll
        for (int t = 0; t < R; ++t)
            if (t0 + t < cnt) C[row[t] + j] = cpx<T>(r[t], m[t]);
    }
}

// The product by one wavefront: 64 / n groups of n lanes, group i0 = lane / n
// taking column j = lane mod n and rows i0, i0 + g, ... (g groups in all).
template <typename T>
__device__ __forceinline__ void lds_mm(T2<T>* C, const T2<T>* A, const T2<T>* B, int n) {
    const int g = kLanes / n, l = (int)threadIdx.x;
    if (l >= g * n) return;
    const int j = l % n, i0 = l / n;
    const int cnt = (n - i0 + g - 1) / g;  // rows i0 + g t < n of this lane
    const int most = (n + g - 1) / g;      // rows of group 0, the most of any group
    if (most >= 4)
        lds_mm_rows<T, 4>(C, A, B, n, g, j, i0, cnt);
    else if (most >= 2)
        lds_mm_rows<T, 2>(C, A, B, n, g, j, i0, cnt);
    else
        lds_mm_rows<T, 1>(C, A, B, n, g, j, i0, cnt);
}

// Change of the site index by one step along direction m (periodic), and the
// value of a run-time direction picked with selects (an array indexed by it
// would live in memory).
__device__ __forceinline__ int step_shift(const Geom& g, const Site& x, bool up, int m) {
    const int wrap = (g.L[m] - 1) * g.stride[m];
    return up ? (x.x[m] == g.L[m] - 1 ? -wrap : g.stride[m]) : (x.x[m] == 0 ? wrap : -g.stride[m]);
}
__device__ __forceinline__ int pick_dir(int a, int b, int c, int d, int m) {
    int v = m == 1 ? b : a;
    v = m == 2 ? c : v;
    return m == 3 ? d : v;
}

// Cross-lane moves of a wavefront without the LDS: lane l receives the
// value of its partner lane, for five pairings that together join all 64
// lanes -- l xor 1 and l xor 2 (quad permutes), 7 - l and 15 - l within
// groups of 8 and 16 (row mirrors), l xor 16 (swizzle) -- and l xor 32
// (the swap of the two halves).
template <int STEP>
__device__ __forceinline__ int partner(int v) {
    if constexpr (STEP == 0) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);   // quad [1,0,3,2]
    if constexpr (STEP == 1) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);   // quad [2,3,0,1]
    if constexpr (STEP == 2) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);  // row half mirror
    if constexpr (STEP == 3) return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row mirror
    if constexpr (STEP == 4) return __builtin_amdgcn_ds_swizzle(v, 0x401F);                     // xor 16
    if constexpr (STEP == 5) {                                                                   // xor 32
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (threadIdx.x & (kLanes - 1)) < 32 ? (int)r[1] : (int)r[0];
    }
    return v;
}
template <int STEP>
__device__ __forceinline__ double partner(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)partner<STEP>((int)(u & 0xffffffffu));
    const unsigned hi = (unsigned)partner<STEP>((int)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Wave reductions over the six pairings above in a fixed order: every lane
// combines the same two partial results at each step (in one order or the
// other, which for + and max gives the same bits), so all lanes end with
// the same deterministic value.
template <typename F>
__device__ __forceinline__ double wave_reduce(double v, F op) {
    v = op(v, partner<0>(v));
    v = op(v, partner<1>(v));
    v = op(v, partner<2>(v));
    v = op(v, partner<3>(v));
    v = op(v, partner<4>(v));
    v = op(v, partner<5>(v));
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
    return wave_reduce(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double v) {
    return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}

// Orders LDS hand-offs between the lanes of one wavefront: its LDS operations
// complete in the order it issues them -- a read issued after a write sees it,
// whichever lane wrote, and a write issued after a read leaves that read's
// value alone -- so they need only compiler ordering (a wavefront-scope fence),
// not a wait for the LDS round trip that a workgroup barrier implies.
// Hand-offs between wavefronts need the barrier.
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// The scalar steps of the subgroup chain -- the block's norm and its
// inverse, 1 / alpha, the draw's square roots -- are computed by the lanes
// of a step for the whole link, one slot after another, so their latency is
// the chain's; the correctly rounded sequences take a dozen dependent
// instructions each.  FP32 takes the hardware forms shared with the
// register path (fast_sqrt, fast_inverse, unit_quat: about 1 ulp each); FP64
// here takes the hardware reciprocal and reciprocal square root refined by
// two Newton steps each (about 1 ulp) and the correctly rounded square root.
// The extra half ulp is far inside the tolerance of a link update.  Zero and
// subnormal arguments keep the correctly rounded forms.
__device__ __forceinline__ double newton_rsqrt(double x) {  // normal x > 0
    double r = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) {  // r <- r + r (1 - x r^2) / 2
        const double e = fma(-x * r, r, 1.0);
        r = fma(0.5 * r, e, r);
    }
    return r;
}
__device__ __forceinline__ double newton_rcp(double x) {  // normal x > 0
    double r = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) {  // r <- r + r (1 - x r)
        const double e = fma(-x, r, 1.0);
        r = fma(r, e, r);
    }
    return r;
}

template <typename T>
__device__ __forceinline__ T chain_inverse(T alpha) {
    if constexpr (sizeof(T) == 8) {
        if (alpha >= DBL_MIN) return newton_rcp(alpha);
    }
    return fast_inverse(alpha);
}

// k = |p| and v = p / k (v = 1 for p = 0), as unit_quat.
template <typename T>
__device__ __forceinline__ T chain_unit_quat(const Quat<T>& p, Quat<T>& v) {
    if constexpr (sizeof(T) == 8) {
        const double k2 = p.q[0] * p.q[0] + p.q[1] * p.q[1] + p.q[2] * p.q[2] + p.q[3] * p.q[3];
        if (k2 >= DBL_MIN) {
            const double r = newton_rsqrt(k2);
#pragma unroll
            for (int c = 0; c < 4; ++c) v.q[c] = p.q[c] * r;
            return k2 * r;
        }
    }
    return unit_quat(p, p.q[0] * p.q[0] + p.q[1] * p.q[1] + p.q[2] * p.q[2] + p.q[3] * p.q[3], v);
}

// ---------------------------------------------------------------------------
// Draws by place: sixteen lanes run one subgroup step, and the terms of its
// draw that do not depend on alpha wait in LDS -- the Kennedy-Pendleton log
// term and r3^2 of its first three attempts, and its direction -- so that
// every lane of the place tries all three with two multiplications and a
// comparison each and none of them has to be moved between lanes.  A step
// whose alpha is in the Creutz range tries the first of them in as many lanes,
// from the words kept beside them (with a Philox call in the chain the
// heatbath at beta 6.2 on 8^4 took 73 instead of 62 us for SU(8) FP64, 83
// instead of 77 for SU(16) FP32).  A step whose attempts on record all reject
// (at most 0.29^3 of the draws, far fewer at the couplings of a run) goes on
// sixteen attempts at a time.  Either way the
// lowest accepting attempt of the counter stream wins, as in the sequential
// sampler, and the accepted attempt's arithmetic is its own.
// ---------------------------------------------------------------------------
constexpr int kPlaceLanes = 16;
constexpr int kQuickHits = 3;              // attempts a record holds
constexpr int kRecLanes = kQuickHits + 1;  // lanes that fill one: its attempts and its direction
// C of the attempts can be taken in the Creutz range too: three up to Nc = 8
// and in the largest form, two between (with three, FP64 records at Nc = 21
// would leave 7 links to a CU).
template <typename T, int C = 2, int ALIGN = 16>
struct alignas(ALIGN) DrawRec {
    T kp[kQuickHits], r3sq[kQuickHits];
    T cos_t, sin_t, cos_p, sin_p;
    uint32_t w0[C], w1[C];  // the words a Creutz attempt takes
};

// Share q of a record: attempt q, or the direction (q = kQuickHits).  One
// Philox call and one cosine serve both kinds.
template <typename T, int C, int A>
__device__ __forceinline__ void fill_draw(DrawRec<T, C, A>& rec, int q, uint32_t k0, uint32_t k1, uint32_t site,
                                          uint32_t step, uint32_t mu_sg) {
    const bool dir = q == kQuickHits;
    const U4 w = philox(site, step, mu_sg, dir ? RNG_DIRECTION << 24 : (RNG_ATTEMPT << 24) | (uint32_t)q, k0, k1);
    const T u0 = uniform<T>(w.w[0]);
    const T angle = Const<T>::two_pi * uniform<T>(w.w[1]);
    const T c = draw_cos(angle);
    if (dir) {
        const T ct = T(1) - T(2) * u0;
        rec.cos_t = ct;
        rec.sin_t = d_sqrt(T(1) - ct * ct);
        rec.cos_p = c;
        rec.sin_p = draw_sin(angle);
    } else {
        const T r2 = uniform<T>(w.w[2]), r3 = uniform<T>(w.w[3]);
        rec.kp[q] = -(draw_log(u0) + c * c * draw_log(r2));
        rec.r3sq[q] = r3 * r3;
        if (q < C) {
            rec.w0[q] = w.w[0];
            rec.w1[q] = w.w[1];
        }
    }
}

// The records of subgroups sg0 .. sg0 + nsteps - 1, by the sixteen lanes of
// a place, four at a time.
template <typename T, int C, int A>
__device__ __forceinline__ void fill_draws(DrawRec<T, C, A>* rec, int nsteps, uint32_t sg0, uint32_t k0, uint32_t k1,
                                           uint32_t site, uint32_t step, uint32_t mu_hi) {
    const int q = (int)threadIdx.x % kPlaceLanes;
    for (int t0 = 0; t0 < nsteps; t0 += kPlaceLanes / kRecLanes) {
        const int t = t0 + q / kRecLanes;
        if (t < nsteps) fill_draw<T>(rec[t], q % kRecLanes, k0, k1, site, step, mu_hi | (sg0 + (uint32_t)t));
    }
}

// The draw of the lane's place: alpha and live (a step is there) are the
// same on its sixteen lanes.  Returns the number of the accepted attempt
// (1-based), or 0 (skip the step) when all kMaxAttempts were rejected.
template <typename T, int C, int A>
__device__ __forceinline__ int place_draw(T alpha, bool live, const DrawRec<T, C, A>& rec, uint32_t k0, uint32_t k1,
                                          uint32_t site, uint32_t step, uint32_t mu_sg, Quat<T>& x) {
    const bool creutz = alpha < Const<T>::switch_alpha;
    const T ia = chain_inverse(alpha);
    T x0 = T(1), rad = T(0);
    int hit = 0;
    {
        const T half = T(0.5) * ia;
        T l2 = T(0), rh = T(1);
#pragma unroll
        for (int a = kQuickHits - 1; a >= 0; --a) {
            const T lam2 = rec.kp[a] * half;
            const T rhs = T(1) - lam2;
            if (rec.r3sq[a] <= rhs) {
                l2 = lam2;
                rh = rhs;
                hit = a + 1;
            }
        }
        x0 = T(1) - T(2) * l2;
        rad = T(2) * fast_sqrt(l2) * fast_sqrt(rh);
    }
    if (__any(live && (creutz || hit == 0))) {
        if (creutz) hit = 0;
        const T em = creutz ? d_expm1(T(-2) * alpha) : T(0);
        const int first_lane = (int)threadIdx.x & (kLanes - kPlaceLanes), lane = (int)threadIdx.x % kPlaceLanes;
        // attempts h0 .. of the place's lanes; the lowest accepting one counts
        auto accept = [&](bool ok, T ax0, T arad, int h0) {
            const uint32_t m = (uint32_t)(__ballot(ok) >> first_lane) & 0xFFFFu;
            const int a = m ? __ffs(m) - 1 : 0;
            ax0 = __shfl(ax0, first_lane + a, kLanes);
            arad = __shfl(arad, first_lane + a, kLanes);
            if (hit == 0 && m != 0) {
                x0 = ax0;
                rad = arad;
                hit = h0 + a + 1;
            }
        };
        if (__any(live && creutz)) {
            T ax0 = T(1), arad = T(0);
            bool ok = false;
            if (creutz && lane < C) {
                const U4 r{{rec.w0[lane], rec.w1[lane], 0u, 0u}};
                ok = su2_attempt(alpha, ia, true, em, r, ax0, arad);
            }
            accept(ok, ax0, arad, 0);
        }
        for (int h0 = C; h0 < kMaxAttempts && __any(live && hit == 0); h0 += kPlaceLanes) {
            const int mine = h0 + lane;
            const U4 r = philox(site, step, mu_sg, (RNG_ATTEMPT << 24) | (uint32_t)mine, k0, k1);
            T ax0 = T(1), arad = T(0);
            const bool ok = mine < kMaxAttempts && su2_attempt(alpha, ia, creutz, em, r, ax0, arad);
            accept(ok, ax0, arad, h0);
        }
    }
    x.q[0] = x0;
    x.q[1] = rad * rec.sin_t * rec.cos_p;
    x.q[2] = rad * rec.sin_t * rec.sin_p;
    x.q[3] = rad * rec.cos_t;
    return hit;
}

// One column of two rows left-multiplied by the 2x2 form of a: entries x, y
// before, *pi, *pj after.
template <typename T>
__device__ __forceinline__ void rows_left_mul_at(T2<T>* pi, T2<T>* pj, const Quat<T>& a, const T2<T>& x,
                                                 const T2<T>& y) {
    *pi = cpx<T>(fmadd(-a.q[1], y.y, fmadd(a.q[2], y.x, fmadd(-a.q[3], x.y, a.q[0] * x.x))),
                 fmadd(a.q[1], y.x, fmadd(a.q[2], y.y, fmadd(a.q[3], x.x, a.q[0] * x.y))));
    *pj = cpx<T>(fmadd(a.q[3], y.y, fmadd(a.q[0], y.x, fmadd(-a.q[1], x.y, -a.q[2] * x.x))),
                 fmadd(-a.q[3], y.x, fmadd(a.q[0], y.y, fmadd(a.q[1], x.x, -a.q[2] * x.y))));
}

// ---------------------------------------------------------------------------
// FP64 helpers on an LDS matrix whose column c belongs to lane c (n <= 32).
// ---------------------------------------------------------------------------

// det by LU with partial pivoting (the first largest pivot), destroying D.
__device__ __forceinline__ void lds_det(double2* D, int n, double& dr, double& di) {
    const int c = threadIdx.x;
    dr = 1.0;
    di = 0.0;
    for (int col = 0; col < n; ++col) {
        wave_lds_order();
        // pivot: the largest |D[r][col]|^2 over r >= col, the lowest r among
        // equals -- a scan by lane 0 for small n, a wave argmax otherwise
        // (the same choice: the scan keeps the first strict maximum)
        int piv = col;
        double best = -1.0;
        if (n <= 8) {
            if (c == 0)
                for (int r = col; r < n; ++r) {
                    const double a = D[r * n + col].x * D[r * n + col].x + D[r * n + col].y * D[r * n + col].y;
                    if (a > best) {
                        best = a;
                        piv = r;
                    }
                }
            piv = __shfl(piv, 0, kLanes);
            best = __shfl(best, 0, kLanes);
        } else {
            piv = c;
            if (c >= col && c < n) best = D[c * n + col].x * D[c * n + col].x + D[c * n + col].y * D[c * n + col].y;
            // the largest, the lowest row among equals: an order-free choice,
            // so every lane ends with the same pair
            auto take = [&](double ob, int op) {
                if (ob > best || (ob == best && op < piv)) {
                    best = ob;
                    piv = op;
                }
            };
            take(partner<0>(best), partner<0>(piv));
            take(partner<1>(best), partner<1>(piv));
            take(partner<2>(best), partner<2>(piv));
            take(partner<3>(best), partner<3>(piv));
            take(partner<4>(best), partner<4>(piv));
            take(partner<5>(best), partner<5>(piv));
        }
        if (best == 0.0) {
            dr = di = 0.0;
            return;
        }
        if (piv != col) {
            if (c < n) {
                const double2 t = D[col * n + c];
                D[col * n + c] = D[piv * n + c];
                D[piv * n + c] = t;
            }
            dr = -dr;
            di = -di;
        }
        wave_lds_order();
        const double pr = D[col * n + col].x, pi = D[col * n + col].y;
        const double nr = dr * pr - di * pi, ni = dr * pi + di * pr;
        dr = nr;
        di = ni;
        const double pm = pr * pr + pi * pi;
        const double inv = pm >= DBL_MIN ? newton_rcp(pm) : 1.0 / pm;
        // rows below the pivot are independent: above n = 8 the lower half
        // of the wavefront eliminates rows col + 1, col + 3, ... and the upper
        // half rows col + 2, col + 4, ..., lane q taking column q (n <= 32);
        // every entry sees the same operations in the same order either way
        const bool split = n > 8;
        const int q = c & 31, half = c >> 5;
        const bool works = (split || half == 0) && q >= col && q < n;
        // the pivot row's entry of column q, read once: only rows below it
        // change in this column's elimination
        const double2 u = works ? D[col * n + q] : make_double2(0.0, 0.0);
        for (int r = col + 1 + (split ? half : 0); r < n; r += split ? 2 : 1) {
            const double2 m = D[r * n + col];
            const double fr = (m.x * pr + m.y * pi) * inv;
            const double fi = (m.y * pr - m.x * pi) * inv;
            if (works) {
                double2 w = D[r * n + q];
                w.x -= fr * u.x - fi * u.y;
                w.y -= fr * u.y + fi * u.x;
                D[r * n + q] = w;
            }
        }
    }
}

// Gram-Schmidt on all rows, then the last row times conj(det)/|det| (paper
// Sec. 2, re-unitarization; Nc > 3).  Each row is orthogonalized against the
// earlier ones by classical Gram-Schmidt, with a second pass where the
// first removed more than half the row's squared norm (Daniel, Gragg,
// Kaufman and Stewart, Math. Comp. 30 (1976): twice is enough, as stable as
// the modified form): lane k forms <r_k, r_i> from LDS, then lane c
// subtracts every projection from column c of r_i, so a row costs two LDS
// hand-offs per pass instead of a chain of wave reductions per projection.  P (n entries)
// holds the projections.  (dr, di) is det M of the matrix before the
// projection: row Gram-Schmidt writes M = L Q with L lower triangular and
// real positive on its diagonal, so det Q = det M / prod L_ii has the phase
// of det M, and the fix needs no determinant of Q.
__device__ __forceinline__ void lds_reunit(double2* M, double2* P, int n, double dr, double di) {
    const int lane = threadIdx.x;
    const bool own = lane < n;
    // n <= 32.  Above n = 8 the two halves of the wavefront share each sum,
    // lane q and lane q + 32 taking half of its terms each (below, the
    // exchange costs more than it saves and the lower half does it all).
    const bool split = n > 8;
    const int q = lane & 31, half = lane >> 5;
    const int m0 = split ? n / 2 : n;                    // columns of the lower half
    const int cbeg = half ? m0 : 0, clen = half ? n - m0 : m0;
    // |r_i|^2, the same value on every lane
    auto row_norm2 = [&](int i) {
        double s = 0.0;
        if (own) s = fmadd(M[i * n + lane].y, M[i * n + lane].y, M[i * n + lane].x * M[i * n + lane].x);
        return wave_sum(s);
    };
    // one classical pass: r_i -= sum_{k < i} <r_k, r_i> r_k
    auto project = [&](int i) {
        // p_q = <r_q, r_i> for q < i; columns taken from a lane-dependent
        // start within the half's range, so lanes hit different banks
        double pr = 0.0, pi = 0.0;
        if (q < i && clen > 0) {
            int t = q % clen;
#pragma unroll 4
            for (int u = 0; u < clen; ++u) {
                const int c = cbeg + t;
                const double2 a = M[q * n + c], b = M[i * n + c];
                cmac(pr, pi, a.x, -a.y, b.x, b.y);
                t = (t + 1 == clen) ? 0 : t + 1;
            }
        }
        if (split) {
            pr += partner<5>(pr);
            pi += partner<5>(pi);
        }
        if (q < i && half == 0) P[q] = make_double2(pr, pi);
        wave_lds_order();
        // r_i -= sum_{k < i} p_k r_k, the k range split between the halves
        double sr = 0.0, si = 0.0;
        if (q < n) {
            const int kmid = split ? i / 2 : i;
            const int kb = half ? kmid : 0, ke = half ? i : kmid;
#pragma unroll 4
            for (int k = kb; k < ke; ++k) {
                const double2 p = P[k], a = M[k * n + q];
                cmac(sr, si, p.x, p.y, a.x, a.y);
            }
        }
        if (split) {
            sr += partner<5>(sr);
            si += partner<5>(si);
        }
        if (own) {
            const double2 b = M[i * n + lane];
            M[i * n + lane] = make_double2(b.x - sr, b.y - si);
        }
        wave_lds_order();
    };
    for (int i = 0; i < n; ++i) {
        double s2;
        if (i > 0) {
            // a second pass only where the first removed more than half of
            // the row's squared norm (the DGKS criterion, "twice is
            // enough"): a row of a nearly unitary link keeps almost all of
            // it, and its one pass is orthogonal to rounding already
            const double s0 = row_norm2(i);
            project(i);
            s2 = row_norm2(i);
            if (s2 < 0.5 * s0) {
                project(i);
                s2 = row_norm2(i);
            }
        } else {
            s2 = row_norm2(i);
        }
        const double inv = s2 >= DBL_MIN ? newton_rsqrt(s2) : rsqrt(s2);
        if (own) {
            M[i * n + lane].x *= inv;
            M[i * n + lane].y *= inv;
        }
        wave_lds_order();
    }
    const double mod = sqrt(dr * dr + di * di);
    const double cr = dr / mod, ci = -di / mod;
    if (own) {
        const double2 r = M[(n - 1) * n + lane];
        M[(n - 1) * n + lane] = make_double2(r.x * cr - r.y * ci, r.x * ci + r.y * cr);
    }
    __syncthreads();
}

// Link id in [0, 4V) -> (mu, parity, h), as the register kernels number them.
__device__ __forceinline__ void link_id(const Geom& g, int id, int& mu, int& par, int& h) {
    mu = id / g.V;
    const int rem = id - mu * g.V;
    par = rem >= g.Vh ? 1 : 0;
    h = rem - par * g.Vh;
}

// Start configuration of link blockIdx.x: identity, or a Haar draw (Gaussian
// entries from Box-Muller on the same Philox counters as the register
// kernels, then re-unitarization).  LDS: M, D (a copy for the determinant,
// then the projections).
template <typename T>
__global__ __launch_bounds__(kLanes) void k_init(T2<T>* __restrict__ U, Geom g, int n, int hot, uint32_t k0,
                                                 uint32_t k1) {
    extern __shared__ double4 smem_init[];
    const int n2 = n * n;
    double2* M = reinterpret_cast<double2*>(smem_init);
    double2* D = M + n2;
    const int id = blockIdx.x;
    int mu, par, h;
    link_id(g, id, mu, par, h);
    if (hot && ((g.present >> mu) & 1)) {
        const uint32_t s = (uint32_t)site_of(g, par, h).s;
        // call q gives the Gaussians of entries 2q and 2q + 1
        for (int q = threadIdx.x; 2 * q < n2; q += kLanes) {
            const U4 r = philox(s, 0xFFFFFFFFu, (uint32_t)mu << 16, (RNG_HOTSTART << 24) | (uint32_t)q, k0, k1);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const double rad = sqrt(-2.0 * log(uniform<double>(r.w[2 * p])));
                const double ang = Const<double>::two_pi * uniform<double>(r.w[2 * p + 1]);
                if (2 * q + p < n2) M[2 * q + p] = make_double2(rad * cos(ang), rad * sin(ang));
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < n2; e += kLanes) D[e] = M[e];
        __syncthreads();
        double dr, di;
        lds_det(D, n, dr, di);
        __syncthreads();
        lds_reunit(M, D, n, dr, di);
    } else {
        for (int e = threadIdx.x; e < n2; e += kLanes) {
            const int i = e / n;
            M[e] = make_double2(i * n + i == e ? 1.0 : 0.0, 0.0);
        }
        __syncthreads();
    }
    T2<T>* dst = const_cast<T2<T>*>(link_at<T>(U, n2, mu, par, h, g.Vh));
    for (int e = threadIdx.x; e < n2; e += kLanes) dst[e] = cpx<T>((T)M[e].x, (T)M[e].y);
}

// One block per chain: out[3 c .. 3 c + 2] from its V site partials.
template <int Dummy = 0>
__global__ __launch_bounds__(kBlock) void k_plaquette_final_batch_wide(const ChainDesc* __restrict__ d, int nchains,
                                                                       int n, double* __restrict__ out) {
    const int c = blockIdx.x;
    if (c >= nchains) return;
    int n_sp = 0, n_tm = 0;
    for (int m = 0; m < 4; ++m)
        for (int k = m + 1; k < 4; ++k)
            if (((d[c].g.present >> m) & 1) && ((d[c].g.present >> k) & 1)) (k == 3 ? n_tm : n_sp)++;
    const double norm = (double)n * (double)d[c].g.V;
    plaquette_final<2>(d[c].scratch, d[c].g.V, out + 3 * (size_t)d[c].out_index, norm * n_sp, norm * n_tm,
                       norm * (n_sp + n_tm));
}

// Polyakov loop at spatial site blockIdx.x: Tr prod_t U_3(x, t), FP64.
// LDS: P, X, Tm.
template <typename T>
__global__ __launch_bounds__(kLanes) void k_polyakov(const T2<T>* __restrict__ U, Geom g, int n,
                                                     double* __restrict__ partial) {
    extern __shared__ double4 smem_poly[];
    const int n2 = n * n;
    double2* P = reinterpret_cast<double2*>(smem_poly);
    double2* X = P + n2;
    double2* Tm = X + n2;
    const int xs = blockIdx.x;
    const int Vs = g.V / g.L[3];
    for (int e = threadIdx.x; e < n2; e += kLanes) {
        const int i = e / n;
        P[e] = make_double2(i * n + i == e ? 1.0 : 0.0, 0.0);
    }
    for (int t = 0; t < g.L[3]; ++t) {
        const int s = xs + t * Vs;
        Site st;
        int r = s;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int q = r / g.L[m];
            st.x[m] = r - q * g.L[m];
            r = q;
        }
        st.s = s;
        lds_load<double, T>(X, link_at<T>(U, n2, 3, parity_of(st), s >> 1, g.Vh), n);
        __syncthreads();
        lds_mm<double>(Tm, P, X, n);
        __syncthreads();
        double2* tmp = P;
        P = Tm;
        Tm = tmp;
    }
    double tr = 0.0, ti = 0.0;
    for (int i = threadIdx.x; i < n; i += kLanes) {
        tr += P[i * n + i].x;
        ti += P[i * n + i].y;
    }
    tr = wave_sum(tr);
    ti = wave_sum(ti);
    if (threadIdx.x == 0) {
        partial[2 * (size_t)xs] = tr;
        partial[2 * (size_t)xs + 1] = ti;
    }
}

// Canonical FP64 field [mu][s][i][j] (re, im) <-> link-major storage; one
// work-item per complex entry.
template <typename T>
__global__ __launch_bounds__(256) void k_export(const T2<T>* __restrict__ U, Geom g, int n,
                                                double* __restrict__ out) {
    const int n2 = n * n;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= 4LL * g.V * n2) return;
    const int id = (int)(idx / n2), e = (int)(idx - (long long)id * n2);
    int mu, par, h;
    link_id(g, id, mu, par, h);
    const int s = site_of(g, par, h).s;
    const T2<T> v = link_at<T>(U, n2, mu, par, h, g.Vh)[e];
    double* o = out + (((size_t)mu * g.V + s) * n2 + e) * 2;
    o[0] = (double)v.x;
    o[1] = (double)v.y;
}

template <typename T>
__global__ __launch_bounds__(256) void k_import(T2<T>* __restrict__ U, Geom g, int n, const double* __restrict__ in) {
    const int n2 = n * n;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= 4LL * g.V * n2) return;
    const int id = (int)(idx / n2), e = (int)(idx - (long long)id * n2);
    int mu, par, h;
    link_id(g, id, mu, par, h);
    const int s = site_of(g, par, h).s;
    const double* p = in + (((size_t)mu * g.V + s) * n2 + e) * 2;
    T2<T>* dst = const_cast<T2<T>*>(link_at<T>(U, n2, mu, par, h, g.Vh));
    dst[e] = cpx<T>((T)p[0], (T)p[1]);
}

// ---------------------------------------------------------------------------
// The draw by place alone, for parity tests: element i is subgroup mu_sg +
// (i mod 8) of site i / 8.  dev_x gets 4n doubles, attempts n ints (the
// accepted attempt's number, 0 when all were rejected).
// ---------------------------------------------------------------------------
constexpr int kSampleSteps = 8;  // subgroups per site (and workgroup)
template <typename T>
__global__ __launch_bounds__(kLanes) void k_sample_su2_batched(const double* __restrict__ alpha, int n, uint32_t k0,
                                                               uint32_t k1, uint32_t step, uint32_t mu_sg,
                                                               double* __restrict__ x, int* __restrict__ attempts) {
    __shared__ DrawRec<T> rec[kSampleSteps];
    const uint32_t site = blockIdx.x;
    if (threadIdx.x < kPlaceLanes) fill_draws<T>(rec, kSampleSteps, mu_sg, k0, k1, site, step, 0u);
    __syncthreads();
    constexpr int kPlaces = kLanes / kPlaceLanes;
    for (int s0 = 0; s0 < kSampleSteps; s0 += kPlaces) {
        const int s = s0 + (int)threadIdx.x / kPlaceLanes, i = (int)site * kSampleSteps + s;
        Quat<T> q;
        const int a = place_draw<T>(i < n ? (T)alpha[i] : T(1), i < n, rec[s], k0, k1, site, step,
                                    mu_sg + (uint32_t)s, q);
        if (i < n && threadIdx.x % kPlaceLanes == 0) {
            if (a == 0) q = Quat<T>{{T(1), T(0), T(0), T(0)}};
#pragma unroll
            for (int c = 0; c < 4; ++c) x[4 * (size_t)i + c] = q.q[c];
            attempts[i] = a;
        }
    }
}

}  // namespace wide
}  // namespace sun
