// sun_wide_large.hpp -- the large-Nc phase update for 9 <= Nc <= 32: one
// link to a workgroup of two wavefronts.
//
// Products run on the matrix cores in both precisions.  Their k terms are
// summed one after another as fused multiply-adds (checked against a host
// chain of fma for the FP32 and FP64 shapes used here), so with the real
// and imaginary terms of a complex k interleaved along the matrix
// instruction's k every entry has the bits of the plain loop of complex
// multiply-adds.  Links are staged in LDS as they are, rows padded to an odd
// stride so that rows start in different banks; a daggered operand is read
// with its indices exchanged and its imaginary part negated.  The links of
// the next product load into registers while the matrix cores work.
//
// In the subgroup steps the first wavefront runs the chain on W = U A, four
// steps to a slot (sun_pairs.hpp), sixteen lanes to a step; the second draws
// the steps' random terms one batch of slots ahead and applies the finished
// rotations to U one batch behind.
//
// Bound at 8^4 (eight links on a CU, four wavefronts on a SIMD) by vector
// issue in the chain (about 1000 cycles per slot at Nc = 16 FP32) and, above
// Nc = 16, by the matrix cores, whose tiles are padded to 32.  Against one
// wavefront per link with products on the vector units (FP32 above Nc = 20 on
// unpadded LDS rows) and draws moved between lanes, 8^4, us per phase,
// overrelaxation and heatbath: SU(12) FP32 44 -> 30 and 74 -> 38, SU(16) FP64
// 89 -> 53 and 184 -> 93, SU(24) FP64 241 -> 191 and 436 -> 346, SU(32) FP32
// 228 -> 155 and 404 -> 196, SU(32) FP64 553 -> 387 and 881 -> 556; where the
// tiles are padded most, SU(17) FP64, 122 -> 115 and 226 -> 160.
#pragma once

#include <type_traits>

#include "sun_wide.hpp"

namespace sun {
namespace wide {

constexpr int kLargeThreads = 2 * kLanes;
constexpr int kSlotSteps = 4;   // steps per slot, one per place of sixteen lanes
constexpr int kBatchSlots = 4;  // slots between two hand-overs
static_assert(kSlotSteps * kPlaceLanes == kLanes, "a slot fills a wavefront");
static_assert(kBatchSlots * kSlotSteps * kRecLanes == kLanes, "a batch's draws fill a wavefront");
constexpr int kTile = 16;       // largest Nc of the one-tile form
constexpr int kMfmaMinN = 20;   // largest Nc whose FP32 products keep one k's terms together

// Ranges of Nc compiled apart: up to 16 (one 16 x 16 tile), to 19, to 25 and to
// 32 (entries of a link per lane: 2, 3, 5, 8).  With five entries a lane the
// FP64 overrelaxation of SU(17) spilled and took 125 us, SU(19) 142; with three
// 115 and 131.
constexpr int kLargeMax[4] = {kTile, 19, 25, kNcMax};
constexpr int large_loads(int range) {
    return (kLargeMax[range] * kLargeMax[range] + kLargeThreads - 1) / kLargeThreads;
}

// LDS matrices have an even number of rows, so that the products take k in
// pairs (row and column Nc of an odd Nc are zero), and an odd row stride; the
// last entry holds no matrix entry.
__host__ __device__ constexpr int row_count(int n) { return n + (n & 1); }
__host__ __device__ constexpr int row_stride(int n) { return row_count(n) + 1; }
__host__ __device__ constexpr int mat_entries(int n) { return row_count(n) * row_stride(n); }

// Attempts of a record that a Creutz draw can take: three in the last range's
// FP64 heatbath, which its registers hold to six links a CU whatever the LDS
// (with two, SU(24) 8^4 at beta 6.2, nearly all draws Creutz, ran 494 us a
// phase), elsewhere two.
template <typename T>
constexpr int creutz_words(int range) {
    return sizeof(T) == 8 && range == 3 ? 3 : 2;
}

// LDS after the two matrices: the rotations of two batches, and (heatbath)
// the draw records of two batches.
template <typename T, int RANGE>
struct alignas(16) LargeRing {
    Quat<T> a[2][kBatchSlots][kSlotSteps];
    // records of three words without padding: SU(26) FP64 with it has 5 links on
    // a CU instead of 6 (heatbath 358 -> 387 us)
    static constexpr int kWords = creutz_words<T>(RANGE);
    DrawRec<T, kWords, kWords == 3 ? 8 : 16> draw[2][kBatchSlots * kSlotSteps];
};
template <typename T, int RANGE>
constexpr size_t large_lds(int n, int hb) {
    using Ring = LargeRing<T, RANGE>;
    return (size_t)2 * mat_entries(n) * sizeof(T2<T>) + (hb ? sizeof(Ring) : sizeof(Ring::a));
}

static __constant__ pairs::Table<kSlotSteps> kSlotTable = pairs::make_table<kSlotSteps>();

// e / n for e < 1024, n <= 32, from inv = ceil(2^16 / n)
__device__ __forceinline__ int div_by(int e, int inv) { return (e * inv) >> 16; }

// Places of the entries threadIdx.x + THREADS c of a link in an LDS matrix;
// those past the link's end go to the entry that holds none.
template <int LOADS, int THREADS = kLargeThreads>
struct Places {
    int at[LOADS];
    __device__ __forceinline__ Places(int n, int n2) {
        const int inv = ((1 << 16) + n - 1) / n, pad = row_stride(n) - n;
#pragma unroll
        for (int c = 0; c < LOADS; ++c) {
            const int e = (int)threadIdx.x + c * THREADS;
            at[c] = e < n2 ? e + pad * div_by(e, inv) : mat_entries(n) - 1;
        }
    }
};
// Those entries of one link, in registers.
template <typename T, int LOADS, int THREADS = kLargeThreads>
struct LinkPart {
    T re[LOADS], im[LOADS];
    __device__ __forceinline__ void load(const T2<T>* __restrict__ src, int n2) {
#pragma unroll
        for (int c = 0; c < LOADS; ++c) {
            const T2<T> v = src[min((unsigned)threadIdx.x + c * THREADS, (unsigned)n2 - 1)];
            re[c] = v.x;
            im[c] = v.y;
        }
    }
    __device__ __forceinline__ void store(T2<T>* dst, const Places<LOADS, THREADS>& pl) const {
#pragma unroll
        for (int c = 0; c < LOADS; ++c) dst[pl.at[c]] = cpx<T>(re[c], im[c]);
    }
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
    using type = f32x4;
};
template <>
struct Vec4<double> {
    using type = f64x4;
};

__device__ __forceinline__ f32x4 mma16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mma16(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Row of result register r of a 16 x 16 tile in lane l (column l mod 16).
template <typename T>
__device__ __forceinline__ int tile_row(int l, int r) {
    return sizeof(T) == 4 ? 4 * (l >> 4) + r : (l >> 4) + 4 * r;
}

// The lane number, computed where it is asked for: the lane's LDS addresses
// of every product of the staple loop, moved out of the loop, would take more
// registers than the loop has (and did: they were spilled).
__device__ __forceinline__ int fresh_lane() {
    int l = (int)threadIdx.x & (kLanes - 1);
    asm volatile("" : "+v"(l));
    return l;
}

// use(read(s)) for s = 0 .. count - 1 (count > 0), the reads of CHUNK steps
// issued together (those past the end repeat the last).
template <int CHUNK, typename R, typename F>
__device__ __forceinline__ void for_steps(int count, R read, F use) {
    int s0 = 0;
    do {
        decltype(read(0)) o[CHUNK];
#pragma unroll
        for (int q = 0; q < CHUNK; ++q) o[q] = read(CHUNK == 1 ? s0 : min(s0 + q, count - 1));
#pragma unroll
        for (int q = 0; q < CHUNK; ++q)
            if (q == 0 || s0 + q < count) use(o[q]);
        s0 += CHUNK;
    } while (s0 < count);
}

// The product accumulator of a wavefront, C += A B with A, B in LDS (row
// stride ns), DA / DB: A^dag / B^dag in their place.
//
// Nc <= 16: one 16 x 16 tile, the real part on the first wavefront, the
// imaginary part on the second.  Lane l holds row (column) l mod 16 of A (B)
// and term l / 16 of the four that an instruction sums: complex k = 2 s + l /
// 32, first the terms of Re A (a_re b_re, a_re b_im), then those of Im A.
template <typename T, bool BIG>
struct Product {
    typename Vec4<T>::type c;
    struct Ops {
        T a, b;
    };
    __device__ __forceinline__ void zero() { c = typename Vec4<T>::type{0, 0, 0, 0}; }
    template <bool DA, bool DB>
    __device__ __forceinline__ void add(const T2<T>* A, const T2<T>* B, int n, int ns, int w) {
        const int l = fresh_lane();
        const int part = (l >> 4) & 1, kk = l >> 5, bpart = part ^ w;
        const int rc = min(l & 15, n - 1);
        const bool neg = (part && !w) ^ (DA && part) ^ (DB && bpart);
        const T* a = reinterpret_cast<const T*>(A) + part + 2 * (DA ? rc + kk * ns : rc * ns + kk);
        const T* b = reinterpret_cast<const T*>(B) + bpart + 2 * (DB ? rc * ns + kk : rc + kk * ns);
        const int da = DA ? 4 * ns : 4, db = DB ? 4 : 4 * ns;
        const int pairs = (n + 1) >> 1;
        for_steps<4>(pairs, [&](int s) { return Ops{a[s * da], b[s * db]}; },
                     [&](const Ops& o) { c = mma16(neg ? -o.a : o.a, o.b, c); });
    }
    __device__ __forceinline__ void store(T2<T>* C, int n, int ns, int w) const {
        const int l = fresh_lane();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = tile_row<T>(l, r), j = l & 15;
            if (i < n && j < n) reinterpret_cast<T*>(C)[2 * (i * ns + j) + w] = c[r];
        }
    }
};

// FP32, 16 < Nc: one 32 x 32 tile, real and imaginary part split as above.
// Up to kMfmaMinN an instruction sums the two terms of one complex k; above
// it the Re A terms of two k, then their Im A terms (both orders are part of
// the results' bits).
template <>
struct Product<float, true> {
    f32x16 c;
    struct Ops {
        float2 a, b;
    };
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] = 0.f;
    }
    template <bool DA, bool DB>
    __device__ __forceinline__ void add(const float2* A, const float2* B, int n, int ns, int w) {
        const int l = fresh_lane();
        const int hi = l >> 5, rc = min(l & 31, n - 1);
        if (n <= kMfmaMinN) {
            const int bpart = hi ^ w;
            const bool neg = (hi && !w) ^ (DA && hi) ^ (DB && bpart);
            const float* a = reinterpret_cast<const float*>(A) + hi + 2 * (DA ? rc : rc * ns);
            const float* b = reinterpret_cast<const float*>(B) + bpart + 2 * (DB ? rc * ns : rc);
            const int da = DA ? 2 * ns : 2, db = DB ? 2 : 2 * ns;
            for_steps<4>(n, [&](int k) { return make_float2(a[k * da], b[k * db]); },
                         [&](const float2& o) {
                             c = __builtin_amdgcn_mfma_f32_32x32x2f32(neg ? -o.x : o.x, o.y, c, 0, 0, 0);
                         });
            return;
        }
        const float2* a = A + (DA ? rc + hi * ns : rc * ns + hi);
        const float2* b = B + (DB ? rc * ns + hi : rc + hi * ns);
        const int da = DA ? 2 * ns : 2, db = DB ? 2 : 2 * ns;
        auto term = [&](float2 av, float2 bv) {
            if (DA) av.y = -av.y;
            if (DB) bv.y = -bv.y;
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, w ? bv.y : bv.x, c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(w ? av.y : -av.y, w ? bv.x : bv.y, c, 0, 0, 0);
        };
        const int pairs = (n + 1) >> 1;
        for_steps<4>(pairs, [&](int s) { return Ops{a[s * da], b[s * db]}; },
                     [&](const Ops& o) { term(o.a, o.b); });
    }
    __device__ __forceinline__ void store(float2* C, int n, int ns, int w) const {
        const int l = fresh_lane();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 8 * (r / 4) + 4 * (l >> 5) + r % 4, j = l & 31;
            if (i < n && j < n) reinterpret_cast<float*>(C)[2 * (i * ns + j) + w] = c[r];
        }
    }
};

// FP64, 16 < Nc: four 16 x 16 tiles, rows 0 .. 15 on the first wavefront, the
// others on the second.
template <>
struct Product<double, true> {
    f64x4 re[2], im[2];
    struct Ops {
        double a, same0, other0, same1, other1;
    };
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int t = 0; t < 2; ++t) re[t] = im[t] = f64x4{0, 0, 0, 0};
    }
    template <bool DA, bool DB>
    __device__ __forceinline__ void add(const double2* A, const double2* B, int n, int ns, int w) {
        const int l = fresh_lane();
        const int part = (l >> 4) & 1, kk = l >> 5;
        const int ra = min(kTile * w + (l & 15), n - 1);
        const int c0 = l & 15, c1 = min(kTile + (l & 15), n - 1);
        // re takes a_re b_re and -a_im b_im, im a_re b_im and a_im b_re: the
        // lane's part of A serves both, signs collected on it and on B's im
        const double* a = reinterpret_cast<const double*>(A + (DA ? ra + kk * ns : ra * ns + kk)) + part;
        const double* b0 = reinterpret_cast<const double*>(B + (DB ? c0 * ns + kk : c0 + kk * ns));
        const double* b1 = reinterpret_cast<const double*>(B + (DB ? c1 * ns + kk : c1 + kk * ns));
        const int da = DA ? 4 * ns : 4, db = DB ? 4 : 4 * ns;
        const bool neg_re = part && (!DA ^ DB), neg_im = (part && DA) ^ (!part && DB);
        for_steps<1>((n + 1) >> 1,
                     [&](int s) {
                         return Ops{a[s * da], b0[s * db + part], b0[s * db + 1 - part], b1[s * db + part],
                                    b1[s * db + 1 - part]};
                     },
                     [&](const Ops& o) {
                         const double ar = neg_re ? -o.a : o.a, am = neg_im ? -o.a : o.a;
                         re[0] = mma16(ar, o.same0, re[0]);
                         im[0] = mma16(am, o.other0, im[0]);
                         re[1] = mma16(ar, o.same1, re[1]);
                         im[1] = mma16(am, o.other1, im[1]);
                     });
    }
    __device__ __forceinline__ void store(double2* C, int n, int ns, int w) const {
        const int l = fresh_lane();
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = kTile * w + tile_row<double>(l, r), j = kTile * t + (l & 15);
                if (i < n && j < n) C[i * ns + j] = make_double2(re[t][r], im[t][r]);
            }
    }
};

// The steps of batch b for the lane's place, i | j << 8 of slot s in bits
// 16 s ..; kNoStep past the last slot.
static_assert(kBatchSlots == 4, "four steps to a 64-bit word");
__device__ __forceinline__ uint64_t batch_steps(const uint16_t* tab, int nslot, int b, int place) {
    uint64_t st = 0;
#pragma unroll
    for (int s = 0; s < kBatchSlots; ++s) {
        const int t = b * kBatchSlots + s;
        st |= (uint64_t)(t < nslot ? tab[t * kSlotSteps + place] : pairs::kNoStep) << (16 * s);
    }
    return st;
}

// The lane's columns c0, c0 + 16 (those below n; others repeat column 0 and
// are not written) of rows at ri and rj of an LDS matrix.
template <typename T, bool BIG>
struct RowPair {
    static constexpr int kCols = BIG ? 2 : 1;
    T2<T> x[kCols], y[kCols];
    __device__ __forceinline__ static int col(int c0, int k, int n) {
        const int c = c0 + k * kPlaceLanes;
        return c < n ? c : 0;
    }
    __device__ __forceinline__ void load(const T2<T>* ri, const T2<T>* rj, int c0, int n) {
#pragma unroll
        for (int k = 0; k < kCols; ++k) {
            x[k] = ri[col(c0, k, n)];
            y[k] = rj[col(c0, k, n)];
        }
    }
    // the rows left-multiplied by the 2x2 form of a
    __device__ __forceinline__ void rotate(T2<T>* ri, T2<T>* rj, int c0, int n, const Quat<T>& a) const {
#pragma unroll
        for (int k = 0; k < kCols; ++k)
            if (c0 + k * kPlaceLanes < n) rows_left_mul_at<T>(ri + c0 + k * kPlaceLanes, rj + c0 + k * kPlaceLanes, a, x[k], y[k]);
    }
};

// One phase of link h of one lattice.
template <typename T, int RANGE, bool HB>
__device__ __forceinline__ void update_link_large(T2<T>* __restrict__ U, const Geom& g, int n, int mu, int par, T beta,
                                                  uint32_t k0, uint32_t k1, uint32_t step, int h) {
    constexpr bool BIG = RANGE > 0;
    constexpr int kLoads = large_loads(RANGE);
    extern __shared__ double4 smem_large[];
    const int n2 = n * n, ns = row_stride(n);
    const Places<kLoads> pl(n, n2);
    T2<T>* const B0 = reinterpret_cast<T2<T>*>(smem_large);
    T2<T>* const B1 = B0 + mat_entries(n);
    LargeRing<T, RANGE>& ring = *reinterpret_cast<LargeRing<T, RANGE>*>(B1 + mat_entries(n));
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLanes);  // wavefront
    const int Vh = g.Vh;
    const Site x = site_of(g, par, h);
    const int op = par ^ 1;
    // The site and its neighbours are the workgroup's: scalar registers.
    const int xs = __builtin_amdgcn_readfirstlane(x.s);
    auto shift = [&](bool up, int m) { return __builtin_amdgcn_readfirstlane(step_shift(g, x, up, m)); };
    const int u0 = shift(true, 0), u1 = shift(true, 1), u2 = shift(true, 2), u3 = shift(true, 3);
    const int d0 = shift(false, 0), d1 = shift(false, 1), d2 = shift(false, 2), d3 = shift(false, 3);
    const int sp = xs + pick_dir(u0, u1, u2, u3, mu);  // x + mu
    auto next_dir = [&](int nu) {
        do ++nu;
        while (nu < 4 && (nu == mu || !((g.present >> nu) & 1)));
        return nu;
    };

    LinkPart<T, kLoads> fa, fb;
    auto load_upper = [&](int nu) {
        fa.load(link_at<T>(U, n2, nu, op, sp >> 1, Vh), n2);
        fb.load(link_at<T>(U, n2, mu, op, (xs + pick_dir(u0, u1, u2, u3, nu)) >> 1, Vh), n2);
    };
    auto load_lower = [&](int nu) {
        const int sh = pick_dir(d0, d1, d2, d3, nu);  // the same from x + mu: nu is another direction
        fa.load(link_at<T>(U, n2, nu, par, (sp + sh) >> 1, Vh), n2);
        fb.load(link_at<T>(U, n2, mu, op, (xs + sh) >> 1, Vh), n2);
    };
    int nu = next_dir(-1);
    if (nu < 4)
        load_upper(nu);
    else
        fb.load(link_at<T>(U, n2, mu, par, h, Vh), n2);
    if ((n & 1) && (int)threadIdx.x <= n) {  // row and column n of both matrices
        const int t = (int)threadIdx.x;
        B0[t * ns + n] = B0[n * ns + t] = B1[t * ns + n] = B1[n * ns + t] = cpx<T>(T(0), T(0));
    }
    Product<T, BIG> acc, m;
    acc.zero();
    while (nu < 4) {
        // upper staple U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
        fa.store(B0, pl);
        fb.store(B1, pl);
        fb.load(link_at<T>(U, n2, nu, par, h, Vh), n2);
        __syncthreads();
        m.zero();
        m.template add<false, true>(B0, B1, n, ns, w);
        __syncthreads();
        m.store(B0, n, ns, w);
        fb.store(B1, pl);
        load_lower(nu);
        __syncthreads();
        acc.template add<false, true>(B0, B1, n, ns, w);
        __syncthreads();
        // lower staple U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
        fa.store(B0, pl);
        fb.store(B1, pl);
        fb.load(link_at<T>(U, n2, nu, op, (xs + pick_dir(d0, d1, d2, d3, nu)) >> 1, Vh), n2);
        __syncthreads();
        m.zero();
        m.template add<true, true>(B0, B1, n, ns, w);
        __syncthreads();
        m.store(B0, n, ns, w);
        fb.store(B1, pl);
        nu = next_dir(nu);
        if (nu < 4)
            load_upper(nu);
        else
            fb.load(link_at<T>(U, n2, mu, par, h, Vh), n2);  // the link itself
        __syncthreads();
        acc.template add<false, false>(B0, B1, n, ns, w);
        __syncthreads();
    }
    T2<T>* const W = B0;
    T2<T>* const Us = B1;
    acc.store(B0, n, ns, w);
    fb.store(Us, pl);
    __syncthreads();
    m.zero();
    m.template add<false, false>(Us, B0, n, ns, w);  // W = U A
    __syncthreads();
    m.store(W, n, ns, w);

    // Batch b of slots: the second wavefront has drawn it before barrier b;
    // after it the first runs it and leaves its rotations in the ring, while
    // the second draws batch b + 1 and applies the rotations of batch b - 1
    // to U.  Both pass the same nbatch + 1 barriers.
    const uint16_t* const tab = reinterpret_cast<const uint16_t*>(kSlotTable.word) + kSlotTable.first[n] * kSlotSteps;
    const int nslot = kSlotTable.first[n + 1] - kSlotTable.first[n];
    const int nbatch = (nslot + kBatchSlots - 1) / kBatchSlots;
    const uint32_t mu_hi = (uint32_t)mu << 16;
    const int lane = (int)threadIdx.x & (kLanes - 1);
    const int place = lane / kPlaceLanes, c0 = lane % kPlaceLanes;
    if (w == 0) {
        const T cb = T(2) * beta / T(n);  // alpha = 2 beta k / n
        uint64_t next = batch_steps(tab, nslot, 0, place);
        for (int b = 0; b < nbatch; ++b) {
            uint64_t st = next;
            next = batch_steps(tab, nslot, b + 1, place);
            __syncthreads();
            const int slots = min(kBatchSlots, nslot - b * kBatchSlots);
#pragma unroll 1
            for (int s = 0; s < slots; ++s, st >>= 16) {
                // the lanes of an empty place read step (0, 1) and write nothing
                const uint32_t e = (uint32_t)st & 0xFFFFu;
                const bool mine = e != pairs::kNoStep;
                const int i = mine ? (int)(e & 0xFF) : 0, j = mine ? (int)(e >> 8) : 1;
                T2<T>* const wi = W + __mul24(i, ns);
                T2<T>* const wj = W + __mul24(j, ns);
                const T2<T> wii = wi[i], wij = wi[j], wji = wj[i], wjj = wj[j];
                RowPair<T, BIG> rows;
                rows.load(wi, wj, c0, n);
                Quat<T> p, v, a;
                p.q[0] = T(0.5) * (wii.x + wjj.x);
                p.q[3] = T(0.5) * (wii.y - wjj.y);
                p.q[2] = T(0.5) * (wij.x - wji.x);
                p.q[1] = T(0.5) * (wij.y + wji.y);
                const T k = chain_unit_quat(p, v);
                bool apply = mine;
                if constexpr (HB) {
                    Quat<T> dr;
                    const uint32_t sg = pairs::step_index(n, i, j);
                    apply = place_draw<T>(cb * k, mine, ring.draw[b & 1][s * kSlotSteps + place], k0, k1,
                                          (uint32_t)xs, step, mu_hi | sg, dr) != 0 && mine;
                    a = qmul(dr, qconj(v));
                    if (!apply) a = Quat<T>{{T(1), T(0), T(0), T(0)}};
                } else {
                    const Quat<T> vc = qconj(v);
                    a = qmul(vc, vc);
                }
                if (c0 == 0) ring.a[b & 1][s][place] = a;
                if (apply) rows.rotate(wi, wj, c0, n, a);
                wave_lds_order();
            }
        }
        __syncthreads();
    } else {
        auto draw = [&](int b) {
            if (!HB || b >= nbatch) return;
            // lanes 4 r ..: the attempts and the direction of record r (slot
            // r / 4, place r mod 4)
            const int r = lane / kRecLanes, t = b * kBatchSlots + r / kSlotSteps;
            const uint32_t e = t < nslot ? tab[t * kSlotSteps + r % kSlotSteps] : pairs::kNoStep;
            const uint32_t sg = e != pairs::kNoStep ? pairs::step_index(n, (int)(e & 0xFF), (int)(e >> 8)) : 0u;
            fill_draw<T>(ring.draw[b & 1][r], lane % kRecLanes, k0, k1, (uint32_t)xs, step, mu_hi | sg);
        };
        draw(0);
        for (int b = 0; b <= nbatch; ++b) {
            __syncthreads();
            draw(b + 1);
            if (b == 0) continue;
            uint64_t st = batch_steps(tab, nslot, b - 1, place);
            const int slots = min(kBatchSlots, nslot - (b - 1) * kBatchSlots);
            for (int s = 0; s < slots; ++s, st >>= 16) {
                const uint32_t e = (uint32_t)st & 0xFFFFu;
                const bool mine = e != pairs::kNoStep;
                T2<T>* const ui = Us + (mine ? __mul24((int)(e & 0xFF), ns) : 0);
                T2<T>* const uj = Us + (mine ? __mul24((int)(e >> 8), ns) : 0);
                RowPair<T, BIG> rows;
                rows.load(ui, uj, c0, n);
                const Quat<T> a = ring.a[(b - 1) & 1][s][place];
                if (mine) rows.rotate(ui, uj, c0, n, a);
                wave_lds_order();
            }
        }
    }
    __syncthreads();
    T2<T>* dst = const_cast<T2<T>*>(link_at<T>(U, n2, mu, par, h, Vh));
#pragma unroll
    for (int c = 0; c < kLoads; ++c) {
        const int e = (int)threadIdx.x + c * kLargeThreads;
        if (e < n2) dst[e] = Us[pl.at[c]];
    }
}

// Wavefronts per SIMD the registers allow: four (eight links on a CU) except
// for the FP64 tiles above Nc = 25, whose LDS leaves at most six links a CU.
constexpr int large_waves(int range, bool f64) { return f64 && range == 3 ? 3 : 4; }

// One phase of one lattice, workgroups in the XCD-aware order.
template <typename T, int RANGE, bool HB>
__global__ __launch_bounds__(kLargeThreads, large_waves(RANGE, sizeof(T) == 8)) void k_update_large(
    T2<T>* __restrict__ U, Geom g, int n, int mu, int par, T beta, uint32_t k0, uint32_t k1, uint32_t step) {
    update_link_large<T, RANGE, HB>(U, g, n, mu, par, beta, k0, k1, step, xcd_tile((int)blockIdx.x, (int)gridDim.x));
}

// One phase of every chain of a batch group (same Nc and precision): one
// workgroup per updated link of each chain, the chain found by binary search
// over the first-link prefix of the descriptor table (TILE_HALF_HB counts
// links here); coupling, Philox key and RNG step come from the table.
template <typename T, int RANGE, bool HB>
__global__ __launch_bounds__(kLargeThreads, large_waves(RANGE, sizeof(T) == 8)) void k_update_large_batch(
    const ChainDesc* __restrict__ d, int nchains, int n, int mu, int par, uint32_t step_offset) {
    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int c = find_chain<TILE_HALF_HB>(d, nchains, tile);
    const Geom g = d[c].g;
    if (!((g.present >> mu) & 1)) return;
    update_link_large<T, RANGE, HB>((T2<T>*)d[c].links, g, n, mu, par, (T)d[c].beta, d[c].k0, d[c].k1,
                                    (uint32_t)(d[c].step + step_offset), tile - d[c].tile0[TILE_HALF_HB]);
}

}  // namespace wide
}  // namespace sun
