// mf_common.hpp -- shared device definitions of the gfx950 matrix-free library.
//
// Q2 Lagrange elements on uniform hexahedra with 3x3x3 Gauss quadrature
// (App. B "Numerical framework": degree-2 elements, (k+1)^dim Gauss points).
// Everything a cell needs is expressed through three 3x3 matrices acting
// along one direction at a time (sum factorization):
//   S[q][a]  = l_a(xi_q)     value of node basis a at Gauss point q
//   D[q][p]  = L_p'(xi_q)    derivative of the Lagrange polynomial through
//                            the Gauss points (collocation derivative):
//                            exact for the quadratic restriction of a Q2
//                            function to a line
//   G[q][a]  = l_a'(xi_q)    = (D S)[q][a]
// With r = sqrt(15)/10 and xi = (1/2 - r, 1/2, 1/2 + r) these are
//   S = [[.3+r, .4, .3-r], [0, 1, 0], [.3-r, .4, .3+r]]
//   D = (1/r) [[-3/2, 2, -1/2], [-1/2, 0, 1/2], [1/2, -2, 3/2]]
//   G = [[-1-4r, 8r, 1-4r], [-1, 0, 1], [-1+4r, -8r, 1+4r]]
// and the weights are (5/18, 4/9, 5/18).  The 1/r of D is folded into the
// stiffness factors (it enters squared), so the kernels use D' = r D.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mf {

constexpr double kR = 0.38729833462074168851792653997823996;  // sqrt(15)/10
constexpr double kW0 = 5.0 / 18.0, kW1 = 4.0 / 9.0;

// Device mesh description (uniform box).
struct KMesh {
    int nx, ny, nz;     // cells
    int NX, NY, NZ;     // nodes per direction (2n+1)
    unsigned dirichlet; // face bits
    double hx, hy, hz;  // cell edges
    double lox, loy, loz;
    // floor(2^32 / d) (all ones for d = 1) of the divisors of a brick's index:
    // bricks along x and y, slabs of two and of four along x (see udiv)
    unsigned rbx, rby, rs2, rs4;
};

// n / d for a uniform d with r = floor(2^32 / d): the product's high word is
// n / d or one less for every n < 2^32, corrected once.  Five scalar
// instructions, where the compiler's division takes a chain of about 25
// through a vector reciprocal.
__host__ __device__ inline unsigned udiv_reciprocal(unsigned d) { return d == 1 ? 0xFFFFFFFFu : (unsigned)(0x100000000ull / d); }
__device__ __forceinline__ unsigned udiv(unsigned n, unsigned d, unsigned r)
{
    const unsigned q = __umulhi(n, r);
    return q + (n - q * d >= d ? 1u : 0u);
}

__device__ __forceinline__ bool node_constrained(const KMesh &m, int i, int j, int k)
{
    const unsigned f = m.dirichlet;
    return ((f & 1u) && i == 0) || ((f & 2u) && i == m.NX - 1) || ((f & 4u) && j == 0) ||
           ((f & 8u) && j == m.NY - 1) || ((f & 16u) && k == 0) || ((f & 32u) && k == m.NZ - 1);
}

__device__ __forceinline__ int64_t node_index(const KMesh &m, int i, int j, int k)
{
    return (int64_t)i + (int64_t)m.NX * ((int64_t)j + (int64_t)m.NY * k);
}

// ---------------------------------------------------------------------------
// 1D line operators on 3 values (in -> out), templated on the real type.
// ---------------------------------------------------------------------------

template <typename T> struct Q2 {
    static constexpr T s0 = T(0.3 + kR), s1 = T(0.4), s2 = T(0.3 - kR);
    static constexpr T g0 = T(-1.0 - 4.0 * kR), g1 = T(8.0 * kR), g2 = T(1.0 - 4.0 * kR);
    static constexpr T w0 = T(kW0), w1 = T(kW1);

    // values at Gauss points: out = S in
    static __device__ __forceinline__ void interp(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        o0 = s0 * i0 + s1 * i1 + s2 * i2;
        o1 = i1;
        o2 = s2 * i0 + s1 * i1 + s0 * i2;
    }
    // integration against node basis: out = S^T in
    static __device__ __forceinline__ void interpT(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        o0 = s0 * i0 + s2 * i2;
        o1 = s1 * (i0 + i2) + i1;
        o2 = s2 * i0 + s0 * i2;
    }
    // collocation derivative (scaled by r): out = D' in, in even/odd form:
    // with h = (i2 - i0) / 2 and w = 2 i1 - (i0 + i2), out = (h + w, h, h - w)
    // (6 operations instead of 8).
    static __device__ __forceinline__ void deriv(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        const T h = T(0.5) * (i2 - i0);
        const T w = T(2) * i1 - (i0 + i2);
        o0 = h + w;
        o1 = h;
        o2 = h - w;
    }
    // out = s D' in for a uniform scale s, in even/odd form:
    // with e = i0 + i2, h = s (i2 - i0) / 2, w = s (2 i1 - e):
    // o0 = w + h, o1 = h, o2 = h - w  (7 operations instead of 8 + 3).
    static __device__ __forceinline__ void deriv_scaled(T i0, T i1, T i2, T s, T &o0, T &o1, T &o2)
    {
        const T e = i0 + i2;
        const T h = (T(0.5) * s) * (i2 - i0);
        const T w = s * (T(2) * i1 - e);
        o0 = w + h;
        o1 = h;
        o2 = h - w;
    }
    // transposed collocation derivative accumulated: out += D'^T in
    static __device__ __forceinline__ void derivT_acc(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        o0 += T(-1.5) * i0 - T(0.5) * i1 + T(0.5) * i2;
        o1 += T(2) * (i0 - i2);
        o2 += T(-0.5) * i0 + T(0.5) * i1 + T(1.5) * i2;
    }
    // D'' = 2 D' = [[-3, 4, -1], [-1, 0, 1], [1, -4, 3]] (integer entries):
    // with d = i2 - i0 and w = 2 i1 - (i0 + i2), out = (d + 2w, d, d - 2w),
    // 5 operations.
    static __device__ __forceinline__ void deriv2(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        const T d = i2 - i0;
        const T w = T(2) * i1 - (i0 + i2);
        o0 = T(2) * w + d;
        o1 = d;
        o2 = T(-2) * w + d;
    }
    // out += D''^T in
    static __device__ __forceinline__ void deriv2T_acc(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        o0 += T(-3) * i0 - i1 + i2;
        o1 += T(4) * (i0 - i2);
        o2 += T(3) * i2 + (i1 - i0);
    }
    // out += 2 D''^T in
    static __device__ __forceinline__ void deriv2T_acc2(T i0, T i1, T i2, T &o0, T &o1, T &o2)
    {
        o0 += T(-6) * i0 - T(2) * (i1 - i2);
        o1 += T(8) * (i0 - i2);
        o2 += T(6) * i2 + T(2) * (i1 - i0);
    }
    static __device__ __forceinline__ T weight(int q) { return q == 1 ? w1 : w0; }
};

// Apply a line operator along direction DIR of a 3x3x3 register array
// (index a + 3b + 9c).
template <int DIR> __device__ __forceinline__ constexpr int lidx(int l, int m, int n)
{
    // l runs along DIR; (m, n) enumerate the other two directions
    return DIR == 0 ? l + 3 * m + 9 * n : (DIR == 1 ? m + 3 * l + 9 * n : m + 3 * n + 9 * l);
}

template <typename T, int DIR, typename F>
__device__ __forceinline__ void line_apply(const T *in, T *out, F f)
{
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            T o0, o1, o2;
            f(in[lidx<DIR>(0, m, n)], in[lidx<DIR>(1, m, n)], in[lidx<DIR>(2, m, n)], o0, o1, o2);
            out[lidx<DIR>(0, m, n)] = o0;
            out[lidx<DIR>(1, m, n)] = o1;
            out[lidx<DIR>(2, m, n)] = o2;
        }
}

// in-place S along all three directions: nodal -> Gauss point values
template <typename T> __device__ __forceinline__ void interp3(T *v)
{
    auto f = [](T a, T b, T c, T &x, T &y, T &z) { Q2<T>::interp(a, b, c, x, y, z); };
    line_apply<T, 0>(v, v, f);
    line_apply<T, 1>(v, v, f);
    line_apply<T, 2>(v, v, f);
}

// in-place S^T along all three directions: Gauss point values -> nodal integrals
template <typename T> __device__ __forceinline__ void interp3T(T *v)
{
    auto f = [](T a, T b, T c, T &x, T &y, T &z) { Q2<T>::interpT(a, b, c, x, y, z); };
    line_apply<T, 0>(v, v, f);
    line_apply<T, 1>(v, v, f);
    line_apply<T, 2>(v, v, f);
}

// Along direction DIR, line by line: t = ih D' u, g = c .* t, acc += D'^T g.
// Working on one 3-point line at a time keeps only 3 temporaries live.
template <typename T, int DIR, typename C>
__device__ __forceinline__ void grad_line_apply(const T *u, const C &c, T ih, T *acc)
{
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int i0 = lidx<DIR>(0, m, n), i1 = lidx<DIR>(1, m, n), i2 = lidx<DIR>(2, m, n);
            T t0, t1, t2;
            Q2<T>::deriv_scaled(u[i0], u[i1], u[i2], ih, t0, t1, t2);
            Q2<T>::derivT_acc(c[i0] * t0, c[i1] * t1, c[i2] * t2, acc[i0], acc[i1], acc[i2]);
        }
}

// The same with D'' and no scale (the scale is in c): acc += D''^T (c .* D'' u).
template <typename T, int DIR, typename C> __device__ __forceinline__ void grad2_line_apply(const T *u, const C &c, T *acc)
{
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int i0 = lidx<DIR>(0, m, n), i1 = lidx<DIR>(1, m, n), i2 = lidx<DIR>(2, m, n);
            T t0, t1, t2;
            Q2<T>::deriv2(u[i0], u[i1], u[i2], t0, t1, t2);
            Q2<T>::deriv2T_acc(c[i0] * t0, c[i1] * t1, c[i2] * t2, acc[i0], acc[i1], acc[i2]);
        }
}

// out = in contracted along direction DIR with M: out[.., a, ..] = sum_q M[q][a] in[.., q, ..]
// (M a 3x3 table over Gauss points q and nodes a; the diagonals and nodal
// blocks contract Gauss-point weights with squares and products of S and G).
template <int DIR, typename T> __device__ __forceinline__ void contract1d(const T *in, T *out, const T (&M)[3][3])
{
    constexpr int st = DIR == 0 ? 1 : (DIR == 1 ? 3 : 9);
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int a = (i / st) % 3, base = i - a * st;
        out[i] = M[0][a] * in[base] + M[1][a] * in[base + st] + M[2][a] * in[base + 2 * st];
    }
}

// Ordering point: all 27 values of v are computed before it and no memory
// access moves across it.  Placed at the phase boundaries of a cell's
// computation, it keeps the compiler from forming later passes early and
// merging them into one long live range.
__device__ __forceinline__ void pin27(double *v)
{
#pragma unroll
    for (int i = 0; i < 27; ++i) asm volatile("" : "+v"(v[i])::"memory");
}

// Velocity component DIR times the derivative along DIR, accumulated:
// cv += s w .* (D'_DIR u), line by line.
template <typename T, int DIR>
__device__ __forceinline__ void vel_grad_acc(const T *u, const T *w, T s, T *cv)
{
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int i0 = lidx<DIR>(0, m, n), i1 = lidx<DIR>(1, m, n), i2 = lidx<DIR>(2, m, n);
            T t0, t1, t2;
            Q2<T>::deriv(u[i0], u[i1], u[i2], t0, t1, t2);
            cv[i0] += s * w[i0] * t0;
            cv[i1] += s * w[i1] * t1;
            cv[i2] += s * w[i2] * t2;
        }
}

// Its transpose: acc += D'_DIR^T (s w .* z), line by line.
template <typename T, int DIR>
__device__ __forceinline__ void vel_gradT_acc(const T *z, const T *w, T s, T *acc)
{
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int i0 = lidx<DIR>(0, m, n), i1 = lidx<DIR>(1, m, n), i2 = lidx<DIR>(2, m, n);
            Q2<T>::derivT_acc(s * w[i0] * z[i0], s * w[i1] * z[i1], s * w[i2] * z[i2], acc[i0], acc[i1], acc[i2]);
        }
}

// Along direction DIR: out += ih * (D' a) .* (D' b), line by line.
template <typename T, int DIR>
__device__ __forceinline__ void grad_dot_acc(const T *a, const T *b, T ih, T *out)
{
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int i0 = lidx<DIR>(0, m, n), i1 = lidx<DIR>(1, m, n), i2 = lidx<DIR>(2, m, n);
            T a0, a1, a2, b0, b1, b2;
            Q2<T>::deriv(a[i0], a[i1], a[i2], a0, a1, a2);
            Q2<T>::deriv(b[i0], b[i1], b[i2], b0, b1, b2);
            out[i0] += ih * a0 * b0;
            out[i1] += ih * a1 * b1;
            out[i2] += ih * a2 * b2;
        }
}

// ---------------------------------------------------------------------------
// Smoothed Heaviside (Sec. 2.3, eq. heaviside) and its derivative.
// kind 0: H = clamp((1+phi)/2, 0, 1).  kind 1: sine form with the signed
// distance d = 2 eps artanh(phi) recovered from the tanh profile.
// ---------------------------------------------------------------------------

// Linear form, branch free.
template <typename T> __device__ __forceinline__ T heaviside_linear(T phi)
{
    return fmin(fmax(T(0.5) + T(0.5) * phi, T(0)), T(1));
}

// Sine form in FP64.  With d = 2 eps artanh(phi) the thickness parameter
// cancels: with L = 2 artanh(phi) = d / eps, the form
//   H = 1/2 + L/6 + sin(pi L/3) / (2 pi)  for |L| < 3 (|phi| < tanh(3/2)), else 0 or 1,
//   dH/dphi = (1 + cos(pi L/3)) / (3 (1 - phi^2))  there, else 0,
// is a function of phi alone: H - 1/2 is phi times an even function and
// dH/dphi is even, both smooth in t = phi^2 on [0, tanh(3/2)^2].  They are
// evaluated as polynomials in x = 2 t / tanh(3/2)^2 - 1 on [-1, 1], the
// Chebyshev interpolants of those functions (computed with 60 digits),
// truncated where the rest is below 3e-17 (H) and 3e-17 (dH/dphi).  Error
// against 64-digit values over 20000 points: H max 2.2e-16, rms 3.8e-17;
// dH/dphi max 3.5e-16, rms 8.3e-17 (through atanh, sin and cos: 2.2e-16,
// 5.3e-17; 5.0e-16, 9.4e-17).  A call through the three library functions
// cost about 1100 SIMD cycles per Gauss point and wavefront, against 39 fused
// multiply-adds here (4 cycles each): FP64 heat apply at 50x37x61 cells 53.2
// -> 24.7 us, source assembly and transport velocity at 64^3 252 -> 189 us.
__device__ constexpr double kSineP = 0.9051482536448664382423037;  // tanh(3/2)
__device__ constexpr double kSineX = 2.441128044016478105990102;   // 2 / tanh(3/2)^2
constexpr int kSineNH = 39, kSineND = 45;
__device__ constexpr double kSineH[39] = {
    6.43520269740246897e-01, -4.43126021180735227e-02, -3.07422505219364268e-02, -1.32877722172321227e-02,
    -4.86526952347678121e-03, -1.27799812199075693e-03, 1.12047235257928406e-04, 5.55960170554967376e-04,
    6.16186723109304652e-04, 5.38839683093071849e-04, 4.27405438207980378e-04, 3.21889722882067689e-04,
    2.35013445340591370e-04, 1.68793312227063304e-04, 1.19557771058572304e-04, 7.97900624346346041e-05,
    5.32658912965180555e-05, 5.47927292189657968e-05, 4.59433262017686170e-05, -3.33605873700981357e-05,
    -4.73178319148966249e-05, 1.46694300141124250e-04, 1.55576753891603620e-04, -2.75924412134287509e-04,
    -2.84670103517266045e-04, 4.37552290079588077e-04, 4.27085646005613269e-04, -5.15154961072379321e-04,
    -4.81870352193232334e-04, 4.58090215840123579e-04, 4.11265987496103403e-04, -2.94906038246385332e-04,
    -2.55217387973624005e-04, 1.31166676993557050e-04, 1.09647570983554440e-04, -3.60687829282825838e-05,
    -2.91975073798846566e-05, 4.73298787729888257e-06, 3.70927825700015205e-06,
};
__device__ constexpr double kSineD[45] = {
    5.54895065504099172e-01, -2.55906808441978995e-01, -2.33437885912560039e-01, -1.31936561704740690e-01,
    -5.65674069933000609e-02, -1.27134128334104590e-02, 9.24005939123523357e-03, 1.81984025501983199e-02,
    2.01742155920174270e-02, 1.87857844953160137e-02, 1.60581769592588464e-02, 1.30477405846037512e-02,
    1.02533638547828553e-02, 7.86678329694943425e-03, 5.93149134900614050e-03, 4.44216665234599059e-03,
    3.29082112994548903e-03, 2.22522258316671870e-03, 1.51143640624501951e-03, 1.99620976918712207e-03,
    1.87169951860786249e-03, -2.24873853880814059e-03, -3.06572474141258121e-03, 9.04569019929043865e-03,
    1.02694728774525741e-02, -2.07138587294071232e-02, -2.27086457803105553e-02, 3.97782942124349920e-02,
    4.14854239906509020e-02, -5.98630433983693006e-02, -5.99021531908460053e-02, 7.13157838918452164e-02,
    6.86417745938329160e-02, -6.61284572939923598e-02, -6.14361358456230328e-02, 4.68670946654939150e-02,
    4.21322547982579676e-02, -2.45305185145998396e-02, -2.13887613793536414e-02, 8.96477507430815460e-03,
    7.59499567634474692e-03, -2.04856393825841648e-03, -1.68895744109442600e-03, 2.22682085091917352e-04,
    1.78752976096558329e-04,
};

// The two constant parts: 0 and 1 outside the interface, and a NaN stays one.
__device__ __forceinline__ double sine_saturated(double p, double inside)
{
    const double r = p >= kSineP ? 1.0 : inside;
    return p <= -kSineP ? 0.0 : r;
}

// N values of H at p (in place).  The points advance together through the
// polynomial, so that each coefficient is brought into scalar registers once
// for N of them and N independent chains cover the multiply-add latency.
template <int N> __device__ __forceinline__ void sine_values(double *p)
{
    double x[N], r[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        x[j] = __builtin_fma(p[j] * p[j], kSineX, -1.0);
        r[j] = kSineH[kSineNH - 1];
    }
#pragma unroll
    for (int k = kSineNH - 2; k >= 0; --k)
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = __builtin_fma(r[j], x[j], kSineH[k]);
#pragma unroll
    for (int j = 0; j < N; ++j) p[j] = sine_saturated(p[j], __builtin_fma(p[j], r[j], 0.5));
}

// dH/dphi at N points p, into d (which may be p).
template <int N> __device__ __forceinline__ void sine_derivatives(const double *p, double *d)
{
    double x[N], r[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        x[j] = __builtin_fma(p[j] * p[j], kSineX, -1.0);
        r[j] = kSineD[kSineND - 1];
    }
#pragma unroll
    for (int k = kSineND - 2; k >= 0; --k)
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = __builtin_fma(r[j], x[j], kSineD[k]);
#pragma unroll
    for (int j = 0; j < N; ++j) d[j] = fabs(p[j]) >= kSineP ? 0.0 : r[j];
}

// Whether any of the wavefront's NQ interpolated level-set values lies inside
// the interface.  Away from it, on most bricks of a mesh with an interface a
// few cells wide, H is 0 or 1 and the polynomials are skipped (a uniform
// branch; NaNs are not seen here and pass through sine_saturated).
template <int NQ, typename T> __device__ __forceinline__ bool sine_inside(const T *p)
{
    T m = fabs(p[0]);
#pragma unroll
    for (int q = 1; q < NQ; ++q) m = fmin(m, fabs(p[q]));
    return __ballot(m < T(kSineP)) != 0;
}

// H of the sine form at NQ points (in place), G points at a time (NQ a
// multiple of G; G sets the registers in flight, 6 G).
template <int NQ, int G, typename T> __device__ __forceinline__ void heaviside_sine(T *p)
{
    static_assert(NQ % G == 0, "whole groups");
    if (sine_inside<NQ>(p)) {
#pragma unroll
        for (int q = 0; q < NQ; q += G) {
            double v[G];
#pragma unroll
            for (int j = 0; j < G; ++j) v[j] = (double)p[q + j];
            sine_values<G>(v);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                p[q + j] = T(v[j]);
                asm volatile("" : "+v"(p[q + j])); // one group at a time
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < NQ; ++q) p[q] = T(sine_saturated((double)p[q], (double)p[q]));
    }
}

// dH/dphi of the sine form at NQ points of p, into d (may be p).
template <int NQ, int G> __device__ __forceinline__ void heaviside_sine_derivative(const double *p, double *d)
{
    static_assert(NQ % G == 0, "whole groups");
    if (sine_inside<NQ>(p)) {
#pragma unroll
        for (int q = 0; q < NQ; q += G) {
            double v[G];
            sine_derivatives<G>(p + q, v);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                d[q + j] = v[j];
                asm volatile("" : "+v"(d[q + j])); // one group at a time
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < NQ; ++q) d[q] = p[q] == p[q] ? 0.0 : p[q];
    }
}

// dH/dphi of the linear form.
__device__ __forceinline__ double heaviside_linear_derivative(double phi) { return (phi > -1.0 && phi < 1.0) ? 0.5 : 0.0; }

// ---------------------------------------------------------------------------
// Deterministic reductions without atomics.  A block sums its threads' values
// in a fixed tree order and stores one partial per set with a plain store
// (layout [NV][nblocks]).  A later launch, whose start makes those stores
// visible, sums the partials in a fixed order: every reader of a partial set
// obtains bitwise the same total, and no workgroup waits on another.
// (A last-block-arrives scheme needs one device-scope acquire-release atomic
// per workgroup on a single address; with thousands of workgroups these
// serialize across the XCDs and cost more than the kernel's own work.)
// ---------------------------------------------------------------------------

template <int NT> __device__ __forceinline__ double block_sum(double v, double *red)
{
    const int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
#pragma unroll
    for (int s = NT / 2; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// Store NV block sums (valid in thread 0) as partial `block` of each set.
template <int NV>
__device__ __forceinline__ void write_partials(const double *v, double *partials, unsigned nblocks, unsigned block)
{
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) partials[(size_t)i * nblocks + block] = v[i];
    }
}

// Sum over the wavefront, identical in every lane.
__device__ __forceinline__ double wave_total(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return __shfl(v, 0, 64);
}

// One lane's share of a set of n partials, entries lane, lane + 64, ..., eight
// loads in flight.
__device__ __forceinline__ double lane_partials(const double *p, unsigned n, unsigned lane)
{
    double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (unsigned b = lane; b < n; b += 512) {
#pragma unroll
        for (unsigned k = 0; k < 8; ++k) s[k] += b + 64 * k < n ? p[b + 64 * k] : 0.0;
    }
    return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// Total of partial set i (nblocks entries written by an earlier launch),
// returned to every thread of an NT-thread block.  Thread t sums entries
// t, t + NT, ... with four interleaved accumulators (combined in a fixed
// order), then the block sums the threads in a fixed tree.
template <int NT>
__device__ __forceinline__ double sum_partials(const double *partials, unsigned nblocks, int i, double *red)
{
    const double *p = partials + (size_t)i * nblocks;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    unsigned b = threadIdx.x;
    for (; b + 3 * NT < nblocks; b += 4 * NT) {
        s0 += p[b];
        s1 += p[b + NT];
        s2 += p[b + 2 * NT];
        s3 += p[b + 3 * NT];
    }
    for (; b < nblocks; b += NT) s0 += p[b];
    return block_sum<NT>((s0 + s1) + (s2 + s3), red);
}

} // namespace mf
