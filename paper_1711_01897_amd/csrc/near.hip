// Singular (vertex-sharing) triangle pairs on the device: the Laplace and
// Helmholtz single and double layer, P0 and P1 (P1: 3 x 3 local matrices,
// summed into the entries by a fixed-order gather), and the P1 Laplace and
// Helmholtz hypersingular operator.
//
// The regular kernels integrate vertex-disjoint pairs only; Section 3.2.3
// gives identical, edge-adjacent and vertex-adjacent pairs to a separate
// singular scheme.  Here each such pair is written in coordinates around its
// singular set in which x - y is (radius) x (a vector of the remaining
// coordinates).  Both kernels are homogeneous in x - y (degree -1 for 1/r,
// -2 for (x-y).n_y / r^3, where only the test side's out-of-plane part
// survives in the numerator), so the radial integral is a polynomial one and
// is done in closed form; what remains is smooth and goes to a composite
// Gauss-Legendre rule:
//   identical:     the six-region decomposition of T x T over the reference
//                  triangle {0 <= x2 <= x1 <= 1} (Jacobian xi^3 eta1^2 eta2);
//                  x - y = xi eta1 eta2 c(eta3) with c one of three lines in
//                  the plane of the edges, so the single layer is
//                  (1/3) sum_c int_0^1 d(eta3) / |c(eta3)| and the double
//                  layer vanishes (x - y lies in the plane);
//   common edge:   affine coordinates x = P + u1 E + s1 a, y = P + u2 E + s2 b
//                  (E the shared edge, a, b to the third vertices); the three
//                  small coordinates (u1 - u2, s1, s2) in cone coordinates of
//                  radius rho = max(s2, s1 + u1 - u2) (or its mirror), the
//                  along-edge coordinate leaving a segment of length 1 - rho:
//                  radial factor int rho (1 - rho) = 1/6 (single layer) or
//                  int (1 - rho) = 1/2 (double layer), four faces of the
//                  unit cone, each a square or a collapsed square;
//   common vertex: Duffy coordinates from the shared vertex ordered by the
//                  larger radius s (Jacobian s^3 z), x - y = s (a(u) - z b(v))
//                  or s (z a(u) - b(v)): radial factor 1/3 or 1/2, a 3D
//                  integral over (z, u, v).
// Rules: 16 points per direction (two panels of the 8-point rule; 32 for the
// identical case's 1D integrals): about 1e-12 relative on these pairs, where
// the full 4D tensor rule with 8 points per direction left ~1e-8.
// Helmholtz: g = e^{ikr}/(4 pi r) and its normal derivative
// e^{ikr} (1 - ikr) (x-y).n_y / (4 pi r^3) are the Laplace kernels times a
// factor smooth in the radius, so the same coordinates apply with the radial
// integral int pi(rho) e^{i omega rho} (1 - i omega rho)^[double layer] d rho
// (omega = k |c|, pi the Laplace case's radial polynomial, identical pairs
// after folding xi eta1 eta2 into one radius with weight (1 - p)^2) taken
// as its power series sum_n (i omega)^n mu_n c_n / n! (mu_n the moments of
// pi, c_n = 1, or 1 - n with the double layer's factor), up to 48 terms in
// Horner form (series_terms): ~1e-14 relative at omega = 6 (two elements per
// wavelength reach omega ~ 2 pi), 5e-10 at omega = 12 where the alternating
// terms cancel.
// What bounds these kernels is FP64 arithmetic: one workgroup per pair, a
// thousand or more products per thread; its 24-byte record, 32 bytes of vertex ids,
// 120 of vertices and 64 of normals and areas come through scalar loads, and 160 bytes
// at most are written (P0: one entry).
// P1 Helmholtz single layer, 2,900 pairs of a 100 x 100 leaf at 10 elements per
// wavelength: 101 us (336 us with 48 terms from LDS, the nine entries
// accumulated at every point and a tree reduction); P1 Laplace, the pairs of
// one dense leaf: 20 us a launch in an H-matrix assembly (41 us).
// The adjoint double layer is the double layer with test and trial exchanged
// (load_pair).
#include <hip/hip_runtime.h>

#include "bem_internal.hpp"
#include "f64_math.hpp"

namespace bem {
namespace {

constexpr int kGL = 8;          // Gauss-Legendre points per panel
constexpr int kPts = 2 * kGL;   // composite rule: two panels per direction
constexpr int kIdPanels = 4;    // identical pairs: 1D integrals on four panels
constexpr int kIdPts = kIdPanels * kGL;
constexpr int kNearThreads = 256;
static_assert(kPts * kPts == kNearThreads, "common-vertex pairs take one (u, v) node per thread");
static_assert(4 * kPts * 4 == kNearThreads, "common-edge pairs take (face, p, q group) per thread");
static_assert(3 * kIdPts <= kNearThreads, "identical pairs take one (line, node) per thread");

// 8-point Gauss-Legendre rule on [0, 1] (nodes (1 + x)/2, weights w/2 of the
// published rule on [-1, 1]).
__constant__ double c_x[kGL] = {0.5 * (1.0 - 0.9602898564975363), 0.5 * (1.0 - 0.7966664774136267),
                                0.5 * (1.0 - 0.5255324099163290), 0.5 * (1.0 - 0.1834346424956498),
                                0.5 * (1.0 + 0.1834346424956498), 0.5 * (1.0 + 0.5255324099163290),
                                0.5 * (1.0 + 0.7966664774136267), 0.5 * (1.0 + 0.9602898564975363)};
__constant__ double c_w[kGL] = {0.5 * 0.1012285362903763, 0.5 * 0.2223810344533745, 0.5 * 0.3137066458778873,
                                0.5 * 0.3626837833783620, 0.5 * 0.3626837833783620, 0.5 * 0.3137066458778873,
                                0.5 * 0.2223810344533745, 0.5 * 0.1012285362903763};

constexpr double kInv4PiD = 0.0795774715459476678844418816862571;

struct V3 {
    double x, y, z;
};
__device__ __forceinline__ V3 ld(const double *p) { return {p[0], p[1], p[2]}; }
__device__ __forceinline__ V3 add(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 sub(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 mul(double s, V3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ V3 fma3(double s, V3 a, V3 b) { return {fma(s, a.x, b.x), fma(s, a.y, b.y), fma(s, a.z, b.z)}; }
__device__ __forceinline__ double dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }

// A vertex-sharing pair as the integrals need it (workgroup-uniform, built
// from the mesh by scalar loads):
//   kind 0, identical:     v = V0, V1, V2 (the triangle in its own order)
//   kind 1, common edge:   v = P, Q, A, B (shared edge P-Q; A the test
//                          triangle's third vertex, B the trial triangle's)
//   kind 2, common vertex: v = P, A, B, C, D (shared P; A, B the test
//                          triangle's others, C, D the trial triangle's)
// ny: unit normal of the trial triangle; jt, js: |cross| of the test and trial
// triangles (twice their areas); pt, ps: the triangles' local vertices in the
// order of v.
struct Pair {
    double v[15];
    double ny[3], nt[3];
    double jt, js, k;
    int kind;
    int T, S;
    int pt[3], ps[3];
};

// Mesh tables and lists in constant memory space: written before the kernels
// that read them, and read here at wave-uniform addresses (scalar loads).
#define BEM_CONST(T) const __attribute__((address_space(4))) T
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ Pair load_pair(const NearReq &R, int a, int b)
{
    Pair q;
    q.T = R.transposed ? b : a;
    q.S = R.transposed ? a : b;
    q.k = R.k;
    BEM_CONST(i32x4) *vtx = (BEM_CONST(i32x4) *)R.vtx;
    const i32x4 tv = vtx[q.T], sv = vtx[q.S];
    // bit 3 i + j: test vertex i is trial vertex j; the first two give the
    // shared vertices' local numbers t0, s0 and t1, s1 in the test triangle's
    // order (scalar arithmetic: the vertices then come through scalar loads)
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) m |= (tv[i] == sv[j] ? 1u : 0u) << (3 * i + j);
    m = __builtin_amdgcn_readfirstlane(m);
    const int n = __builtin_popcount(m);
    const unsigned m2 = m & (m - 1);
    const int b0 = m ? __builtin_ctz(m) : 0, b1 = m2 ? __builtin_ctz(m2) : 0;
    const int t0 = b0 / 3, s0 = b0 - 3 * t0, t1 = b1 / 3, s1 = b1 - 3 * t1;
    q.kind = n >= 3 ? 0 : (n == 2 ? 1 : 2);
    auto next = [](int i) { return i == 2 ? 0 : i + 1; };
    // identical: t0 = 0, t1 = 1 and s0, s1 where the trial triangle, which may list
    // the three vertices in another order (a triangle that the mesh holds twice),
    // has them
    q.pt[0] = t0;
    q.pt[1] = q.kind == 2 ? next(t0) : t1;
    q.pt[2] = 3 - q.pt[0] - q.pt[1];
    q.ps[0] = s0;
    q.ps[1] = q.kind == 2 ? next(s0) : s1;
    q.ps[2] = 3 - q.ps[0] - q.ps[1];
    auto pick = [](const i32x4 &v, int i) { return i == 0 ? v.x : (i == 1 ? v.y : v.z); };
    // v[3], v[4]: the trial triangle's vertices that are not shared (B; C, D),
    // the shared vertex where there is no such vertex
    const int id[5] = {pick(tv, q.pt[0]), pick(tv, q.pt[1]), pick(tv, q.pt[2]),
                       q.kind == 0 ? pick(tv, 0) : pick(sv, q.kind == 1 ? q.ps[2] : q.ps[1]),
                       q.kind == 2 ? pick(sv, q.ps[2]) : pick(tv, q.pt[0])};
    BEM_CONST(double) *xyz = (BEM_CONST(double) *)R.xyz;
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int d = 0; d < 3; ++d) q.v[3 * i + d] = xyz[3 * (size_t)id[i] + d];
    BEM_CONST(double) *gt = (BEM_CONST(double) *)(R.g64 + (size_t)q.T * kGeo64Stride);
    BEM_CONST(double) *gs = (BEM_CONST(double) *)(R.g64 + (size_t)q.S * kGeo64Stride);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        q.nt[d] = gt[d];
        q.ny[d] = gs[d];
    }
    q.jt = gt[3];
    q.js = gs[3];
    return q;
}

struct Cx {
    double re, im;
};

// Power series of the radial integrals
//   int_0^1 rho^A (1 - rho)^B e^{i om rho} (1 - i om rho)^[DL] d rho  (B <= 2):
// coefficients of om^(2m) (real part) and om^(2m+1) (imaginary part), signs of
// i^n included, moments of rho^A (1 - rho)^B.  N = 1: one integral; N = 3: A,
// A + 1 and A + 2 interleaved (the P1 local matrices, whose barycentrics are
// affine in rho).
constexpr int kSeries = 48;
template <int A, int B, bool DL, int N>
struct RadialTable {
    double v[2 * N * (kSeries / 2)];
    constexpr RadialTable() : v()
    {
        for (int j = 0; j < N; ++j) {
            double fact = 1.0;
            for (int n = 0; n < kSeries; ++n) {
                if (n > 0) fact *= n;
                const double e = n + A + j;
                const double mu = B == 0 ? 1.0 / (e + 1)
                                : B == 1 ? 1.0 / ((e + 1) * (e + 2))
                                         : 2.0 / ((e + 1) * (e + 2) * (e + 3));
                const double a = mu * (DL ? 1.0 - n : 1.0) / fact;
                const int m = n / 2;
                v[2 * N * m + 2 * j + n % 2] = (m % 2) ? -a : a;
            }
        }
    }
};
// P0: identical (after folding xi eta1 eta2 into one radius), common edge and
// common vertex; single and double layer
__constant__ RadialTable<0, 2, false, 1> c_rad_s0{};
__constant__ RadialTable<1, 1, false, 1> c_rad_s1{};
__constant__ RadialTable<2, 0, false, 1> c_rad_s2{};
__constant__ RadialTable<0, 1, true, 1> c_rad_d1{};
__constant__ RadialTable<1, 0, true, 1> c_rad_d2{};
// P1: identical and common vertex, common edge
__constant__ RadialTable<2, 0, false, 3> c_tab_s2{};
__constant__ RadialTable<1, 1, false, 3> c_tab_s1{};
__constant__ RadialTable<1, 0, true, 3> c_tab_d2{};
__constant__ RadialTable<0, 1, true, 3> c_tab_d1{};

// Series terms a pair needs: the smallest multiple of 8 for which
// om^n / n! <= 2^-64 at the largest omega of its integration domain, so that
// what is left out is far below the rounding of what is kept; all 48 beyond
// om = 5.2.  omega = k |c| <= k times the largest distance of two of the pair's
// vertices (c is a difference of points of the two triangles, |c| convex in
// both).  Ten elements per wavelength reach om = 1.3 and take 24 terms, half
// the work of the fixed 48; the count is the workgroup's, so the coefficients
// come through scalar loads and feed two evaluations each (held in LDS they
// cost a broadcast read per product, which bound the kernel).
__device__ __forceinline__ int series_terms(const Pair &it)
{
    double d2 = 0.0;
#pragma unroll
    for (int i = 0; i < 5; ++i)   // vertices a kind lacks repeat the first
#pragma unroll
        for (int j = i + 1; j < 5; ++j) {
            const double x = it.v[3 * i] - it.v[3 * j], y = it.v[3 * i + 1] - it.v[3 * j + 1],
                         z = it.v[3 * i + 2] - it.v[3 * j + 2];
            d2 = fmax(d2, x * x + y * y + z * z);
        }
    const double w2 = d2 * it.k * it.k;
    const int n = w2 <= 0.0147 * 0.0147 ? 8 : w2 <= 0.425 * 0.425 ? 16 : w2 <= 1.54 * 1.54 ? 24
                : w2 <= 3.19 * 3.19 ? 32 : w2 <= 5.2 * 5.2 ? 40 : kSeries;
    return __builtin_amdgcn_readfirstlane(n);
}

// N radial integrals at two omegas, Horner in omega^2, highest term first.
template <int N>
__device__ __forceinline__ void radial2(double oa, double ob, const double *tab, int terms, Cx *Ja, Cx *Jb)
{
    const double wa = oa * oa, wb = ob * ob;
#pragma unroll
    for (int j = 0; j < N; ++j) Ja[j] = Jb[j] = {0.0, 0.0};
#pragma unroll 1
    for (int m = terms / 2 - 4; m >= 0; m -= 4) {
#pragma unroll
        for (int u = 3; u >= 0; --u) {
            const double *c = tab + 2 * N * (m + u);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                Ja[j].re = fma(Ja[j].re, wa, c[2 * j]);
                Ja[j].im = fma(Ja[j].im, wa, c[2 * j + 1]);
                Jb[j].re = fma(Jb[j].re, wb, c[2 * j]);
                Jb[j].im = fma(Jb[j].im, wb, c[2 * j + 1]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        Ja[j].im *= oa;
        Jb[j].im *= ob;
    }
}

// Helmholtz share of this thread (op 2 single layer, op 3 double layer),
// without jt js / 4 pi and (a.n_y) for common-edge double layers.
template <int OP>
__device__ Cx pair_part_helmholtz(const Pair &it, const double *sx, const double *sw)
{
    constexpr bool DL = OP == 3;
    const int t = threadIdx.x;
    const double k = it.k;
    const int terms = series_terms(it);
    if (it.kind == 0) {
        if (DL || t >= 3 * kIdPts) return {0.0, 0.0};
        const V3 V0 = ld(it.v), V1 = ld(it.v + 3), V2 = ld(it.v + 6);
        const V3 E1 = sub(V1, V0), E2 = sub(V2, V1);
        const int line = t / kIdPts, kk = t - line * kIdPts;
        const double e = (c_x[kk % kGL] + (double)(kk / kGL)) * (1.0 / kIdPanels);
        const double w = c_w[kk % kGL] * (1.0 / kIdPanels);
        const V3 c = line == 0 ? fma3(e, E1, E2) : (line == 1 ? fma3(e, E2, E1) : fma3(-e, E1, mul(1.0 - e, E2)));
        const double c2 = dot(c, c), ri = rsqrt64(c2);
        Cx rad, unused;
        radial2<1>(k * c2 * ri, 0.0, c_rad_s0.v, terms, &rad, &unused);
        return {w * ri * rad.re, w * ri * rad.im};
    }
    double ar = 0.0, ai = 0.0;
    if (it.kind == 1) {
        const V3 P = ld(it.v), Q = ld(it.v + 3), A = ld(it.v + 6), B = ld(it.v + 9);
        const V3 E = sub(Q, P), a = sub(A, P), b = sub(B, P);
        const int face = t >> 6, ip = (t >> 2) & (kPts - 1), g = t & 3;
        const double p = sx[ip], q1 = 1.0 - p;
        V3 c0, c1;
        double s1c, s1q, fw;
        if (face == 0) {
            c0 = sub(mul(p, E), b), c1 = mul(q1, a), s1c = 0.0, s1q = q1, fw = q1;
        } else if (face == 1) {
            c0 = fma3(p, E, mul(q1, a)), c1 = mul(-1.0, b), s1c = q1, s1q = 0.0, fw = 1.0;
        } else if (face == 2) {
            c0 = fma3(-p, E, a), c1 = mul(-q1, b), s1c = 1.0, s1q = 0.0, fw = q1;
        } else {
            c0 = fma3(-p, E, mul(-q1, b)), c1 = a, s1c = 0.0, s1q = 1.0, fw = 1.0;
        }
        for (int j = 0; j < kPts / 4; j += 2) {
            double f[2], om[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double q = sx[g + 4 * (j + h)];
                const V3 c = fma3(q, c1, c0);
                const double c2 = dot(c, c), ri = rsqrt64(c2);
                f[h] = sw[g + 4 * (j + h)] * (DL ? fma(q, s1q, s1c) * ri * ri * ri : ri);
                om[h] = k * c2 * ri;
            }
            Cx J[2];
            radial2<1>(om[0], om[1], DL ? c_rad_d1.v : c_rad_s1.v, terms, J, J + 1);
            ar += f[0] * J[0].re + f[1] * J[1].re;
            ai += f[0] * J[0].im + f[1] * J[1].im;
        }
        const double wf = sw[ip] * fw;
        return {wf * ar, wf * ai};
    }
    const V3 P = ld(it.v), A = ld(it.v + 3), B = ld(it.v + 6), C = ld(it.v + 9), D = ld(it.v + 12);
    const int iu = t / kPts, iv = t % kPts;
    const V3 a = fma3(sx[iu], sub(B, A), sub(A, P));
    const V3 b = fma3(sx[iv], sub(D, C), sub(C, P));
    const double an = DL ? dot(a, ld(it.ny)) : 1.0;
    for (int kz = 0; kz < kPts; ++kz) {
        const double z = sx[kz], wz = sw[kz] * z;
        const V3 d1 = fma3(-z, b, a), d2 = fma3(z, a, mul(-1.0, b));
        const double q1 = dot(d1, d1), q2 = dot(d2, d2), r1 = rsqrt64(q1), r2 = rsqrt64(q2);
        Cx g1, g2;
        radial2<1>(k * q1 * r1, k * q2 * r2, DL ? c_rad_d2.v : c_rad_s2.v, terms, &g1, &g2);
        const double f1 = wz * an * (DL ? r1 * r1 * r1 : r1);
        const double f2 = wz * an * (DL ? z * r2 * r2 * r2 : r2);
        ar += f1 * g1.re + f2 * g2.re;
        ai += f1 * g1.im + f2 * g2.im;
    }
    const double wuv = sw[iu] * sw[iv];
    return {wuv * ar, wuv * ai};
}

// Kernel of the remaining integral at the scaled difference c: 1/|c| for
// the single layer, num/|c|^3 for the double layer.
template <int OP>
__device__ __forceinline__ double kern(V3 c, double num)
{
    const double ri = rsqrt64(dot(c, c));
    if constexpr (OP == 0) return ri;
    return num * ri * ri * ri;
}

// This thread's share of the pair integral (without jt js / 4 pi and the
// radial factor, which pair_scale gives); sx, sw hold the 16-point rule.
template <int OP>
__device__ double pair_part(const Pair &it, const double *sx, const double *sw)
{
    const int t = threadIdx.x;
    if (it.kind == 0) {
        if constexpr (OP == 1) return 0.0;
        if (t >= 3 * kIdPts) return 0.0;
        const V3 V0 = ld(it.v), V1 = ld(it.v + 3), V2 = ld(it.v + 6);
        const V3 E1 = sub(V1, V0), E2 = sub(V2, V1);
        const int line = t / kIdPts, k = t - line * kIdPts;
        const double e = (c_x[k % kGL] + (double)(k / kGL)) * (1.0 / kIdPanels);
        const double w = c_w[k % kGL] * (1.0 / kIdPanels);
        const V3 c = line == 0 ? fma3(e, E1, E2) : (line == 1 ? fma3(e, E2, E1) : fma3(-e, E1, mul(1.0 - e, E2)));
        return w * kern<0>(c, 0.0);
    }
    if (it.kind == 1) {
        const V3 P = ld(it.v), Q = ld(it.v + 3), A = ld(it.v + 6), B = ld(it.v + 9);
        const V3 E = sub(Q, P), a = sub(A, P), b = sub(B, P);
        const int face = t >> 6, ip = (t >> 2) & (kPts - 1), g = t & 3;
        const double p = sx[ip], q1 = 1.0 - p;
        // c = c0 + q c1 on the face; s1 = s1c + q s1q is the test side's
        // distance from the edge (the double layer's numerator / (a.n_y))
        V3 c0, c1;
        double s1c, s1q, fw;
        if (face == 0) {          // s2 = 1, s1 = (1 - d) q
            c0 = sub(mul(p, E), b), c1 = mul(q1, a), s1c = 0.0, s1q = q1, fw = q1;
        } else if (face == 1) {   // s1 + d = 1, s2 = q
            c0 = fma3(p, E, mul(q1, a)), c1 = mul(-1.0, b), s1c = q1, s1q = 0.0, fw = 1.0;
        } else if (face == 2) {   // s1 = 1, s2 = (1 - e) q, d = -e
            c0 = fma3(-p, E, a), c1 = mul(-q1, b), s1c = 1.0, s1q = 0.0, fw = q1;
        } else {                  // s2 + e = 1, s1 = q, d = -e
            c0 = fma3(-p, E, mul(-q1, b)), c1 = a, s1c = 0.0, s1q = 1.0, fw = 1.0;
        }
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < kPts / 4; ++j) {
            const double q = sx[g + 4 * j];
            s += sw[g + 4 * j] * kern<OP>(fma3(q, c1, c0), fma(q, s1q, s1c));
        }
        return sw[ip] * fw * s;
    }
    const V3 P = ld(it.v), A = ld(it.v + 3), B = ld(it.v + 6), C = ld(it.v + 9), D = ld(it.v + 12);
    const int iu = t / kPts, iv = t % kPts;
    const V3 a = fma3(sx[iu], sub(B, A), sub(A, P));
    const V3 b = fma3(sx[iv], sub(D, C), sub(C, P));
    const double an = OP == 1 ? dot(a, ld(it.ny)) : 0.0;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kPts; ++k) {
        const double z = sx[k], wz = sw[k] * z;
        s += wz * (kern<OP>(fma3(-z, b, a), an) + (OP == 1 ? z : 1.0) * kern<OP>(fma3(z, a, mul(-1.0, b)), an));
    }
    return sw[iu] * sw[iv] * s;
}

// jt js / 4 pi times the closed-form radial integral of the pair's kind.
template <int OP>
__device__ double pair_scale(const Pair &it)
{
    if constexpr (OP >= 2) {
        const double an = (OP == 3 && it.kind == 1) ? dot(sub(ld(it.v + 6), ld(it.v)), ld(it.ny)) : 1.0;
        return an * it.jt * it.js * kInv4PiD;
    }
    double radial;
    if (it.kind == 0)
        radial = OP == 0 ? 1.0 / 3.0 : 0.0;
    else if (it.kind == 1)
        radial = OP == 0 ? 1.0 / 6.0 : 0.5 * dot(sub(ld(it.v + 6), ld(it.v)), ld(it.ny));
    else
        radial = OP == 0 ? 1.0 / 3.0 : 0.5;
    return radial * it.jt * it.js * kInv4PiD;
}

// Sum of x over the wavefront in a fixed order (butterfly), in every lane.
__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) x += __shfl_xor(x, h);
    return x;
}

// The pair's value, in thread 0: butterfly sums within the wavefronts, then
// the four wavefronts in order (a tree over 256 LDS words took eight barriers
// for what is a few hundred products per thread).
template <int OP>
__device__ Cx pair_value(const Pair &it)
{
    __shared__ double sx[kPts], sw[kPts];
    __shared__ double red[2][kNearThreads / 64];
    const int t = threadIdx.x;
    if (t < kPts) {
        sx[t] = 0.5 * (c_x[t % kGL] + (double)(t / kGL));
        sw[t] = 0.5 * c_w[t % kGL];
    }
    __syncthreads();
    Cx v{0.0, 0.0};
    if constexpr (OP >= 2)
        v = pair_part_helmholtz<OP>(it, sx, sw);
    else
        v.re = pair_part<OP>(it, sx, sw);
    v.re = wave_sum(v.re);
    if constexpr (OP >= 2) v.im = wave_sum(v.im);
    if ((t & 63) == 0) {
        red[0][t >> 6] = v.re;
        red[1][t >> 6] = v.im;
    }
    __syncthreads();
    const double sc = pair_scale<OP>(it);
    return {(red[0][0] + red[0][1] + red[0][2] + red[0][3]) * sc,
            (red[1][0] + red[1][1] + red[1][2] + red[1][3]) * sc};
}

// P0: one workgroup per pair, which is one entry.
template <int OP, bool FP32>
__global__ __launch_bounds__(kNearThreads) void k_near_p0(const NearReq *__restrict__ reqs,
                                                          const NearPair *__restrict__ pairs, int64_t n)
{
    if ((int64_t)blockIdx.x >= n) return;
    const NearPair np = pairs[blockIdx.x];
    const NearReq &R = reqs[np.req];
    const Cx v = pair_value<OP>(load_pair(R, np.a, np.b));
    if (threadIdx.x == 0) {
        constexpr int kParts = OP >= 2 ? 2 : 1;   // complex entries: (re, im)
        if constexpr (FP32) {
            float *o = static_cast<float *>(R.out) + kParts * np.entry;
            o[0] = (float)((double)o[0] + v.re);
            if constexpr (kParts == 2) o[1] = (float)((double)o[1] + v.im);
        } else {
            double *o = static_cast<double *>(R.out) + kParts * np.entry;
            o[0] = o[0] + v.re;
            if constexpr (kParts == 2) o[1] = o[1] + v.im;
        }
    }
}

// ---------------------------------------------------------------------------
// P1 pairs: the 3 x 3 local matrix M[a][b] = int_T lambda_a int_S mu_b K of
// the pair's barycentrics in the item's vertex order (test (V0, V1, V2),
// (P, Q, A), (P, A, B); trial (V0, V1, V2), (P, Q, B), (P, C, D) for the
// identical, common-edge and common-vertex kinds).  Same coordinates and face
// rules as P0.  The barycentrics are affine in the radius, so every point of
// the remaining rule needs the radial integral against 1, rho and rho^2
// (J0, J1, J2: numbers for Laplace, the power series for Helmholtz).  What the
// barycentrics add over the loops a thread runs is polynomial, so the loops
// sum a few moments and the nine entries are formed from them: at the end
// (common vertex: the loop coordinate z enters linearly) or per point from
// averages over the along-edge coordinate (common edge).

// Radial moments of the kernel: Laplace closed forms, 1 / (n + 1) or
// 1 / ((n + 1) (n + 2)).
template <int OP, bool EDGE>
__device__ __forceinline__ void moments(double oa, double ob, int terms, Cx *Ja, Cx *Jb)
{
    constexpr bool DL = OP == 1 || OP == 3;
    if constexpr (OP >= 2) {
        if constexpr (EDGE) radial2<3>(oa, ob, DL ? c_tab_d1.v : c_tab_s1.v, terms, Ja, Jb);
        else radial2<3>(oa, ob, DL ? c_tab_d2.v : c_tab_s2.v, terms, Ja, Jb);
    } else {
        constexpr double n = (EDGE ? 1 : 2) - (DL ? 1 : 0);
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Ja[j] = Jb[j] = {EDGE ? 1.0 / ((n + j + 1) * (n + j + 2)) : 1.0 / (n + j + 1), 0.0};
    }
}

template <int OP>
__device__ __forceinline__ void cfma(Cx &acc, double w, const Cx &x)
{
    acc.re = fma(w, x.re, acc.re);
    if constexpr (OP >= 2) acc.im = fma(w, x.im, acc.im);
}

// This thread's share of the 9 local integrals (row-major; without jt js / 4 pi
// and, for the common-edge double layer, without (a.n_y)).  Op 0, 1: Laplace
// single, double layer; 2, 3: Helmholtz.
template <int OP>
__device__ __forceinline__ void pair_part_p1(const Pair &it, const double *sx, const double *sw, Cx *M)
{
    constexpr bool CPLX = OP >= 2, DL = OP == 1 || OP == 3;
    const int t = threadIdx.x;
    const double k = it.k;
    int terms = 0;
    if constexpr (CPLX) terms = series_terms(it);
    if (it.kind == 0) {
        if constexpr (DL) return;
        const V3 V0 = ld(it.v), V1 = ld(it.v + 3), V2 = ld(it.v + 6);
        const V3 E1 = sub(V1, V0), E2 = sub(V2, V1);
        // |c| on line `line` at eta3 = e3
        auto length2 = [&](int line, double e3) {
            const V3 c = line == 0 ? fma3(e3, E1, E2) : (line == 1 ? fma3(e3, E2, E1) : fma3(-e3, E1, mul(1.0 - e3, E2)));
            return dot(c, c);
        };
        // adds the node (line, e1, e2, e3), region and mirror (x and y exchanged: symmetric)
        auto node = [&](int line, double e1, double e2, double e3, double w, const Cx *J) {
            // x = xi (A1, B1), y = xi (A2, B2) in the (a, b) coordinates, barycentrics (1 - a, a - b, b)
            double A1, B1, A2, B2;
            if (line == 0) {
                A1 = 1.0, B1 = 1.0 - e1 + e1 * e2, A2 = 1.0 - e1 * e2 * e3, B2 = 1.0 - e1;
            } else if (line == 1) {
                A1 = 1.0, B1 = e1 * (1.0 - e2 + e2 * e3), A2 = 1.0 - e1 * e2, B2 = e1 * (1.0 - e2);
            } else {
                A1 = 1.0 - e1 * e2 * e3, B1 = e1 * (1.0 - e2 * e3), A2 = 1.0, B2 = e1 * (1.0 - e2);
            }
            const double x[3] = {-A1, A1 - B1, B1}, y[3] = {-A2, A2 - B2, B2};
            cfma<OP>(M[0], 2.0 * w, J[0]);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                cfma<OP>(M[a], (a == 0 ? 2.0 : 1.0) * w * (x[a] + y[a]), J[1]);
#pragma unroll
                for (int b = a; b < 3; ++b) cfma<OP>(M[3 * a + b], w * fma(x[a], y[b], x[b] * y[a]), J[2]);
            }
        };
        if constexpr (CPLX) {
            // Thread t takes the point (eta1, eta2) of the 8 x 8 rule and every
            // fourth (line, eta3) node, two at a time: a wavefront shares its
            // line.  Beyond omega = 3.2 e^{i omega eta1 eta2} needs two panels per
            // direction (one left 7e-8 at omega = 11).
            const int panels = terms > 32 ? 2 : 1;
            const double sc = 1.0 / panels;
#pragma unroll 1
            for (int pp = 0; pp < panels * panels; ++pp) {
                const double e1 = (c_x[(t >> 3) & 7] + (pp >> 1)) * sc, e2 = (c_x[t & 7] + (pp & 1)) * sc;
                const double w12 = c_w[(t >> 3) & 7] * c_w[t & 7] * e1 * sc * sc;
#pragma unroll 1
                for (int i = 0; i < 3 * kIdPts / 8; ++i) {
                    double om[2], e3[2], w[2];
                    int line = 0;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {   // four nodes apart, on one line
                        const int n = (t >> 6) + 4 * (2 * i + h);
                        line = n / kIdPts;
                        const int kk = n - line * kIdPts;
                        e3[h] = (c_x[kk % kGL] + (double)(kk / kGL)) * (1.0 / kIdPanels);
                        const double c2 = length2(line, e3[h]), ic = rsqrt64(c2);
                        om[h] = k * c2 * ic * e1 * e2;
                        w[h] = w12 * c_w[kk % kGL] * (1.0 / kIdPanels) * ic;
                    }
                    Cx J[2][3];
                    moments<OP, false>(om[0], om[1], terms, J[0], J[1]);
                    node(line, e1, e2, e3[0], w[0], J[0]);
                    node(line, e1, e2, e3[1], w[1], J[1]);
                }
            }
        } else {
            // polynomial in eta1, eta2 too (degrees 3 and 2): 2 x 2 points times
            // the (line, eta3) nodes, spread over the threads
            constexpr double g2x[2] = {0.5 - 0.28867513459481288225, 0.5 + 0.28867513459481288225};
            Cx J[3], unused[3];
            moments<OP, false>(0.0, 0.0, 0, J, unused);
            for (int n = t; n < 4 * 3 * kIdPts; n += kNearThreads) {
                const int q = n / (3 * kIdPts), lk = n - q * (3 * kIdPts), line = lk / kIdPts, kk = lk - line * kIdPts;
                const double e1 = g2x[q >> 1], e2 = g2x[q & 1];
                const double e3 = (c_x[kk % kGL] + (double)(kk / kGL)) * (1.0 / kIdPanels);
                node(line, e1, e2, e3, 0.25 * e1 * c_w[kk % kGL] * (1.0 / kIdPanels) * rsqrt64(length2(line, e3)), J);
            }
        }
        M[3] = M[1];
        M[6] = M[2];
        M[7] = M[5];
        return;
    }
    if (it.kind == 1) {
        const V3 P = ld(it.v), Q = ld(it.v + 3), A = ld(it.v + 6), B = ld(it.v + 9);
        const V3 E = sub(Q, P), a = sub(A, P), b = sub(B, P);
        const int face = t >> 6, ip = (t >> 2) & (kPts - 1), g = t & 3;
        const bool ahead = face < 2, odd = face & 1;   // faces 0, 1: the test point ahead along the edge
        const double p = sx[ip], q1 = 1.0 - p;
#pragma unroll 1
        for (int j = 0; j < kPts / 4; j += 2) {
            double dh[2], s1[2], s2[2], K[2], om[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // (dh, s1, s2): face 0 (p, q1 q, 1), 1 (p, q1, q), 2 (-p, 1, q1 q), 3 (-p, q, q1)
                const double q = sx[g + 4 * (j + h)];
                const double X = odd ? q1 : q1 * q, Y = odd ? q : 1.0, fw = odd ? 1.0 : q1;
                dh[h] = ahead ? p : -p;
                s1[h] = ahead ? X : Y;
                s2[h] = ahead ? Y : X;
                const V3 c = fma3(dh[h], E, fma3(s1[h], a, mul(-s2[h], b)));
                const double c2 = dot(c, c), ic = rsqrt64(c2);
                K[h] = sw[ip] * sw[g + 4 * (j + h)] * fw * (DL ? s1[h] * ic * ic * ic : ic);
                om[h] = k * c2 * ic;
            }
            Cx J[2][3];
            moments<OP, true>(om[0], om[1], terms, J[0], J[1]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // With tau in [0, 1] along the edge the barycentrics are
                // (1 - tau, tau, 0) + rho be(tau) on the test side and
                // (1 - tau, tau, 0) + rho de(tau) on the trial side, be =
                // (tau - bx - s1, bx - tau, s1), de = (tau - dx - s2, dx - tau,
                // s2), where faces 0, 1 (x ahead along the edge) have bx = dh,
                // dx = 0 and faces 2, 3 bx = 0, dx = -dh.  Below, the averages
                // over tau of their products (<tau> = 1/2, <tau^2> = 1/3).
                const double bx = ahead ? dh[h] : 0.0, dx = ahead ? 0.0 : -dh[h];
                const double be[3] = {-bx - s1[h], bx, s1[h]}, de[3] = {-dx - s2[h], dx, s2[h]};   // at tau = 0
                constexpr double sl[3] = {1.0, -1.0, 0.0};                     // slopes in tau
                constexpr double a0[3] = {0.5, 0.5, 0.0}, a1[3] = {1.0 / 6.0, 1.0 / 3.0, 0.0};   // <al>, <tau al>
                constexpr double aa[3][3] = {{1.0 / 3.0, 1.0 / 6.0, 0.0}, {1.0 / 6.0, 1.0 / 3.0, 0.0}, {0.0, 0.0, 0.0}};
                Cx k0{K[h] * J[h][0].re, K[h] * J[h][0].im}, k1{K[h] * J[h][1].re, K[h] * J[h][1].im},
                    k2{K[h] * J[h][2].re, K[h] * J[h][2].im};
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        Cx &m = M[3 * r + s];
                        if (r < 2 && s < 2) cfma<OP>(m, aa[r][s], k0);
                        cfma<OP>(m, fma(a0[r], de[s], a1[r] * sl[s]) + fma(a0[s], be[r], a1[s] * sl[r]), k1);
                        cfma<OP>(m, fma(be[r], de[s], 0.5 * fma(be[r], sl[s], de[s] * sl[r])) + sl[r] * sl[s] * (1.0 / 3.0), k2);
                    }
            }
        }
        return;
    }
    const V3 P = ld(it.v), A = ld(it.v + 3), B = ld(it.v + 6), C = ld(it.v + 9), D = ld(it.v + 12);
    const int iu = t / kPts, iv = t % kPts;
    const double u = sx[iu], v = sx[iv];
    const V3 av = fma3(u, sub(B, A), sub(A, P));
    const V3 bv = fma3(v, sub(D, C), sub(C, P));
    const double an = DL ? dot(av, ld(it.ny)) : 1.0;
    const double wuv = sw[iu] * sw[iv];
    // x = P + s a(u), y = P + s z b(v) and x = P + s z a(u), y = P + s b(v):
    // barycentrics e0 + s X, e0 + s z Y (resp. z on X), X = (-1, 1 - u, u), Y =
    // (-1, 1 - v, v).  Sums over z of the coefficients of e0 e0, X e0, e0 Y, X Y.
    Cx S0{0.0, 0.0}, Sx{0.0, 0.0}, Sy{0.0, 0.0}, Sxy{0.0, 0.0};
#pragma unroll 1
    for (int kz = 0; kz < kPts; ++kz) {
        const double z = sx[kz];
        const V3 c1 = fma3(-z, bv, av), c2 = fma3(z, av, mul(-1.0, bv));
        const double q1 = dot(c1, c1), q2 = dot(c2, c2), i1 = rsqrt64(q1), i2 = rsqrt64(q2);
        const double f = wuv * sw[kz] * z * an;
        const double k1 = f * (DL ? i1 * i1 * i1 : i1), k2 = f * (DL ? z * i2 * i2 * i2 : i2);
        Cx J[3], H[3];
        moments<OP, false>(k * q1 * i1, k * q2 * i2, terms, J, H);
        cfma<OP>(S0, k1, J[0]);
        cfma<OP>(S0, k2, H[0]);
        cfma<OP>(Sx, k1, J[1]);
        cfma<OP>(Sx, k2 * z, H[1]);
        cfma<OP>(Sy, k1 * z, J[1]);
        cfma<OP>(Sy, k2, H[1]);
        cfma<OP>(Sxy, k1 * z, J[2]);
        cfma<OP>(Sxy, k2 * z, H[2]);
    }
    const double X[3] = {-1.0, 1.0 - u, u}, Y[3] = {-1.0, 1.0 - v, v};
    M[0] = S0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cfma<OP>(M[3 * a], X[a], Sx);
        cfma<OP>(M[a], Y[a], Sy);
#pragma unroll
        for (int b = 0; b < 3; ++b) cfma<OP>(M[3 * a + b], X[a] * Y[b], Sxy);
    }
}

// One workgroup per pair: its 3 x 3 local matrix in the triangles' own vertex
// orders (row-major test x trial, complex (re, im)) into local[pair], and the
// column dofs of its column-side triangle into keys[pair].  The 9 (18: complex)
// sums over 256 threads go through LDS once: eight threads per value add 32
// partials each, a butterfly adds the eight (fixed order, two barriers; a tree
// over all values took eight).
// HYP: the hypersingular operator (Eq. hypsHelmholtz), from the single layer's
// matrix M: curl_a . curl_b times the pair's P0 value, which is the sum of M
// (the hat functions sum to one), minus k^2 n_x . n_y M.
template <int OP, bool HYP>
__global__ __launch_bounds__(kNearThreads, OP >= 2 ? 4 : 5) void k_near_p1(const NearReq *__restrict__ reqs,
                                                          const NearPair *__restrict__ pairs, int64_t n,
                                                          int4 *__restrict__ keys, double *__restrict__ local)
{
    constexpr int NV = OP >= 2 ? 18 : 9, NR = NV / 9;
    if ((int64_t)blockIdx.x >= n) return;
    const NearPair np = pairs[blockIdx.x];
    const NearReq &R = reqs[np.req];
    const Pair it = load_pair(R, np.a, np.b);
    __shared__ double sx[kPts], sw[kPts];
    __shared__ double red[NV][kNearThreads + 8];   // rows 8 words of 64 bits apart from a multiple of the banks
    const int t = threadIdx.x;
    if (t < kPts) {
        sx[t] = 0.5 * (c_x[t % kGL] + (double)(t / kGL));
        sw[t] = 0.5 * c_w[t % kGL];
    }
    __syncthreads();
    Cx M[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) M[i] = {0.0, 0.0};
    pair_part_p1<OP>(it, sx, sw, M);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        red[NR * i][t] = M[i].re;
        if constexpr (OP >= 2) red[2 * i + 1][t] = M[i].im;
    }
    __syncthreads();
    const int e = (t >> 3) / NR, part = (t >> 3) % NR;   // entry in the order of v, (re, im)
    double s = 0.0;
    if (t < 8 * NV) {
        const double *r = red[t >> 3] + (t & 7);
#pragma unroll 8
        for (int i = 0; i < kNearThreads / 8; ++i) s += r[8 * i];
#pragma unroll
        for (int h = 4; h > 0; h >>= 1) s += __shfl_xor(s, h);
        const double an = ((OP == 1 || OP == 3) && it.kind == 1) ? dot(sub(ld(it.v + 6), ld(it.v)), ld(it.ny)) : 1.0;
        s *= an * it.jt * it.js * kInv4PiD;
    }
    if (t < 8 * NV && (t & 7) == 0) {
        if constexpr (HYP) red[t >> 3][0] = s;
    }
    if constexpr (HYP) __syncthreads();
    if (t < 8 * NV && (t & 7) == 0) {
        const int i = e / 3, j = e - 3 * i;
        const int tl = i == 0 ? it.pt[0] : (i == 1 ? it.pt[1] : it.pt[2]);
        const int sl = j == 0 ? it.ps[0] : (j == 1 ? it.ps[1] : it.ps[2]);
        if constexpr (HYP) {
            double p0 = 0.0;
#pragma unroll
            for (int x = 0; x < 9; ++x) p0 += red[NR * x + part][0];
            // surface curl of local vertex i: (v_{i+1} - v_{i+2}) / J in the mesh's order
            const int4 tv = R.vtx[it.T], sv = R.vtx[it.S];
            auto id = [](const int4 &v, int x) { return x == 0 ? v.x : (x == 1 ? v.y : v.z); };
            auto edge = [&](const int4 &v, int x) {
                return sub(ld(R.xyz + 3 * (size_t)id(v, (x + 1) % 3)), ld(R.xyz + 3 * (size_t)id(v, (x + 2) % 3)));
            };
            const double cc = dot(edge(tv, tl), edge(sv, sl)) / (it.jt * it.js);
            const double nn = dot(ld(it.nt), ld(it.ny));
            s = cc * p0 - it.k * it.k * nn * s;
        }
        local[(size_t)NV * blockIdx.x + NR * (3 * tl + sl) + part] = s;
    }
    if (t == 0) {
        int4 kv = R.vtx[np.b];
        if (R.dp1) kv = make_int4(3 * np.b, 3 * np.b + 1, 3 * np.b + 2, 0);
        keys[blockIdx.x] = kv;
    }
}

// Adds the local matrices to the entries: one workgroup per row and 256
// columns, one thread per entry.  The row's pairs (about 80: six triangles
// with 13 neighbours each) and their matrices are gathered in LDS, and every
// thread then adds those whose column-side triangle has its dof, in the order
// of the row's star and of each triangle's list.  Entries without a pair are
// not touched.  Bound by latency, not by its few bytes: with the matrices read
// where they are added (a wait per pair) it took 30 us on a 100 x 100 leaf, from
// LDS 9.9 us.
constexpr int kGatherPairs = 128;   // pairs in LDS at a time

template <bool FP32, bool CPLX>
__global__ __launch_bounds__(256) void k_near_gather(const NearReq *__restrict__ reqs,
                                                     const NearBlock *__restrict__ blocks,
                                                     const int4 *__restrict__ keys, const double *__restrict__ local)
{
    constexpr int NR = CPLX ? 2 : 1;
    __shared__ int4 star[256];                        // per star triangle: first pair, pairs, local vertex
    __shared__ int4 list[kGatherPairs];               // column dofs of a pair's three vertices, its vertex of the row
    __shared__ int pair[kGatherPairs];
    __shared__ double val[kGatherPairs * 9 * NR];
    const NearBlock B = blocks[blockIdx.x];
    const NearReq &R = reqs[B.req];
    const int t = threadIdx.x;
    const int c = B.col0 + t;
    const int key = c < R.ncols ? R.cols[c] : -1;
    const int step = R.transposed ? 3 : 1;   // the row-side triangle's vertex is the second index
    const int lead = R.transposed ? 1 : 3;
    const int e0 = R.rptr[B.row], ne = R.rptr[B.row + 1] - e0;   // at most 256 triangles around a vertex
    if (t < ne) {
        const int pk = R.rs[e0 + t], p0 = R.gptr[pk >> 2];
        star[t] = make_int4(p0, R.gptr[(pk >> 2) + 1] - p0, pk & 3, 0);
    }
    __syncthreads();
    double sr = 0.0, si = 0.0;
    bool any = false;
    for (int first = 0;; first += kGatherPairs) {
        // entry first + t of the row's list
        int at = first + t, total = 0, p = -1, i = 0;
        for (int e = 0; e < ne; ++e) {
            const int4 s = star[e];
            if (p < 0 && at < total + s.y) {
                p = s.x + at - total;
                i = s.z;
            }
            total += s.y;
        }
        const int count = min(kGatherPairs, total - first);
        if (t < count) {
            int4 kv = keys[p];
            kv.w = 9 * t + lead * i;
            list[t] = kv;
            pair[t] = p;
        }
        __syncthreads();
        for (int x = t; x < count * 9 * NR; x += 256) {
            const int q = x / (9 * NR);
            val[x] = local[(size_t)(9 * NR) * pair[q] + (x - q * (9 * NR))];
        }
        __syncthreads();
#pragma unroll 4
        for (int x = 0; x < count; ++x) {
            const int4 kv = list[x];
            const bool m0 = key == kv.x, m1 = key == kv.y, m2 = key == kv.z, m = m0 || m1 || m2;
            const int at = NR * (kv.w + (m1 ? step : (m2 ? 2 * step : 0)));
            const double vr = val[at];
            sr += m ? vr : 0.0;
            if constexpr (CPLX) {
                const double vi = val[at + 1];
                si += m ? vi : 0.0;
            }
            any = any || m;
        }
        if (first + kGatherPairs >= total) break;
        __syncthreads();   // the list has been read
    }
    if (!any) return;
    const int64_t o = (int64_t)B.row * R.ncols + c;
    if constexpr (FP32) {
        float *w = static_cast<float *>(R.out) + NR * o;
        w[0] = (float)((double)w[0] + sr);
        if constexpr (CPLX) w[1] = (float)((double)w[1] + si);
    } else {
        double *w = static_cast<double *>(R.out) + NR * o;
        w[0] += sr;
        if constexpr (CPLX) w[1] += si;
    }
}

template <int OP, bool HYP>
void launch_p1(const NearLayout &L, const NearCount &n, char *dev, hipStream_t s)
{
    hipLaunchKernelGGL((k_near_p1<OP, HYP>), dim3((unsigned)n.pairs), dim3(kNearThreads), 0, s,
                       reinterpret_cast<const NearReq *>(dev), reinterpret_cast<const NearPair *>(dev + L.pairs),
                       n.pairs, reinterpret_cast<int4 *>(dev + L.keys), reinterpret_cast<double *>(dev + L.local));
}

template <int OP>
void launch_p0(bool fp32, const NearLayout &L, const NearCount &n, char *dev, hipStream_t s)
{
    const NearReq *reqs = reinterpret_cast<const NearReq *>(dev);
    const NearPair *pairs = reinterpret_cast<const NearPair *>(dev + L.pairs);
    const dim3 grid((unsigned)n.pairs), block(kNearThreads);
    if (fp32)
        hipLaunchKernelGGL((k_near_p0<OP, true>), grid, block, 0, s, reqs, pairs, n.pairs);
    else
        hipLaunchKernelGGL((k_near_p0<OP, false>), grid, block, 0, s, reqs, pairs, n.pairs);
}

template <bool FP32, bool CPLX>
void launch_gather_p1(const NearLayout &L, const NearCount &n, char *dev, hipStream_t s)
{
    hipLaunchKernelGGL((k_near_gather<FP32, CPLX>), dim3((unsigned)n.blocks), dim3(256), 0, s,
                       reinterpret_cast<const NearReq *>(dev), reinterpret_cast<const NearBlock *>(dev + L.blocks),
                       reinterpret_cast<const int4 *>(dev + L.keys), reinterpret_cast<const double *>(dev + L.local));
}

}  // namespace

hipError_t launch_near(int kind, const NearLayout &L, const NearCount &n, char *dev, hipStream_t s)
{
    if (n.pairs <= 0) return hipSuccess;
    if (n.pairs > INT32_MAX / 9 || n.blocks > INT32_MAX || kind < 0 || kind >= kNearKinds) return hipErrorInvalidValue;
    const bool fp32 = kind & 1;
    bool cplx = false;
    switch (kind >> 1) {
    case 0: launch_p0<0>(fp32, L, n, dev, s); break;
    case 1: launch_p0<1>(fp32, L, n, dev, s); break;
    case 2: launch_p0<2>(fp32, L, n, dev, s); break;
    case 3: launch_p0<3>(fp32, L, n, dev, s); break;
    case 4: launch_p1<0, false>(L, n, dev, s); break;
    case 5: launch_p1<1, false>(L, n, dev, s); break;
    case 6: launch_p1<2, false>(L, n, dev, s); cplx = true; break;
    case 7: launch_p1<3, false>(L, n, dev, s); cplx = true; break;
    case 8: launch_p1<0, true>(L, n, dev, s); break;
    default: launch_p1<2, true>(L, n, dev, s); cplx = true; break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n.blocks == 0) return e;
    if (fp32 && cplx) launch_gather_p1<true, true>(L, n, dev, s);
    else if (fp32) launch_gather_p1<true, false>(L, n, dev, s);
    else if (cplx) launch_gather_p1<false, true>(L, n, dev, s);
    else launch_gather_p1<false, false>(L, n, dev, s);
    return hipGetLastError();
}

}  // namespace bem
