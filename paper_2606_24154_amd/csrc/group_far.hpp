// group_far.hpp -- far field of a group of elements by its multipole
// expansion, FP64 (device code shared by the moment and evaluation kernels).
//
// A group is up to 64 consecutive elements.  Far enough from it, the sum of
// its elements' potentials and fields is evaluated as one expansion about
// the group's centre c (the centre of its vertices' box) instead of element by
// element.  With a the largest vertex distance from c, d = P - c - t for a
// copy translated by t, r = |d| and u = d/r:
//   E   = r^-2 sum_{L=1}^{p+1} (a/r)^(L-1) S_L(u),   S_L a vector harmonic of degree L
//   phi = r^-1 sum_L (a/r)^(L-1) (S_L . u) / L
// (the degree-n term of the potential is -r.grad/(n+1) of itself, so the
// field's terms give the potential).  Each component of S_L is
//   sum_{m=0}^{L} Re(conj(C_{L,m}) J_L^m(u)),
//   J_L^m = lam_{L,m} P_L^(m)(u_z) (u_x + i u_y)^m,
// P_L^(m) the m-th derivative of the Legendre polynomial, with lam chosen so
// that the recurrence in L has one constant:
//   J_m^m = (u_x + i u_y)^m, J_{m+1}^m = u_z J_m^m,
//   J_{n+1}^m = c_{n,m} u_z J_n^m - J_{n-1}^m.
// The coefficients C come from the group's moments
//   B_{n,m} = (2 - [m=0]) (n-m)!/(n+m)! / lam_{n,m} sum q (s/a)^n J_n^m(s/|s|)
// through the derivatives of the irregular harmonics I_n^m (same indices,
// r^-(n+1) scaling): d_z I_n^m = -(n-m+1) I_{n+1}^m, (d_x + i d_y) I_n^m =
// -I_{n+1}^{m+1}, (d_x - i d_y) I_n^m = (n-m+1)(n-m+2) I_{n+1}^{m-1}.
//
// The truncation after degree p is at most ~(p+2) (a/r)^(p+1) of
// sum |q| / r^2; tier_ratio2 gives the (r/a)^2 from which a degree keeps that
// bound below 3e-12.  On meshes it comes out 10 to 100 times smaller at the
// threshold itself, below the closed forms' own rounding (1e-11 of an element's
// field beyond 25 diameters), and it falls with (a/r)^(p+1).  Errors against 64-bit
// sums (closed forms near, Gauss rules far) over field-map points and, a third, points
// in the GEM's hole, GEM cells of 1648 x 121, 2960 x 49, 8064 x 121 and 8064 x 9 copies,
// THGEM of 5792 x 49 and 41 600 x 121: of E, in the 2-norm over the points, 1.1, 1.2, 1.7,
// 2.1, 1.4, 1.8e-15 (closed forms throughout 1.3, 2.4, 1.9, 3.7, 2.1, 1.8e-15), of phi
// 0.7, 1.2, 1.1, 4.0, 0.5, 0.7e-15 (2.6, 5.8, 2.6, 11, 1.2, 0.9e-15); largest pointwise
// of E 1e-14 .. 1e-13 both.  With a bound of 1e-12 E's are 1.0, 1.2, 1.8, 2.0, 1.4,
// 1.8e-15 and calls take 4 to 7 % longer; with 1e-11 2.7, 1.3, 1.8, 2.2, 1.8, 1.9e-15,
// on the first mesh twice the closed forms'.
#pragma once
#include <hip/hip_runtime.h>

#include "nebem_internal.hpp"

namespace nebem {

constexpr int kGroupP = 14;           // highest degree of the potential's expansion
constexpr int kGroupL = kGroupP + 1;  // highest degree of the field's
// Record of a group: centre, a, the squared distances from which the degrees
// 14, 12, 10, 8, 6, 4 apply; then one entry of 8 doubles (one scalar load) per
// harmonic (L, m), L = 1 .. kGroupL, m = 0 .. L: the coefficient C of Ex, Ey, Ez
// (real and imaginary parts), the recurrence constant c_{L-1,m} and a pad.  The
// harmonics are taken in two passes, orders m < kOrderSplit first: a pass keeps
// the last two degrees of its own orders only, which brings the working set of
// degree 15 (16 orders) from 180 registers to the ~120 of degree 7.
constexpr int kGroupHead = 16;
constexpr int kHeadTier = 4;  // index of the first threshold
constexpr int kTiers = 6;
constexpr int kHeadSuper = 10;  // the parent's centre and far threshold (none: NaN, no point is far)
constexpr int kHeadDiffer = 14;  // of a group, column 0: not 0 if the columns' thresholds differ
constexpr int kEntry = 8;
constexpr int kOrderSplit = 8;
// entries of the degrees below L in the first and in the second pass
__host__ __device__ constexpr int pass1_entries(int L)
{
    int e = 0;
    for (int n = 1; n < L; ++n) e += n + 1 < kOrderSplit ? n + 1 : kOrderSplit;
    return e;
}
__host__ __device__ constexpr int pass2_entries(int L)
{
    int e = 0;
    for (int n = kOrderSplit; n < L; ++n) e += n - kOrderSplit + 1;
    return e;
}
constexpr int kPass2 = pass1_entries(kGroupL + 1);
constexpr int kGroupEntries = kPass2 + pass2_entries(kGroupL + 1);
__host__ __device__ constexpr int entry_index(int L, int m)
{
    return m < kOrderSplit ? pass1_entries(L) + m : kPass2 + pass2_entries(L) + m - kOrderSplit;
}
constexpr int kGroupStride = kGroupHead + kEntry * kGroupEntries;

// squares of r/a = ((p + 2) / 3e-12)^(1/(p + 1)) for p = 14, 12, 10, 8, 6, 4
__host__ __device__ constexpr double tier_ratio2(int k)
{
    return k == 0 ? 49.77 : k == 1 ? 88.94 : k == 2 ? 195.6 : k == 3 ? 606.6 : k == 4 ? 3551.0 : 83260.0;
}

struct HarmonicTables {
    double lam[kGroupL + 1][kGroupL + 1];  // lam_{n,m}
    double c[kGroupL + 1][kGroupL + 1];    // c_{n,m} of the step n -> n + 1
    double bf[kGroupL + 1][kGroupL + 1];   // (2 - [m=0]) (n-m)!/(n+m)! / lam_{n,m}
};

constexpr HarmonicTables make_harmonic_tables()
{
    HarmonicTables t{};
    double df = 1.0;  // (2m - 1)!!
    for (int m = 0; m <= kGroupL; ++m) {
        if (m > 0) df *= 2.0 * m - 1.0;
        t.lam[m][m] = 1.0 / df;
        if (m + 1 <= kGroupL) t.lam[m + 1][m] = 1.0 / ((2.0 * m + 1.0) * df);
        for (int n = m + 1; n < kGroupL; ++n) {
            t.lam[n + 1][m] = t.lam[n - 1][m] * (n + 1 - m) / (n + m);
            t.c[n][m] = (2.0 * n + 1.0) * t.lam[n + 1][m] / ((n + 1 - m) * t.lam[n][m]);
        }
        for (int n = m; n <= kGroupL; ++n) {
            double f = m == 0 ? 1.0 : 2.0;
            for (int k = n - m + 1; k <= n + m; ++k) f /= k;
            t.bf[n][m] = f / t.lam[n][m];
        }
    }
    return t;
}
inline constexpr HarmonicTables kHarm = make_harmonic_tables();

// Uniform reads of data that no kernel in flight writes: the constant
// address space makes them scalar loads.
typedef const __attribute__((address_space(4))) double *cdouble_p;
typedef double d8 __attribute__((ext_vector_type(8), aligned(8)));  // scalar loads need no more, nor do its users
static_assert(alignof(d8) == alignof(double), "group records start at any double");
typedef const __attribute__((address_space(4))) d8 *cd8_p;
__device__ __forceinline__ cdouble_p uniform_ptr(const double *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (cdouble_p)(((uint64_t)hi << 32) | lo);
}

// The same address, opaque to the optimiser: reads through it stay inside the
// loop that takes it (hoisted out, a few hundred loop-invariant coefficients
// would be spilled).
__device__ __forceinline__ cdouble_p in_loop(cdouble_p p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// Offset of a point from the group's centre for copy (i1, i2) of one
// reflection, and its square.  Every kernel that decides near or far calls
// these, so that all of them take the same decision from the same bits.
struct GroupVec {
    double x, y, z;
};
__device__ __forceinline__ GroupVec group_origin(const ImgArgs &img, int ax, double Px, double Py, double Pz,
                                                 cdouble_p head)
{
#pragma clang fp contract(off)
    const double Qx = (ax & 1) ? 2.0 * img.mpos[0] - Px : Px;
    const double Qy = (ax & 2) ? 2.0 * img.mpos[1] - Py : Py;
    const double Qz = (ax & 4) ? 2.0 * img.mpos[2] - Pz : Pz;
    return {Qx - head[0], Qy - head[1], Qz - head[2]};
}
__device__ __forceinline__ GroupVec group_step(const GroupVec &v, double f, const double *a)
{
    return {fma(f, a[0], v.x), fma(f, a[1], v.y), fma(f, a[2], v.z)};
}
__device__ __forceinline__ double group_r2(const GroupVec &d) { return fma(d.x, d.x, fma(d.y, d.y, d.z * d.z)); }

// Whether a copy is far from the group's parent, whose expansion (or whose own
// parent's) then serves it.
__device__ __forceinline__ bool super_far(const ImgArgs &img, int r, int i1, int i2, double Px, double Py, double Pz,
                                          cdouble_p head)
{
    const GroupVec v0 = group_origin(img, img.axes[r], Px, Py, Pz, head + kHeadSuper);
    const GroupVec d = group_step(group_step(v0, -(double)i1, img.a1[r]), -(double)i2, img.a2[r]);
    return group_r2(d) >= head[kHeadSuper + 3];
}

// The expansion through degree L of the field (entries at coef), added to
// acc = (phi, Ex, Ey, Ez).  The entries run through two buffers of kAhead
// scalar loads: the wait for a buffer comes before the next one's loads are
// issued (scalar loads return out of order, so a wait takes all of them), and
// those then have kAhead entries' arithmetic to arrive in.  The empty asm
// statements and scheduling barriers keep one entry's harmonics next to its
// products: left alone, the compiler computes every harmonic first and spills
// them.
constexpr int kAhead = 2;

template <int L>
__device__ __forceinline__ void group_far(const GroupVec &d, double r2, double a, cdouble_p coef, double (&acc)[4])
{
#pragma clang fp contract(off)
    constexpr int kFirst = pass1_entries(L + 1), kEnd = kFirst + pass2_entries(L + 1);
    // 1/r: estimate (5e-8) with the two leading terms of its correction, error below 1e-16
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y), y, 1.0);
    const double ir = fma(y * e, fma(e, 0.375, 0.5), y);
    const double ux = d.x * ir, uy = d.y * ir, uz = d.z * ir;
    const double rho = a * ir;
    double p, ex, ey, ez;
    d8 buf[2][kAhead];
    auto fetch = [&](int u0) {
        coef = in_loop(coef);  // keeps the loads at their place
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
            if (u0 + q < kEnd) {
                const int at = u0 + q < kFirst ? u0 + q : u0 + q - kFirst + kPass2;
                buf[(u0 / kAhead) & 1][q] = *(cd8_p)(coef + kEntry * at);
            }
    };
    fetch(0);
    double w = 1.0, wsplit = 1.0;  // rho^(n-1); where the second pass starts
    double dr = 1.0, di = 0.0;     // the last J_m^m
    int u = 0;
#pragma unroll
    for (int pass = 0; pass < (L >= kOrderSplit ? 2 : 1); ++pass) {
        const int mlo = pass ? kOrderSplit : 0;
        double re[2][kOrderSplit], im[2][kOrderSplit];  // J of the last two degrees, this pass's orders
        if (pass) w = wsplit;
#pragma unroll
        for (int n = pass ? kOrderSplit : 1; n <= L; ++n) {
            const int cur = n & 1, prv = cur ^ 1;
            const int mhi = pass ? n : (n < kOrderSplit ? n : kOrderSplit - 1);
            if (!pass && n == kOrderSplit) wsplit = w;
            double sx, sy, sz;
#pragma unroll
            for (int m = mlo; m <= mhi; ++m, ++u) {
                const int i = m - mlo;
                if (u % kAhead == 0) {
                    // everything so far is computed, this buffer has arrived
                    if (m > mlo) asm volatile("" : "+v"(sx), "+v"(sy), "+v"(sz));
                    if (m == mlo && n > 1) asm volatile("" : "+v"(ex), "+v"(ey), "+v"(ez), "+v"(p));
                    asm volatile("" ::"s"(buf[(u / kAhead) & 1][0]));
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(u + kAhead);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const d8 c = buf[(u / kAhead) & 1][u % kAhead];
                if (m == n) {
                    const double tr = n == 1 ? ux : fma(dr, ux, -(di * uy));
                    di = n == 1 ? uy : fma(dr, uy, di * ux);
                    dr = tr;
                    re[cur][i] = dr;
                    im[cur][i] = di;
                } else if (m == n - 1) {
                    re[cur][i] = m == 0 ? uz : uz * re[prv][i];
                    im[cur][i] = m == 0 ? 0.0 : uz * im[prv][i];
                } else {
                    const double t = c[6] * uz;
                    re[cur][i] = fma(t, re[prv][i], n == 2 && m == 0 ? -1.0 : -re[cur][i]);
                    if (m > 0) im[cur][i] = fma(t, im[prv][i], -im[cur][i]);
                }
                if (m == mlo) {
                    sx = m == 0 ? c[0] * re[cur][i] : fma(c[0], re[cur][i], c[1] * im[cur][i]);
                    sy = m == 0 ? c[2] * re[cur][i] : fma(c[2], re[cur][i], c[3] * im[cur][i]);
                    sz = m == 0 ? c[4] * re[cur][i] : fma(c[4], re[cur][i], c[5] * im[cur][i]);
                } else {
                    sx = fma(c[0], re[cur][i], fma(c[1], im[cur][i], sx));
                    sy = fma(c[2], re[cur][i], fma(c[3], im[cur][i], sy));
                    sz = fma(c[4], re[cur][i], fma(c[5], im[cur][i], sz));
                }
            }
            const double su = fma(sx, ux, fma(sy, uy, sz * uz));
            p = n == 1 ? su : fma(w * (1.0 / n), su, p);
            ex = n == 1 ? sx : fma(w, sx, ex);
            ey = n == 1 ? sy : fma(w, sy, ey);
            ez = n == 1 ? sz : fma(w, sz, ez);
            w = n == 1 ? rho : w * rho;
        }
    }
    const double ir2 = ir * ir;
    acc[0] = fma(ir, p, acc[0]);
    acc[1] = fma(ir2, ex, acc[1]);
    acc[2] = fma(ir2, ey, acc[2]);
    acc[3] = fma(ir2, ez, acc[3]);
}

}  // namespace nebem
