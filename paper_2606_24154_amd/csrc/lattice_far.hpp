// lattice_far.hpp -- far copies of a group of elements in the assembly, FP64:
// the irregular harmonics of the offsets summed over the lattice (device code of
// k_assemble_grouped; indices, normalisation and thresholds as in group_far.hpp).
//
// The far copies' share of the matrix entries of one row and one group's 64
// elements is, with t = a/r,
//   kKe/a   sum_{n,m} Re(conj(b_{n,m}) F_n^m),    F_n^m = sum_copies t^(n+1) J_n^m(u),
// b the element's own moments about the group's centre, so the sum over the
// copies is done once for all 64 elements.  A dielectric row takes the normal
// component of the field instead: -N.grad of the irregular harmonic (n, m) is a
// combination of (n + 1, m) and (n + 1, m +- 1), one more degree of the same
// sums, and is put in their place before the products.
#pragma once
#include "group_far.hpp"

namespace nebem {

// The orders m go to the workgroup's four waves: 0..2, 3..5, 6..8, 9..15
// (74, 72, 54 and 56 real sums; all 136 complex ones would be 512 registers).
constexpr int kSets = 4;
__host__ __device__ constexpr int set_lo(int w) { return 3 * w; }
__host__ __device__ constexpr int set_hi(int w) { return w == 3 ? kGroupL : 3 * w + 2; }
// slot of (n, m) in its set, degrees through top
__host__ __device__ constexpr int set_slot(int w, int n, int m, int top)
{
    int s = 0;
    for (int k = set_lo(w); k < m; ++k) s += top + 1 - k;
    return s + n - m;
}
__host__ __device__ constexpr int set_terms(int w, int top) { return set_slot(w, set_hi(w) + 1, set_hi(w) + 1, top); }
// An element's moments: set by set, (re, im) by slot, each set padded to whole
// scalar loads of 8.
__host__ __device__ constexpr int set_coefs(int w)
{
    int s = 0;
    for (int m = set_lo(w); m <= set_hi(w) && m <= kGroupP; ++m) s += kGroupP + 1 - m;
    return (2 * s + 7) / 8 * 8;
}
__host__ __device__ constexpr int set_offset(int w)
{
    int s = 0;
    for (int k = 0; k < w; ++k) s += set_coefs(k);
    return s;
}
constexpr int kElemCoefs = set_offset(kSets);

// The orders that a neighbouring set needs, 2, 3, 5, 6, 8, 9: slots of
// (n, m) in the exchange buffer.
__host__ __device__ constexpr int exchange_slot(int n, int m)
{
    int s = 0;
    for (int k = 2; k < m; ++k)
        if (k % 3 != 1) s += kGroupL + 1 - k;
    return s + n - m;
}
constexpr int kExchange = exchange_slot(kGroupL, 9) + 1;

// Factors of the normal component's terms (n + 1, m), (n + 1, m + 1), (n + 1, m - 1)
// in that of (n, m).
struct NormalFactors {
    double f[(kGroupP + 1) * (kGroupP + 1) * 4];
};
constexpr NormalFactors make_normal_factors()
{
    NormalFactors t{};
    for (int n = 0; n <= kGroupP; ++n)
        for (int m = 0; m <= n; ++m) {
            double *f = t.f + (n * (kGroupP + 1) + m) * 4;
            const HarmonicTables &h = kHarm;
            f[0] = h.lam[n][m] * (n - m + 1) / h.lam[n + 1][m];
            f[1] = 0.5 * h.lam[n][m] / h.lam[n + 1][m + 1];
            f[2] = m > 0 ? 0.5 * h.lam[n][m] * (n - m + 1) * (n - m + 2) / h.lam[n + 1][m - 1] : 0.0;
        }
    return t;
}

template <int W>
struct LatticeSums {
    static constexpr int LO = set_lo(W), HI = set_hi(W), NT = set_terms(W, kGroupL);
    double re[NT], im[NT];  // F_n^m; those of m = 0 are real

    __device__ __forceinline__ static constexpr int at(int n, int m) { return set_slot(W, n, m, kGroupL); }

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < NT; ++k) re[k] = im[k] = 0.0;
    }

    // par x one copy at offset d, degrees through deg (7, 11 or 15, uniform)
    __device__ __forceinline__ void add(const GroupVec &d, double r2, double a, double par, int deg)
    {
        const double y = __builtin_amdgcn_rsq(r2);
        const double e = fma(-(r2 * y), y, 1.0);
        const double ir = fma(y * e, fma(e, 0.375, 0.5), y);
        const double t = a * ir, s = t * ir, t2 = t * t;
        const double xt = d.x * s, yt = d.y * s, zt = d.z * s;
        double pr = par * t, pi = 0.0;  // par t (x + i y)^m, scaled
        auto times = [&](double br, double bi) {
            const double q = fma(pr, br, -(pi * bi));
            pi = fma(pr, bi, pi * br);
            pr = q;
        };
        if constexpr (LO > 0) {
            const double x2 = fma(xt, xt, -(yt * yt)), y2 = 2.0 * xt * yt;
            const double x3 = fma(x2, xt, -(y2 * yt)), y3 = fma(x2, yt, y2 * xt);
#pragma unroll
            for (int k = 0; k < LO / 3; ++k) times(x3, y3);
        }
#pragma unroll
        for (int m = LO; m <= HI; ++m) {
            double q0 = 0.0, q1 = 1.0;
            auto term = [&](int n) {
                if (n > m) {
                    const double q = n == m + 1 ? zt : fma(kHarm.c[n - 1][m] * zt, q1, -(t2 * q0));
                    q0 = q1;
                    q1 = q;
                }
                re[at(n, m)] = n == m ? re[at(n, m)] + pr : fma(q1, pr, re[at(n, m)]);
                if (m > 0) im[at(n, m)] = n == m ? im[at(n, m)] + pi : fma(q1, pi, im[at(n, m)]);
            };
            if (LO <= 7 || deg > 7) {
#pragma unroll
                for (int n = m; n <= (LO <= 7 ? 7 : 11); ++n) term(n);
                if (deg > (LO <= 7 ? 7 : 11)) {
#pragma unroll
                    for (int n = (LO <= 7 ? 8 : 12) > m ? (LO <= 7 ? 8 : 12) : m; n <= (LO <= 7 ? 11 : kGroupL); ++n) term(n);
                    if (LO <= 7 && deg > 11)
#pragma unroll
                        for (int n = 12; n <= kGroupL; ++n) term(n);
                }
            }
            if (m == 0) {
                pi = pr * yt;
                pr = pr * xt;
            } else if (m < HI) {
                times(xt, yt);
            }
        }
    }

    // orders that the neighbouring sets read, to x[slot][re, im][lane]
    __device__ __forceinline__ void put_exchange(double *x) const
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int m = LO; m <= HI; ++m)
            if ((m == LO && W > 0) || (m == HI && W + 1 < kSets))
#pragma unroll
                for (int n = m; n <= kGroupL; ++n) {
                    x[exchange_slot(n, m) * 128 + lane] = re[at(n, m)];
                    x[exchange_slot(n, m) * 128 + 64 + lane] = im[at(n, m)];
                }
    }

    // where `normal`, F_n^m -> a times -N.grad of its harmonic, n <= kGroupP
    __device__ __forceinline__ void normal_component(const double *x, cdouble_p tab, bool normal, double Nx, double Ny, double Nz)
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int n = LO; n <= kGroupP; ++n)
#pragma unroll
            for (int m = LO; m <= (HI < n ? HI : n); ++m) {
                __builtin_amdgcn_sched_barrier(0);
                const double f0 = tab[(n * (kGroupP + 1) + m) * 4], f1 = tab[(n * (kGroupP + 1) + m) * 4 + 1],
                             f2 = tab[(n * (kGroupP + 1) + m) * 4 + 2];
                double ur, ui;
                if (m < HI) {
                    ur = re[at(n + 1, m + 1)];
                    ui = im[at(n + 1, m + 1)];
                } else {
                    ur = x[exchange_slot(n + 1, m + 1) * 128 + lane];
                    ui = x[exchange_slot(n + 1, m + 1) * 128 + 64 + lane];
                }
                double vr, vi;
                if (m == 0) {
                    vr = fma(f0 * Nz, re[at(n + 1, 0)], 2.0 * f1 * fma(Nx, ur, Ny * ui));
                    vi = 0.0;
                } else {
                    double lr, li;
                    if (m > LO) {
                        lr = re[at(n + 1, m - 1)];
                        li = m == 1 ? 0.0 : im[at(n + 1, m - 1)];
                    } else {
                        lr = x[exchange_slot(n + 1, m - 1) * 128 + lane];
                        li = x[exchange_slot(n + 1, m - 1) * 128 + 64 + lane];
                    }
                    vr = fma(f0 * Nz, re[at(n + 1, m)],
                             fma(f1, fma(Nx, ur, Ny * ui), -f2 * fma(Nx, lr, -(Ny * li))));
                    vi = fma(f0 * Nz, im[at(n + 1, m)],
                             fma(f1, fma(Nx, ui, -(Ny * ur)), -f2 * fma(Nx, li, Ny * lr)));
                }
                re[at(n, m)] = normal ? vr : re[at(n, m)];
                im[at(n, m)] = normal ? vi : im[at(n, m)];
            }
    }

    // this set's part of sum Re(conj(b) F), b an element's moments of the set
    __device__ __forceinline__ double dot(cdouble_p b) const
    {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int v = 0; v < set_coefs(W) / 8; ++v) {
            const d8 c = *(cd8_p)(b + 8 * v);
#pragma unroll
            for (int m = LO; m <= (HI < kGroupP ? HI : kGroupP); ++m)
#pragma unroll
                for (int n = m; n <= kGroupP; ++n) {
                    const int k = set_slot(W, n, m, kGroupP);
                    if (k / 4 == v) {
                        s0 = fma(c[2 * (k % 4)], re[at(n, m)], s0);
                        if (m > 0) s1 = fma(c[2 * (k % 4) + 1], im[at(n, m)], s1);
                    }
                }
        }
        return s0 + s1;
    }
};

}  // namespace nebem
