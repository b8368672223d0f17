// group_kernels.hip -- moments of the element groups and the far part of a
// grouped FP64 evaluation (expansion and tables: group_far.hpp).
//
// An evaluation of N elements x C copies at M points is N C M closed forms,
// ~73 VALU instructions each, though in a lattice nearly all of them are tens
// to hundreds of element sizes away.  Here the far copies of each group of 64
// elements cost one expansion (9 instructions per harmonic: ~390 through
// degree 6, ~1400 through degree 14) instead of 64 closed forms (~4700); the
// copies nearer than ~7 group radii are left to k_group_near
// (field_kernels.hip), which evaluates them element by element.
//
// Copies far from four consecutive groups at once take one expansion of the
// four, whose moments follow from theirs; with copies up to 5 cells away that is
// nearly all of them, at a degree two to four higher.
//
// Measured (double THGEM, 41 600 elements, 121 copies, 40 000 points): 469 ms
// with the closed forms everywhere, 102 ms with groups (far pass 74 ms, near pass
// 26), 59 ms with four at once (far 30, near 28), 37 with sixteen, the bound at 3e-12
// and the widest segments first (far 18, near 17); the far pass issues at ~75 % of the
// FP64 rate.  Three waves per SIMD and two entries ahead: two waves 79 ms (of 74),
// four 76, one entry ahead 87, three 83.  64 points of the GEM cell, one row of an
// expansion or 8 elements of a group per wave: 23.5 ms -> 0.58 ms.  Errors against
// 64-bit sums: group_far.hpp.
#include <hip/hip_runtime.h>

#include "lattice_far.hpp"
#include "nebem_internal.hpp"

namespace nebem {

// ----------------------------------------------------------------- moments
// One workgroup per group and density column, one wave per order m, one lane
// per element: the 8 x 8 Gauss rule (collapsed onto the triangle) integrates
// the degree-14 polynomials of an element's moments exactly.  Compute bound
// and short (~6000 instructions a wave); the coefficient columns are written
// once, 8.8 KB per group.
constexpr int kMomWaves = kGroupP + 1;
constexpr int kRule = 8;
__constant__ double kRuleX[kRule] = {0.0198550717512318841, 0.1016667612931866302, 0.2372337950418355070,
                                     0.4082826787521750975, 0.5917173212478249024, 0.7627662049581644929,
                                     0.8983332387068133697, 0.9801449282487681158};
__constant__ double kRuleW[kRule] = {0.0506142681451881295, 0.1111905172266872352, 0.1568533229389436436,
                                     0.1813418916891809914, 0.1813418916891809914, 0.1568533229389436436,
                                     0.1111905172266872352, 0.0506142681451881295};

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
    return v;
}

struct MomElem {
    double ox, oy, oz;  // corner relative to the centre, over a
    double ux, uy, uz, wx, wy, wz;  // edges over a
    double q;           // density x |u| |w|
    bool tri;
};

struct Quad {
    double v[4][3];  // vertices (a triangle's third one twice)
};
__device__ __forceinline__ Quad element_vertices(const double *__restrict__ r)
{
    Quad e;
    const double lx = r[R_LX], lz = r[R_LZ];
    const bool tri = r[R_KIND] != 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        e.v[0][k] = r[R_OX + k];
        e.v[1][k] = e.v[0][k] + lx * r[R_E1X + k];
        e.v[2][k] = e.v[0][k] + lz * r[R_E2X + k];
        e.v[3][k] = tri ? e.v[2][k] : e.v[1][k] + lz * r[R_E2X + k];
    }
    return e;
}
// least and largest coordinate k of the wave's vertices
__device__ __forceinline__ void wave_box(const Quad &e, int k, double &lo, double &hi)
{
    lo = wave_min(fmin(fmin(e.v[0][k], e.v[1][k]), fmin(e.v[2][k], e.v[3][k])));
    hi = -wave_min(-fmax(fmax(e.v[0][k], e.v[1][k]), fmax(e.v[2][k], e.v[3][k])));
}
// largest squared distance of the wave's vertices from c, NaN if one is
__device__ __forceinline__ double wave_radius2(const Quad &e, const double (&c)[3])
{
    double a2 = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double d2 = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double d = e.v[q][k] - c[k];
            d2 = fma(d, d, d2);
        }
        a2 = d2 > a2 || d2 != d2 ? d2 : a2;
    }
    return __ballot(a2 != a2) ? __builtin_nan("") : -wave_min(-a2);
}
// Centre c and squared radius a2 of up to 64 elements, one per lane, one wave.
__device__ __forceinline__ void group_sphere(const double *__restrict__ recs, int cnt, double (&c)[3], double &a2)
{
    const Quad e = element_vertices(recs + (size_t)min((int)(threadIdx.x & 63), cnt - 1) * R_STRIDE);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double lo, hi;
        wave_box(e, k, lo, hi);
        c[k] = 0.5 * (lo + hi);
    }
    a2 = wave_radius2(e, c);
}

// an element (record r, density sg) in the frame of a sphere
__device__ __forceinline__ MomElem sphere_element(const double *r, double sg, const double (&c)[3], double ia)
{
    const double lx = r[R_LX], lz = r[R_LZ], x = lx * ia, z = lz * ia;
    MomElem e;
    e.ox = (r[R_OX] - c[0]) * ia;
    e.oy = (r[R_OY] - c[1]) * ia;
    e.oz = (r[R_OZ] - c[2]) * ia;
    e.ux = x * r[R_E1X];
    e.uy = x * r[R_E1Y];
    e.uz = x * r[R_E1Z];
    e.wx = z * r[R_E2X];
    e.wy = z * r[R_E2Y];
    e.wz = z * r[R_E2Z];
    e.q = sg * (lx * lz);
    e.tri = r[R_KIND] != 0.0;
    return e;
}

// adds q (s/a)^n J_n^m(s/|s|) integrated over the lane's element, n = M .. kGroupP
template <int M>
__device__ __forceinline__ void element_order(const MomElem &e, double (&ar)[kGroupP + 1 - M],
                                              double (&ai)[kGroupP + 1 - M])
{
#pragma unroll 1
    for (int iv = 0; iv < kRule; ++iv) {
        const double v = kRuleX[iv], sv = e.tri ? 1.0 - v : 1.0;
#pragma unroll 1
        for (int iu = 0; iu < kRule; ++iu) {
            const double s = kRuleX[iu] * sv;
            const double w = e.q * (kRuleW[iu] * kRuleW[iv] * sv);
            const double x = fma(s, e.ux, fma(v, e.wx, e.ox)), y = fma(s, e.uy, fma(v, e.wy, e.oy)),
                         z = fma(s, e.uz, fma(v, e.wz, e.oz));
            const double s2 = fma(x, x, fma(y, y, z * z));
            double cr = w, ci = 0.0;  // w (x + i y)^m
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const double t = fma(cr, x, -(ci * y));
                ci = fma(cr, y, ci * x);
                cr = t;
            }
            double pr = 0.0, pi = 0.0;  // degree n - 1
#pragma unroll
            for (int n = M; n <= kGroupP; ++n) {
                ar[n - M] += cr;
                if (M > 0) ai[n - M] += ci;
                if (n < kGroupP) {
                    const double c = n == M ? z : kHarm.c[n][M] * z;
                    const double nr = fma(c, cr, -(s2 * pr)), ni = fma(c, ci, -(s2 * pi));
                    pr = cr;
                    pi = ci;
                    cr = nr;
                    ci = ni;
                }
            }
        }
    }
}

// the group's sums times their factors, in bre / bim[n]
template <int M>
__device__ __forceinline__ void moment_order(const double *__restrict__ recs, const double *__restrict__ sigma, int cnt,
                                             const double (&c)[3], double ia, double *__restrict__ bre,
                                             double *__restrict__ bim)
{
    double ar[kGroupP + 1 - M], ai[kGroupP + 1 - M];
#pragma unroll
    for (int k = 0; k <= kGroupP - M; ++k) ar[k] = ai[k] = 0.0;
#pragma unroll 1
    for (int i = threadIdx.x & 63; i < cnt; i += 64)
        element_order<M>(sphere_element(recs + (size_t)i * R_STRIDE, sigma[i], c, ia), ar, ai);
#pragma unroll
    for (int n = M; n <= kGroupP; ++n) {
        const double r = wave_sum(ar[n - M]), i = M > 0 ? wave_sum(ai[n - M]) : 0.0;
        if ((threadIdx.x & 63) == 0) {
            bre[n * (kGroupP + 1) + M] = kHarm.bf[n][M] * r;
            bim[n * (kGroupP + 1) + M] = kHarm.bf[n][M] * i;
        }
    }
}

// an element's moments (lattice_far.hpp) of order M, lane by lane
template <int M>
__device__ __forceinline__ void coef_order(const MomElem &e, double *__restrict__ out)
{
    constexpr int W = M / 3 < kSets ? M / 3 : kSets - 1;
    double ar[kGroupP + 1 - M], ai[kGroupP + 1 - M];
#pragma unroll
    for (int k = 0; k <= kGroupP - M; ++k) ar[k] = ai[k] = 0.0;
    element_order<M>(e, ar, ai);
#pragma unroll
    for (int n = M; n <= kGroupP; ++n) {
        const double f = kHarm.bf[n][M] / kHarm.lam[n][M];
        double *q = out + set_offset(W) + 2 * set_slot(W, n, M, kGroupP);
        q[0] = f * ar[n - M];
        q[1] = f * ai[n - M];
    }
}

__device__ const HarmonicTables kHarmDev = make_harmonic_tables();

// Record of a group: its head (centre c, squared radius a2; no super-group, see
// k_parent_moments; differ: kHeadDiffer) and, one (L, m) per thread, the field's
// coefficients from the moments B = bre + i bim.
__device__ __forceinline__ void write_record(double *__restrict__ out, const double (&c)[3], double a2, bool bad,
                                             bool differ, const double *__restrict__ bre,
                                             const double *__restrict__ bim)
{
    if (threadIdx.x < kGroupHead) {
        const int k = threadIdx.x;
        const double inf = __builtin_inf();
        const double t = k < kHeadTier + kTiers ? a2 * tier_ratio2(k - kHeadTier) : 0.0;
        double v = k < 3 ? c[min(k, 2)] : k == 3 ? sqrt(a2) : bad ? inf : t;
        if (k >= kHeadSuper && k < kHeadSuper + 3) v = c[min(k - kHeadSuper, 2)];
        if (k == kHeadSuper + 3) v = __builtin_nan("");
        if (k == kHeadDiffer) v = differ ? 1.0 : 0.0;
        out[k] = v;
    }
    for (int t = threadIdx.x; t < kGroupEntries; t += blockDim.x) {
        int L = 1, m = t;
        while (m > L) {
            m -= L + 1;
            ++L;
        }
        auto B = [&](int mm, double &br, double &bi) {  // B_{L-1, mm}, 0 outside
            const bool in = mm >= 0 && mm <= L - 1;
            br = in ? bre[(L - 1) * (kGroupP + 1) + mm] : 0.0;
            bi = in ? bim[(L - 1) * (kGroupP + 1) + mm] : 0.0;
        };
        double br, bi, ur, ui, dr, di;
        B(m, br, bi);      // d_z
        B(m - 1, ur, ui);  // raised order
        B(m + 1, dr, di);  // lowered order
        const double h = m == 1 ? 1.0 : 0.5;  // from m = 0 both shifts are the one harmonic of order 1
        const double gl = 0.5 * (L - 1 - m) * (L - m);
        const double il = 1.0 / kHarmDev.lam[L][m];
        ui = m == 1 ? 0.0 : ui;
        const double xr = fma(h, ur, -gl * dr) * il, xi = fma(h, ui, -gl * di) * il;
        const double yr = -fma(h, ui, gl * di) * il, yi = fma(h, ur, gl * dr) * il;
        const double zr = (L - m) * br * il, zi = (L - m) * bi * il;
        double *q = out + kGroupHead + kEntry * entry_index(L, m);
        q[0] = xr;
        q[1] = xi;
        q[2] = yr;
        q[3] = yi;
        q[4] = zr;
        q[5] = zi;
        q[6] = m <= L - 2 ? kHarmDev.c[L - 1][m] : 0.0;
        q[7] = 0.0;
    }
}

// Records of the groups (kGroupStride doubles each, record q of segment s at
// (s rps + q): gps groups, then the super-groups); density column k at gdata + k
// gstride.  A group with a density or a vertex that is not finite gets
// infinite thresholds: its elements are all evaluated one by one, and so is a
// super-group's share left to its groups.
__global__ __launch_bounds__(64 * kMomWaves) void k_group_moments(const double *__restrict__ drec,
                                                                  const double *__restrict__ sigma, int n,
                                                                  int64_t sig_stride, int segsz, int gps, int rps,
                                                                  double *__restrict__ gdata, int64_t gstride)
{
    __shared__ double bre[(kGroupP + 1) * (kGroupP + 1)], bim[(kGroupP + 1) * (kGroupP + 1)];
    const int seg = blockIdx.x / gps, q = blockIdx.x % gps;
    const int end = min(n, (seg + 1) * segsz), e0 = seg * segsz + q * kGroupElems;
    if (e0 >= end) return;  // uniform: this group does not exist in a short last segment
    const int cnt = min(kGroupElems, end - e0);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double *recs = drec + (size_t)e0 * R_STRIDE;
    const double *sg = sigma + (size_t)blockIdx.y * sig_stride;
    double c[3], a2;
    group_sphere(recs, cnt, c, a2);
    const bool inf = __ballot(lane < cnt && !isfinite(sg[e0 + lane])) != 0;
    const bool bad = !(a2 > 0.0) || !isfinite(a2) || inf;
    bool differ = false;  // column 0 knows for all
    if (blockIdx.y == 0)
        for (unsigned k = 1; k < gridDim.y; ++k)
            differ = differ || (__ballot(lane < cnt && !isfinite(sg[(size_t)k * sig_stride + e0 + lane])) != 0) != inf;
    const double ia = 1.0 / sqrt(a2);
    sg += e0;
    switch (wave) {
    case 0: moment_order<0>(recs, sg, cnt, c, ia, bre, bim); break;
    case 1: moment_order<1>(recs, sg, cnt, c, ia, bre, bim); break;
    case 2: moment_order<2>(recs, sg, cnt, c, ia, bre, bim); break;
    case 3: moment_order<3>(recs, sg, cnt, c, ia, bre, bim); break;
    case 4: moment_order<4>(recs, sg, cnt, c, ia, bre, bim); break;
    case 5: moment_order<5>(recs, sg, cnt, c, ia, bre, bim); break;
    case 6: moment_order<6>(recs, sg, cnt, c, ia, bre, bim); break;
    case 7: moment_order<7>(recs, sg, cnt, c, ia, bre, bim); break;
    case 8: moment_order<8>(recs, sg, cnt, c, ia, bre, bim); break;
    case 9: moment_order<9>(recs, sg, cnt, c, ia, bre, bim); break;
    case 10: moment_order<10>(recs, sg, cnt, c, ia, bre, bim); break;
    case 11: moment_order<11>(recs, sg, cnt, c, ia, bre, bim); break;
    case 12: moment_order<12>(recs, sg, cnt, c, ia, bre, bim); break;
    case 13: moment_order<13>(recs, sg, cnt, c, ia, bre, bim); break;
    default: moment_order<14>(recs, sg, cnt, c, ia, bre, bim); break;
    }
    __syncthreads();
    write_record(gdata + (int64_t)blockIdx.y * gstride + (int64_t)(seg * rps + q) * kGroupStride, c, a2, bad, differ, bre,
                 bim);
}

// Records of the parents -- super-groups of four groups (level 1), then of four
// super-groups (level 2) -- from those of their children: the moments about
// the common centre are exact finite sums over the children's (addition theorem of
// R_n^m = r^n P_n^m e^(i m phi) / (n+m)!, with R_n^-m = (-1)^m conj R_n^m and the
// Condon-Shortley sign),
//   R_n^m(s + d) = sum_{k,l} R_k^l(d) R_{n-k}^{m-l}(s).
// One thread per child and (n, m).  Integrating the elements again about the
// common centre took 150 us for 8064 elements; this takes 26.
//
// A parent's radius is its elements' or, if that is more, so large that a copy
// far from it is far from every child too (far: beyond rho radii; a copy at rho
// a of the parent is at least rho a - |offset| from the child): so a record
// leaves to its parent what is far from that, and nobody needs to look further
// up.
constexpr int kTerms = (kGroupP + 1) * (kGroupP + 2) / 2;
constexpr int kOrders = (kGroupP + 1) * (kGroupP + 1);
__device__ __forceinline__ int order(int n, int m) { return n * (n + 1) + m; }
// (n, m) and (n, -m), m >= 0, from R_n^m without the Condon-Shortley sign
__device__ __forceinline__ void put_orders(double2 *t, int n, int m, double re, double im)
{
    const double s = m & 1 ? -1.0 : 1.0;
    t[order(n, m)] = {s * re, s * im};
    if (m > 0) t[order(n, -m)] = {re, -im};
}
constexpr int kParentThreads = 128 * kSuper;
__global__ __launch_bounds__(kParentThreads) void k_parent_moments(const double *__restrict__ drec, int n, int segsz,
                                                                  int gps, int rps, int level,
                                                                  double *__restrict__ gdata, int64_t gstride)
{
    __shared__ double2 R[kSuper][kOrders];  // a child's sums, orders -n .. n
    __shared__ double2 T[kSuper][kOrders];  // R of its offset
    __shared__ double bre[(kGroupP + 1) * (kGroupP + 1)], bim[(kGroupP + 1) * (kGroupP + 1)];
    __shared__ double fact[kGroupP + 1];
    constexpr int kWaves = kParentThreads / 64;
    const int sps = parents_of(gps), count = level == 1 ? sps : parents_of(sps);
    const int seg = blockIdx.x / count, sq = blockIdx.x % count;
    const int span = kGroupElems * (level == 1 ? 1 : kSuper);  // elements per child
    const int end = min(n, (seg + 1) * segsz), s0 = seg * segsz + sq * (kSuper * span);
    if (s0 >= end) return;
    double *const seg_data = gdata + (int64_t)blockIdx.y * gstride + (int64_t)seg * rps * kGroupStride;
    double *const children = seg_data + (int64_t)((level == 1 ? 0 : gps) + sq * kSuper) * kGroupStride;
    double *const self = seg_data + (int64_t)((level == 1 ? gps : gps + sps) + sq) * kGroupStride;
    const int nchild = min(kSuper, (end - s0 + span - 1) / span);
    const int wave = threadIdx.x >> 6;
    double sc[3], sa2;
    bool bad = false;
    {  // the sphere
        __shared__ double box[kWaves][6], rad[kWaves];
        const int cnt = min(kSuper * span, end - s0);
        double lo[3], hi[3];
        for (int i0 = 0; i0 < cnt; i0 += kParentThreads) {
            const Quad e = element_vertices(drec + (size_t)(s0 + min(i0 + (int)threadIdx.x, cnt - 1)) * R_STRIDE);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                double l, h;
                wave_box(e, k, l, h);
                lo[k] = i0 ? fmin(lo[k], l) : l;
                hi[k] = i0 ? fmax(hi[k], h) : h;
            }
        }
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                box[wave][k] = lo[k];
                box[wave][3 + k] = hi[k];
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double l = box[0][k], h = box[0][3 + k];
#pragma unroll
            for (int j = 1; j < kWaves; ++j) {
                l = fmin(l, box[j][k]);
                h = fmax(h, box[j][3 + k]);
            }
            sc[k] = 0.5 * (l + h);
        }
        double a2 = 0.0;
        for (int i0 = 0; i0 < cnt; i0 += kParentThreads) {
            const double r2 = wave_radius2(
                element_vertices(drec + (size_t)(s0 + min(i0 + (int)threadIdx.x, cnt - 1)) * R_STRIDE), sc);
            a2 = r2 > a2 || r2 != r2 ? r2 : a2;
        }
        if ((threadIdx.x & 63) == 0) rad[wave] = a2;
        __syncthreads();
        sa2 = rad[0];
#pragma unroll
        for (int j = 1; j < kWaves; ++j) sa2 = rad[j] > sa2 || rad[j] != rad[j] ? rad[j] : sa2;
        for (int k = 0; k < nchild; ++k) {
            const double *h = children + (int64_t)k * kGroupStride;
            const double x = h[0] - sc[0], y = h[1] - sc[1], z = h[2] - sc[2];
            // rho > 7; the last factor is far above the rounding of a copy's distance
            const double r = (h[3] + sqrt(x * x + y * y + z * z) * (1.0 / 7.0)) * (1.0 + 1e-9);
            sa2 = r * r > sa2 ? r * r : sa2;
            bad = bad || h[kHeadTier] == __builtin_inf();
        }
        bad = bad || !(sa2 > 0.0) || !isfinite(sa2);
    }
    const double ia = 1.0 / sqrt(sa2);
    const int child = threadIdx.x >> 7, q = threadIdx.x & 127;
    const bool has = child < nchild;
    double *rec = children + (int64_t)(has ? child : 0) * kGroupStride;
    if (threadIdx.x == 0) {
        double f = 1.0;
        for (int k = 0; k <= kGroupP; ++k) {
            fact[k] = f;
            f *= k + 1;
        }
    }
    int tn = 0, tm = q;
    while (tm > tn) {
        tm -= tn + 1;
        ++tn;
    }
    __syncthreads();
    if (q < kTerms) {  // from the coefficient of Ez at (n + 1, m)
        const double *e = rec + kGroupHead + kEntry * entry_index(tn + 1, tm);
        double f = kHarmDev.lam[tn + 1][tm] / ((tn + 1 - tm) * (tm ? 2.0 : 1.0) * fact[tn - tm]);
        const double ratio = rec[3] * ia;
        for (int k = 0; k < tn; ++k) f *= ratio;
        put_orders(R[child], tn, tm, has ? f * e[4] : 0.0, has ? f * e[5] : 0.0);
    }
    if (q <= kGroupP) {  // column q of the offset's table
        const double x = (rec[0] - sc[0]) * ia, y = (rec[1] - sc[1]) * ia, z = (rec[2] - sc[2]) * ia;
        const double r2 = fma(x, x, fma(y, y, z * z));
        double cr = 1.0, ci = 0.0, pr = 0.0, pi = 0.0;
        for (int k = 1; k <= q; ++k) {
            const double h = 0.5 / k, t = h * fma(cr, x, -(ci * y));
            ci = h * fma(cr, y, ci * x);
            cr = t;
        }
        for (int k = q; k <= kGroupP; ++k) {
            put_orders(T[child], k, q, cr, ci);
            const double d = 1.0 / ((k + q + 1.0) * (k - q + 1.0)), w = (2 * k + 1) * z;
            const double nr = d * fma(w, cr, -(r2 * pr)), ni = d * fma(w, ci, -(r2 * pi));
            pr = cr;
            pi = ci;
            cr = nr;
            ci = ni;
        }
    }
    __syncthreads();
    double sr = 0.0, si = 0.0;
    if (q < kTerms)
        for (int k = 0; k <= tn; ++k) {
            const int j = tn - k, l0 = max(-k, tm - j), l1 = min(k, tm + j);
            const double2 *t = &T[child][order(k, 0)], *r = &R[child][order(j, tm)];
#pragma unroll 4
            for (int l = l0; l <= l1; ++l) {
                const double2 u = t[l], v = r[-l];
                sr = fma(u.x, v.x, fma(-u.y, v.y, sr));
                si = fma(u.x, v.y, fma(u.y, v.x, si));
            }
        }
    __syncthreads();
    if (q < kTerms) T[child][q] = {sr, si};
    __syncthreads();
    if (child == 0 && q < kTerms) {
        const double f = (tm ? 2.0 : 1.0) * fact[tn - tm] * (tm & 1 ? -1.0 : 1.0);
        double r = T[0][q].x, i = T[0][q].y;
#pragma unroll
        for (int c = 1; c < kSuper; ++c) {
            r += T[c][q].x;
            i += T[c][q].y;
        }
        bre[tn * (kGroupP + 1) + tm] = f * r;
        bim[tn * (kGroupP + 1) + tm] = f * i;
    }
    __syncthreads();
    // a child that is not fit leaves its parent's share to the children
    if (has && q < 4) rec[kHeadSuper + q] = q < 3 ? sc[min(q, 2)] : bad ? __builtin_inf() : sa2 * tier_ratio2(0);
    write_record(self, sc, sa2, bad, false, bre, bim);
}

void launch_group_moments(const double *drec, const double *sigma, int64_t n, int64_t sig_stride, int ncol,
                          const SegPlan &sp, double *gdata, hipStream_t s)
{
    if (n <= 0 || ncol <= 0) return;
    const int gps = groups_per_seg(sp), rps = records_per_seg(sp);
    const int64_t gstride = (int64_t)sp.nseg * rps * kGroupStride;
    hipLaunchKernelGGL(k_group_moments, dim3((unsigned)(sp.nseg * gps), (unsigned)ncol), dim3(64 * kMomWaves), 0, s,
                       drec, sigma, (int)n, sig_stride, sp.segsz, gps, rps, gdata, gstride);
    const int sps = parents_of(gps);
    for (int level = 1; level <= far_levels(sp); ++level)
        hipLaunchKernelGGL(k_parent_moments, dim3((unsigned)(sp.nseg * (level == 1 ? sps : parents_of(sps))), (unsigned)ncol),
                           dim3(kParentThreads), 0, s, drec, (int)n, sp.segsz, gps, rps, level, gdata, gstride);
}

// Moments of every element about its group's centre, kElemCoefs each, and
// the groups' heads: the assembly's far field.  As k_group_moments, but each lane
// keeps its element's integrals; the 2 KB per element are a 32nd of a matrix column
// of 8000 rows.
__global__ __launch_bounds__(64 * kMomWaves) void k_element_moments(const double *__restrict__ drec, int n,
                                                                    double *__restrict__ heads,
                                                                    double *__restrict__ coef)
{
    const int e0 = blockIdx.x * kGroupElems, cnt = min(kGroupElems, n - e0);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double c[3], a2;
    group_sphere(drec + (size_t)e0 * R_STRIDE, cnt, c, a2);
    const MomElem e = sphere_element(drec + (size_t)(e0 + min(lane, cnt - 1)) * R_STRIDE, 1.0, c, 1.0 / sqrt(a2));
    if (threadIdx.x < kGroupHead) {
        const int k = threadIdx.x;
        const double inf = __builtin_inf();
        const bool bad = !(a2 > 0.0) || !isfinite(a2);
        const double t = k < kHeadTier + kTiers ? a2 * tier_ratio2(k - kHeadTier) : 0.0;
        heads[(size_t)blockIdx.x * kGroupHead + k] = k < 3 ? c[min(k, 2)] : k == 3 ? sqrt(a2) : bad ? inf : t;
    }
    if (lane >= cnt) return;
    double *out = coef + (size_t)(e0 + lane) * kElemCoefs;
    switch (__builtin_amdgcn_readfirstlane(wave)) {
    case 0: coef_order<0>(e, out); break;
    case 1: coef_order<1>(e, out); break;
    case 2: coef_order<2>(e, out); break;
    case 3: coef_order<3>(e, out); break;
    case 4: coef_order<4>(e, out); break;
    case 5: coef_order<5>(e, out); break;
    case 6: coef_order<6>(e, out); break;
    case 7: coef_order<7>(e, out); break;
    case 8: coef_order<8>(e, out); break;
    case 9: coef_order<9>(e, out); break;
    case 10: coef_order<10>(e, out); break;
    case 11: coef_order<11>(e, out); break;
    case 12: coef_order<12>(e, out); break;
    case 13: coef_order<13>(e, out); break;
    default: coef_order<14>(e, out); break;
    }
    // the sets' padding is read with them
    if (wave < kSets) {
        int used = 0;
        for (int m = set_lo(wave); m <= set_hi(wave) && m <= kGroupP; ++m) used += kGroupP + 1 - m;
        for (int k = 2 * used; k < set_coefs(wave); ++k) out[set_offset(wave) + k] = 0.0;
    }
}

size_t assemble_scratch_doubles(int64_t n)
{
    return (size_t)((n + kGroupElems - 1) / kGroupElems) * kGroupHead + (size_t)n * kElemCoefs;
}

void launch_element_moments(const double *drec, int64_t n, double *heads, double *coef, hipStream_t s)
{
    hipLaunchKernelGGL(k_element_moments, dim3((unsigned)((n + kGroupElems - 1) / kGroupElems)), dim3(64 * kMomWaves),
                       0, s, drec, (int)n, heads, coef);
}

// Segments by falling sum of their groups' squared radii, which goes with
// their near copies: in unsplit passes a segment's waves at points near its
// widest groups run for milliseconds (the planes of a THGEM: 16 groups of 64
// elements x 25 copies), and started last they leave the device idle.  Near pass of
// 40 000 THGEM points 26 ms in index order, 19 with these first (17 with
// waves of their own workgroup); far pass 21, 18.
__global__ __launch_bounds__(64) void k_segment_order(const double *__restrict__ gdata, int n, int nseg, int segsz,
                                                      int rps, int *__restrict__ order)
{
    const int s = threadIdx.x;
    double cost = 0.0;
    if (s < nseg) {
        const int ng = (min(segsz, n - s * segsz) + kGroupElems - 1) / kGroupElems;
#pragma unroll 8
        for (int g = 0; g < ng; ++g) {
            const double a = gdata[((int64_t)s * rps + g) * kGroupStride + 3];
            cost = fma(a, a, cost);
        }
        if (!(cost <= 1e300)) cost = 1e300;  // not finite: all its groups may be near
    }
    int rank = 0;
    for (int t = 0; t < nseg; ++t) {
        const double c = __shfl(cost, t);
        rank += c > cost || (c == cost && t < s);
    }
    if (s < nseg) order[rank] = s;
}

int *segment_order(double *gdata, int ncol, const SegPlan &sp)
{
    return reinterpret_cast<int *>(gdata + (size_t)sp.nseg * records_per_seg(sp) * kGroupStride * (size_t)ncol);
}

void launch_segment_order(const double *gdata, int64_t n, const SegPlan &sp, int *order, hipStream_t s)
{
    hipLaunchKernelGGL(k_segment_order, dim3(1), dim3(64), 0, s, gdata, (int)n, sp.nseg, sp.segsz, records_per_seg(sp),
                       order);
}

// --------------------------------------------------------------------- far
// Place of expansion k among a segment's records: those of gps groups, of
// their parents and of these ones' parents, of which ng groups and their
// ancestors exist.
__device__ __forceinline__ int record_index(int k, int ng, int gps)
{
    const int ns = parents_of(ng);
    return k < ng ? k : k < ng + ns ? gps + k - ng : gps + parents_of(gps) + k - ng - ns;
}

// Far copies of the expansions [g0, g1) of a segment at one point per lane, lattice
// rows [q0, q1) (row q: reflection q / (2 n1 + 1), translation i1 = q % (2 n1 +
// 1) - n1): rows added into the group's sum, groups into acc, in that order.
// FP64 VALU bound; the coefficients come through the scalar cache (64 bytes per
// nine vector instructions), nothing is staged in LDS and the waves of a
// workgroup run independently.
__device__ __forceinline__ void far_unit(cdouble_p gd, int ng, int gps, const ImgArgs &img, double Px, double Py,
                                         double Pz, int g0, int g1, int q0, int q1, double (&acc)[4])
{
#pragma clang fp contract(off)
    for (int c = 0; c < 4; ++c) acc[c] = 0.0;
    const int nrow = 2 * img.n1 + 1;
#pragma unroll 1
    for (int g = g0; g < g1; ++g) {
        cdouble_p h = gd + (int64_t)record_index(g, ng, gps) * kGroupStride;
        const double a = h[3];
        double grp[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int q = q0; q < q1; ++q) {
            const int r = q / nrow, i1 = q % nrow - img.n1;
            const int ax = img.axes[r];
            const GroupVec v0 = group_origin(img, ax, Px, Py, Pz, h);
            const GroupVec v1 = group_step(v0, -(double)i1, img.a1[r]);
            const GroupVec s1 =
                group_step(group_origin(img, ax, Px, Py, Pz, h + kHeadSuper), -(double)i1, img.a1[r]);
            double row[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
            for (int i2 = -img.n2; i2 <= img.n2; ++i2) {
                // copies far from the parent are its own
                const bool own = !(group_r2(group_step(s1, -(double)i2, img.a2[r])) >= h[kHeadSuper + 3]);
                if (__ballot(own) == 0) continue;
                const GroupVec d = group_step(v1, -(double)i2, img.a2[r]);
                const double r2 = group_r2(d);
                if (own && r2 >= h[kHeadTier]) {
                    if (r2 >= h[kHeadTier + 3]) {
                        if (r2 >= h[kHeadTier + 5])
                            group_far<5>(d, r2, a, h + kGroupHead, row);
                        else if (r2 >= h[kHeadTier + 4])
                            group_far<7>(d, r2, a, h + kGroupHead, row);
                        else
                            group_far<9>(d, r2, a, h + kGroupHead, row);
                    } else {
                        if (r2 >= h[kHeadTier + 2])
                            group_far<11>(d, r2, a, h + kGroupHead, row);
                        else if (r2 >= h[kHeadTier + 1])
                            group_far<13>(d, r2, a, h + kGroupHead, row);
                        else
                            group_far<15>(d, r2, a, h + kGroupHead, row);
                    }
                }
            }
            const double par = img.parity[r];
            grp[0] = fma(par, row[0], grp[0]);
            grp[1] = fma((ax & 1) ? -par : par, row[1], grp[1]);
            grp[2] = fma((ax & 2) ? -par : par, row[2], grp[2]);
            grp[3] = fma((ax & 4) ? -par : par, row[3], grp[3]);
        }
        for (int c = 0; c < 4; ++c) acc[c] += grp[c];
    }
}

// Grid: x over points, y over units -- whole segments (split 0), expansions
// (split 1) or lattice rows of them (split 2; y = record * rows + row) --, z
// over density columns (their shared harmonics are a third of the work, but
// two columns at once need more registers than three waves per SIMD leave).
// Unit y's unscaled sums go to the outputs + y * unit_stride.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_group_far(
    const double *__restrict__ gdata, int64_t gstride, int n, int segsz, int gps, int rps, int levels, ImgArgs img, int split,
    const int *__restrict__ order,
    const double *__restrict__ px, const double *__restrict__ py, const double *__restrict__ pz, int m, OutCols out,
    int64_t unit_stride)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = min(i, m - 1);  // lanes past the last point repeat it
    const int rows = img.nref * (2 * img.n1 + 1);
    int y = blockIdx.y, q0 = 0, q1 = rows;
    if (split == 2) {
        q0 = y % rows;
        q1 = q0 + 1;
        y /= rows;
    }
    const int seg = split ? y / rps : order[y];
    const int ng = (min(segsz, n - seg * segsz) + kGroupElems - 1) / kGroupElems;
    int g0 = 0, g1 = records_of(ng, levels);
    if (split) {  // record q of the segment, if it exists
        const int q = y % rps, sps = parents_of(gps), ns = parents_of(ng);
        const int k = q < gps ? q : q < gps + sps ? ng + q - gps : ng + ns + q - gps - sps;
        const bool exists = q < gps ? q < ng : q < gps + sps ? q - gps < ns : k < g1;
        g0 = k;
        g1 = exists ? k + 1 : k;
    }
    double acc[4];
    far_unit(uniform_ptr(gdata + (int64_t)blockIdx.z * gstride + (int64_t)seg * rps * kGroupStride), ng, gps, img, px[j],
             py[j], pz[j], g0, g1, q0, q1, acc);
    if (i >= m) return;
    const int64_t o = (int64_t)(split ? (int)blockIdx.y : seg) * unit_stride + (int64_t)blockIdx.z * out.stride + i;
    for (int c = 0; c < 4; ++c)
        if (out.c[c]) out.c[c][o] = acc[c];
}

void launch_group_far(const double *gdata, int64_t n, int ncol, const SegPlan &sp, const ImgArgs &img, int split, const int *order,
                      const double *px, const double *py, const double *pz, int64_t m, const OutCols &out,
                      int64_t unit_stride, hipStream_t s)
{
    if (m <= 0 || n <= 0) return;
    const int gps = groups_per_seg(sp), rps = records_per_seg(sp);
    const int64_t nrec = (int64_t)sp.nseg * rps, rows = (int64_t)img.nref * (2 * img.n1 + 1);
    const int64_t units = split == 0 ? sp.nseg : split == 1 ? nrec : nrec * rows;
    const int bs = split == 0 ? 256 : 64;
    hipLaunchKernelGGL(k_group_far, dim3((unsigned)((m + bs - 1) / bs), (unsigned)units, (unsigned)ncol), dim3(bs), 0,
                       s, gdata, nrec * kGroupStride, (int)n, sp.segsz, gps, rps, far_levels(sp), img, split, order, px, py, pz, (int)m, out,
                       unit_stride);
}

// Serving: workgroup (one wave) b takes work item b where its geometry is
// grouped -- the far part of one segment at up to 64 points of one request, or
// (units set) of expansion y of it, whose sums go to units[b][y][component][lane].
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_items_far(
    const WorkItem *__restrict__ items, const ImgArgs *__restrict__ imgs, double *__restrict__ units)
{
    const WorkItem &w = items[blockIdx.x];
    if (!w.gdata) return;
    const ImgArgs &img = imgs[w.geom];
    const int j = min((int)threadIdx.x, w.count - 1);
    const int ng = (w.n + kGroupElems - 1) / kGroupElems;
    const int nrec = records_of(ng, w.levels);
    const int g0 = units ? (int)blockIdx.y : 0, g1 = units ? g0 + 1 : nrec;
    if (g0 >= nrec) return;
    double acc[4];
    far_unit(uniform_ptr(w.gdata), ng, w.groups, img, w.px[j], w.py[j], w.pz[j], g0, g1, 0,
             img.nref * (2 * img.n1 + 1), acc);
    if ((int)threadIdx.x >= w.count) return;
    if (units) {
        double *u = units + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kUnitDoubles + threadIdx.x;
        for (int c = 0; c < 4; ++c) u[64 * c] = acc[c];
        return;
    }
    w.phi[threadIdx.x] = acc[0];
    w.ex[threadIdx.x] = acc[1];
    w.ey[threadIdx.x] = acc[2];
    w.ez[threadIdx.x] = acc[3];
}

void launch_items_far(const WorkItem *items, int nitems, const ImgArgs *imgs, double *units, int per, hipStream_t s)
{
    if (nitems <= 0) return;
    hipLaunchKernelGGL(k_items_far, dim3(nitems, units ? per : 1), dim3(64), 0, s, items, imgs, units);
}

// The items' units back to one value per point, in the order in which a whole
// item adds them.
__global__ __launch_bounds__(256) void k_items_fold(const WorkItem *__restrict__ items,
                                                    const double *__restrict__ far,
                                                    const double *__restrict__ near, int far_per, int per)
{
    const WorkItem &w = items[blockIdx.x];
    const int lane = threadIdx.x & 63, c = threadIdx.x >> 6;
    if (lane >= w.count) return;
    const double *u = near + (int64_t)blockIdx.x * per * kUnitDoubles + threadIdx.x;
    const bool grouped = w.gdata != nullptr;
    const int cnt = item_units(w.n, grouped);
    double n = 0.0;
    if (grouped) {
        for (int g = 0; g < cnt; g += kNearRuns) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < kNearRuns; ++q) t += u[(int64_t)(g + q) * kUnitDoubles];
            n += t;
        }
        const double *v = far + (int64_t)blockIdx.x * far_per * kUnitDoubles + threadIdx.x;
        const int nfar = item_far_units(w.n, w.levels);
        double f = 0.0;
        for (int q = 0; q < nfar; ++q) f += v[(int64_t)q * kUnitDoubles];
        n = f + n;
    } else {
        for (int q = 0; q < cnt; ++q) n += u[(int64_t)q * kUnitDoubles];
    }
    (c == 0 ? w.phi : c == 1 ? w.ex : c == 2 ? w.ey : w.ez)[lane] = n;
}

void launch_items_fold(const WorkItem *items, int nitems, const double *far, const double *near, int far_per, int per,
                       hipStream_t s)
{
    if (nitems <= 0) return;
    hipLaunchKernelGGL(k_items_fold, dim3(nitems), dim3(256), 0, s, items, far, near, far_per, per);
}

// ------------------------------------------------------------ finer units
// Sums of a split evaluation back to one value per segment, in the order the
// unsplit kernels add them: rows / runs into their group, groups into their
// segment, the segment's far and near sums added last.
__global__ __launch_bounds__(256) void k_fold_units(const double *__restrict__ in, int per, int64_t len,
                                                    double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    const double *p = in + (int64_t)blockIdx.y * per * len + i;
    double acc = 0.0;
    for (int k = 0; k < per; ++k) acc += p[k * len];
    out[(int64_t)blockIdx.y * len + i] = acc;
}

__global__ __launch_bounds__(256) void k_fold_groups(const double *__restrict__ far, const double *__restrict__ near,
                                                     int rps, int gps, int64_t len, double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    far += (int64_t)blockIdx.y * rps * len + i;
    near += (int64_t)blockIdx.y * gps * len + i;
    double f = 0.0, n = 0.0;
    for (int g = 0; g < rps; ++g) f += far[g * len];
    for (int g = 0; g < gps; ++g) n += near[g * len];
    out[(int64_t)blockIdx.y * len + i] = f + n;
}

void launch_fold_units(const double *in, int64_t groups, int per, int64_t len, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_fold_units, dim3((unsigned)((len + 255) / 256), (unsigned)groups), dim3(256), 0, s, in, per,
                       len, out);
}

void launch_fold_groups(const double *far, const double *near, const SegPlan &sp, int64_t len, double *out,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_fold_groups, dim3((unsigned)((len + 255) / 256), (unsigned)sp.nseg), dim3(256), 0, s, far,
                       near, records_per_seg(sp), groups_per_seg(sp), len, out);
}

// ----------------------------------------------------------------- the rule
bool eval_grouped(int64_t n, const ImgArgs &img) { return img.hole < 0 && grouping_pays(n, img_copies(img)); }

size_t group_record_bytes() { return kGroupStride * sizeof(double); }

}  // namespace nebem
