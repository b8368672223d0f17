// field_kernels.hip -- element preparation, field evaluation and influence
// matrix assembly on gfx950.
//
// Work decomposition (both field kernels): one lane owns one observation
// point (an evaluation point, or a collocation row of the matrix) and keeps
// its sums in FP64 registers; the lanes of a wave walk the elements together,
// so element data are wave-uniform and live in scalar registers (evaluation:
// scalar loads; direct assembly: an LDS tile shared by a workgroup's four waves).  The
// element kind (rectangle / right triangle) is
// therefore a uniform branch, and the copy loops (lattice translations and
// reflections) are uniform loops.  Each point sums elements in index order
// and copies in lattice order, independent of which other points share its
// wave: results are deterministic and do not depend on the batch a point
// arrives in.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>
#include <cmath>

#include "nebem_internal.hpp"
#include "farfield_mixed.hpp"
#include "lattice_far.hpp"
#include "panel_fp64.hpp"

namespace nebem {

constexpr int kBlock = 256;
constexpr int kTileE = kGroupElems;  // elements within which triangle pairs are taken, evaluation
constexpr int kRunElems = kGroupElems / kNearRuns;    // elements per unit of a split near pass
constexpr int kSubElems = kGroupElems / kNearParts;  // elements per unit of a split evaluation
constexpr int kTileA = 32;   // elements (columns) per workgroup, assembly

// wave-uniform copy of a value held identically by all lanes -> SGPRs
__device__ __forceinline__ double uni(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// ------------------------------------------------------------------- prep
__global__ __launch_bounds__(kBlock) void k_prep(nebem_panels p, double *__restrict__ drec, int *__restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= p.n) return;
    const int kind = p.kind[i];
    const int bc = p.bc[i];
    const double ox = p.ox[i], oy = p.oy[i], oz = p.oz[i];
    const double ux = p.ux[i], uy = p.uy[i], uz = p.uz[i];
    const double wx = p.wx[i], wy = p.wy[i], wz = p.wz[i];
    const double lu = sqrt(ux * ux + uy * uy + uz * uz);
    const double lw = sqrt(wx * wx + wy * wy + wz * wz);
    const double uw = ux * wx + uy * wy + uz * wz;
    bool ok = (kind == 0 || kind == 1) && (bc == 0 || bc == 1) && lu > 0.0 && lw > 0.0 &&
              isfinite(lu) && isfinite(lw) && isfinite(ox) && isfinite(oy) && isfinite(oz) &&
              fabs(uw) <= 1e-9 * lu * lw;
    double jump = 0.0;
    if (bc == 1) {
        const double ep = p.eps_pos[i], en = p.eps_neg[i];
        ok = ok && ep > 0.0 && en > 0.0 && ep != en && isfinite(ep) && isfinite(en);
        jump = (ep + en) / (2.0 * kEps0 * (ep - en));
    }
    if (!ok) {
        atomicAdd(&bad[0], 1);
        atomicMin(&bad[1], (int)i);
        return;
    }
    const double e1x = ux / lu, e1y = uy / lu, e1z = uz / lu;
    const double c = wx * e1x + wy * e1y + wz * e1z;
    double vx = wx - c * e1x, vy = wy - c * e1y, vz = wz - c * e1z;
    const double lz = sqrt(vx * vx + vy * vy + vz * vz);
    vx /= lz;
    vy /= lz;
    vz /= lz;
    const double e3x = e1y * vz - e1z * vy, e3y = e1z * vx - e1x * vz, e3z = e1x * vy - e1y * vx;
    const double lx = lu;
    const double hyp = sqrt(lx * lx + lz * lz);
    const double f = kind == 0 ? 0.5 : (1.0 / 3.0);
    double *r = drec + i * R_STRIDE;
    r[R_OX] = ox;
    r[R_OY] = oy;
    r[R_OZ] = oz;
    r[R_E1X] = e1x;
    r[R_E1Y] = e1y;
    r[R_E1Z] = e1z;
    r[R_E2X] = vx;
    r[R_E2Y] = vy;
    r[R_E2Z] = vz;
    r[R_E3X] = e3x;
    r[R_E3Y] = e3y;
    r[R_E3Z] = e3z;
    r[R_LX] = lx;
    r[R_LZ] = lz;
    r[R_HYP] = hyp;
    r[R_IHYP] = 1.0 / hyp;
    r[R_CX] = ox + f * (ux + wx);
    r[R_CY] = oy + f * (uy + wy);
    r[R_CZ] = oz + f * (uz + wz);
    r[R_DIAM] = hyp;
    r[R_AREA] = kind == 0 ? lx * lz : 0.5 * lx * lz;
    r[R_KIND] = (double)kind;
    r[R_JUMP] = jump;
    r[R_BC] = (double)bc;
}

// Triangle pairs: two consecutive right triangles with the same right-angle
// corner, one leg shared (same direction and length) and the other legs
// opposite -- the two halves of a triangle cut at the foot of its altitude,
// as a mesher emits them -- all to 1e-12 relative.  Element i is marked
// kind 2 when its second leg is the shared one (the pair's first triangle
// is i), kind 3 when its first leg is (the first triangle is i + 1).  The
// field kernels then evaluate the two together (rtri_pair_far), taking the
// second triangle's legs as c e2 and -b e1 in the first one's frame: a
// change of its geometry of at most 1e-12 relative, below the far forms'
// own rounding error (~R/D ulps).  Only i's kind is written, so launches
// over any ranges of elements agree.
__device__ __forceinline__ double dist3(const double *a, const double *b, double sb)
{
    const double x = a[0] - sb * b[0], y = a[1] - sb * b[1], z = a[2] - sb * b[2];
    return sqrt(x * x + y * y + z * z);
}

__global__ __launch_bounds__(kBlock) void k_pair_flags(nebem_panels p, double *__restrict__ drec)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i + 1 >= p.n) return;
    if (p.kind[i] != 1 || p.kind[i + 1] != 1) return;
    double *r = drec + i * R_STRIDE;
    const double *q = r + R_STRIDE;
    constexpr double tol = 1e-12;
    if (!(dist3(r + R_OX, q + R_OX, 1.0) <= tol * fmax(r[R_DIAM], q[R_DIAM]))) return;
    if (dist3(r + R_E2X, q + R_E1X, 1.0) <= tol && dist3(r + R_E1X, q + R_E2X, -1.0) <= tol &&
        fabs(r[R_LZ] - q[R_LX]) <= tol * r[R_LZ])
        r[R_KIND] = 2.0;
    else if (dist3(q + R_E2X, r + R_E1X, 1.0) <= tol && dist3(q + R_E1X, r + R_E2X, -1.0) <= tol &&
             fabs(q[R_LZ] - r[R_LX]) <= tol * q[R_LZ])
        r[R_KIND] = 3.0;
}

void launch_prep(const nebem_panels *p, double *drec, int *bad, hipStream_t s)
{
    if (p->n <= 0) return;
    const unsigned g = (unsigned)((p->n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_prep, dim3(g), dim3(kBlock), 0, s, *p, drec, bad);
    hipLaunchKernelGGL(k_pair_flags, dim3(g), dim3(kBlock), 0, s, *p, drec);
}

// ------------------------------------------------------------- one element
// Uniform element data, loaded from an LDS record.
struct Elem {
    double ox, oy, oz, e1x, e1y, e1z, e2x, e2y, e2z, e3x, e3y, e3z;
    double lx, lz, hyp, ihyp;
    double diam, area;
    int kind;
};

__device__ __forceinline__ Elem load_elem(const double *d)
{
    Elem e;
    e.ox = uni(d[R_OX]);
    e.oy = uni(d[R_OY]);
    e.oz = uni(d[R_OZ]);
    e.e1x = uni(d[R_E1X]);
    e.e1y = uni(d[R_E1Y]);
    e.e1z = uni(d[R_E1Z]);
    e.e2x = uni(d[R_E2X]);
    e.e2y = uni(d[R_E2Y]);
    e.e2z = uni(d[R_E2Z]);
    e.e3x = uni(d[R_E3X]);
    e.e3y = uni(d[R_E3Y]);
    e.e3z = uni(d[R_E3Z]);
    e.lx = uni(d[R_LX]);
    e.lz = uni(d[R_LZ]);
    e.hyp = uni(d[R_HYP]);
    e.ihyp = uni(d[R_IHYP]);
    e.diam = uni(d[R_DIAM]);
    e.area = uni(d[R_AREA]);
    e.kind = uni((int)d[R_KIND]);
    return e;
}

// The second triangle of a pair (element records of kind 2 or 3: see
// k_pair_flags): what the pair form needs from its record.
struct PairB {
    double lz, hyp, ihyp, diam, area;
};

// The same from the records in memory, by scalar loads: no staging in LDS and
// no moves to scalar registers (38 per element, a tenth of an element's work when
// it has one copy), and the waves of a workgroup run independently.
__device__ __forceinline__ Elem load_elem_c(cdouble_p d)
{
    return {d[R_OX],  d[R_OY],  d[R_OZ], d[R_E1X], d[R_E1Y], d[R_E1Z], d[R_E2X],  d[R_E2Y],  d[R_E2Z], d[R_E3X],
            d[R_E3Y], d[R_E3Z], d[R_LX], d[R_LZ],  d[R_HYP], d[R_IHYP], d[R_DIAM], d[R_AREA], uni((int)d[R_KIND])};
}
__device__ __forceinline__ PairB load_pair_b_c(cdouble_p d)
{
    return {d[R_LZ], d[R_HYP], d[R_IHYP], d[R_DIAM], d[R_AREA]};
}

// Sum over lattice translations of one element, local frame; (X0,Z0,H0) is
// the (reflected) point in the element frame for the zero translation, and
// (aX,aZ,aH), (bX,bZ,bH) the lattice vectors in that frame.  `self` zeroes H
// for the zero translation (collocation point on its own element).
// MIXED: copies far enough for a low-order FP32 correction to stay within
// its error budget (R >= 24 D rectangles, 48 D triangles, and never below
// near_factor D) take the FP64 monopole + FP32 correction far field (per
// lane); nearer copies take the exact FP64 closed form, which in that band is
// no more expensive than a higher-order rule would be.
// The exact form is taken per lane in its far-regime evaluation when the
// point is at least kFarDiam diameters from the element's corner o, else in
// the cancellation-free general one; the choice depends on the point alone.
struct MixParams {
    double low2;    // squared distance from which the FP32 low-order rule is used
    double quad2;   // squared distance from which the quadrupole expansion is used
};

template <int KIND, bool MIXED, bool HOLE>
__device__ __forceinline__ void sum_translations(const Elem &e, int n1, int n2, int hole, double X0, double Z0,
                                                 double H0, double aX, double aZ, double aH, double bX, double bZ,
                                                 double bH, bool self, const MixParams &mp, double &sp,
                                                 double &sx, double &sz, double &sn)
{
    const double cxl = KIND == 0 ? 0.5 * e.lx : e.lx * (1.0 / 3.0);
    const double czl = KIND == 0 ? 0.5 * e.lz : e.lz * (1.0 / 3.0);
    const double far2 = (kFarDiam * kFarDiam) * (e.diam * e.diam);
    const double vfar2 = (kVeryFarDiam * kVeryFarDiam) * (e.diam * e.diam);
    FarCorr fc = {0.0f, 0.0f, 0.0f, 0.0f};
    // MIXED: the copies are translated in centroid-relative coordinates,
    // which the far tiers use directly; the exact tiers add the centroid
    // offset back
    if (MIXED) {
        X0 -= cxl;
        Z0 -= czl;
    }
#pragma unroll 1
    for (int i1 = -n1; i1 <= n1; ++i1) {
        const double f1 = -(double)i1;
        const double X1 = fma(f1, aX, X0), Z1 = fma(f1, aZ, Z0), H1 = fma(f1, aH, H0);
        // HOLE: a row that crosses the hole runs as two ranges of i2, so the
        // inner loop itself carries no test for it
        const bool cut = HOLE && abs(i1) <= hole;
#pragma unroll 1
        for (int seg = 0; seg <= (int)cut; ++seg) {
            const int i2a = seg == 0 ? -n2 : hole + 1;
            const int i2b = (cut && seg == 0) ? -hole - 1 : n2;
#pragma unroll 1
            for (int i2 = i2a; i2 <= i2b; ++i2) {
                const double f2 = -(double)i2;
                double X = fma(f2, bX, X1), Z = fma(f2, bZ, Z1);
                double H = fma(f2, bH, H1);
                H = (self && i1 == 0 && i2 == 0) ? 0.0 : H;
                if (MIXED) {
                    const double rc2 = fma(X, X, fma(Z, Z, H * H));
                    if (rc2 >= mp.quad2) {
                        far_quadrupole<KIND>(X, Z, H, rc2, e.lx, e.lz, e.area, sp, sx, sz, sn, fc);
                        continue;
                    }
                    if (rc2 >= mp.low2) {
                        far_mixed<KIND>(X, Z, H, rc2, e.lx, e.lz, e.area, sp, sx, sz, sn, fc);
                        continue;
                    }
                    X += cxl;
                    Z += czl;
                }
                Kern k;
                const double r0sq = fma(X, X, fma(Z, Z, H * H));
                if (r0sq >= vfar2) {  // far forms return the potential added to sp
                    if (KIND == 0)
                        k = rect_far<true>(X, H, Z, e.lx, e.lz, r0sq, sp);
                    else
                        k = rtri_far<true>(X, H, Z, e.lx, e.lz, e.hyp, r0sq, sp);
                } else if (r0sq >= far2) {
                    if (KIND == 0)
                        k = rect_far<false>(X, H, Z, e.lx, e.lz, r0sq, sp);
                    else
                        k = rtri_far<false>(X, H, Z, e.lx, e.lz, e.hyp, r0sq, sp);
                } else {
                    if (KIND == 0)
                        k = rect_fp64(X, H, Z, e.lx, e.lz, r0sq);
                    else
                        k = rtri_fp64(X, H, Z, e.lx, e.lz, e.hyp, e.ihyp, r0sq);
                    k.phi += sp;
                }
                sp = k.phi;
                sx += k.ex;
                sz += k.ez;
                sn += k.en;
            }
        }
    }
    if (MIXED) {
        sp = fma(e.area, (double)fc.p, sp);
        sx = fma(e.area, (double)fc.x, sx);
        sz = fma(e.area, (double)fc.z, sz);
        sn = fma(e.area, (double)fc.n, sn);
    }
}

// phi', E' (global frame) of one element with all its copies at P.
template <bool MIXED, bool HOLE = false>
__device__ __forceinline__ void element_copies(const Elem &e, const ImgArgs &img, double Px, double Py, double Pz,
                                               bool self, double near_factor, double &ophi, double &oex,
                                               double &oey, double &oez)
{
    MixParams mp;
    if (MIXED) {
        const double nd = near_factor * e.diam;
        const double ld = fmax(nd, (e.kind == 0 ? 24.0 : 48.0) * e.diam);
        const double qd = fmax(nd, (e.kind == 0 ? 32.0 : 96.0) * e.diam);
        mp.low2 = ld * ld;
        mp.quad2 = qd * qd;
    }
    ophi = oex = oey = oez = 0.0;
    for (int r = 0; r < img.nref; ++r) {
        const int ax = img.axes[r];
        const double Qx = (ax & 1) ? 2.0 * img.mpos[0] - Px : Px;
        const double Qy = (ax & 2) ? 2.0 * img.mpos[1] - Py : Py;
        const double Qz = (ax & 4) ? 2.0 * img.mpos[2] - Pz : Pz;
        const double rx = Qx - e.ox, ry = Qy - e.oy, rz = Qz - e.oz;
        const double X0 = rx * e.e1x + ry * e.e1y + rz * e.e1z;
        const double Z0 = rx * e.e2x + ry * e.e2y + rz * e.e2z;
        const double H0 = rx * e.e3x + ry * e.e3y + rz * e.e3z;
        const double *a = img.a1[r], *b = img.a2[r];
        const double aX = a[0] * e.e1x + a[1] * e.e1y + a[2] * e.e1z;
        const double aZ = a[0] * e.e2x + a[1] * e.e2y + a[2] * e.e2z;
        const double aH = a[0] * e.e3x + a[1] * e.e3y + a[2] * e.e3z;
        const double bX = b[0] * e.e1x + b[1] * e.e1y + b[2] * e.e1z;
        const double bZ = b[0] * e.e2x + b[1] * e.e2y + b[2] * e.e2z;
        const double bH = b[0] * e.e3x + b[1] * e.e3y + b[2] * e.e3z;
        double sp = 0.0, sx = 0.0, sz = 0.0, sn = 0.0;
        const bool s = self && r == 0;
        if (e.kind == 0)
            sum_translations<0, MIXED, HOLE>(e, img.n1, img.n2, img.hole, X0, Z0, H0, aX, aZ, aH, bX, bZ, bH, s, mp, sp,
                                       sx, sz, sn);
        else
            sum_translations<1, MIXED, HOLE>(e, img.n1, img.n2, img.hole, X0, Z0, H0, aX, aZ, aH, bX, bZ, bH, s, mp, sp,
                                       sx, sz, sn);
        double gx = sx * e.e1x + sz * e.e2x + sn * e.e3x;
        double gy = sx * e.e1y + sz * e.e2y + sn * e.e3y;
        double gz = sx * e.e1z + sz * e.e2z + sn * e.e3z;
        gx = (ax & 1) ? -gx : gx;
        gy = (ax & 2) ? -gy : gy;
        gz = (ax & 4) ? -gz : gz;
        const double par = img.parity[r];
        ophi += par * sp;
        oex += par * gx;
        oey += par * gy;
        oez += par * gz;
    }
}

// Sum over lattice translations of a triangle pair (FP64 evaluation only),
// in the first triangle's frame: the second triangle's legs are c = e.lz
// along e2 and b = f.lz along -e1 (the geometry the pair flag was tested
// for, within 1e-12 of its own record), so its frame is (e2, -e1, e3) and
// its sums come back in that frame.  Tiers as in sum_translations, by the
// distance from the shared corner in units of the larger diameter; below
// the far regime each triangle takes the general form.
template <bool HOLE>
__device__ __forceinline__ void sum_translations_pair(const Elem &e, const PairB &f, int n1, int n2, int hole,
                                                      double X0, double Z0, double H0, double aX, double aZ,
                                                      double aH, double bX, double bZ, double bH, double (&s1)[4],
                                                      double (&s2)[4])
{
    const double a = e.lx, c = e.lz, b = f.lz;
    const double dp = fmax(e.diam, f.diam);
    const double far2 = (kFarDiam * kFarDiam) * (dp * dp);
    const double vfar2 = (kVeryFarDiam * kVeryFarDiam) * (dp * dp);
#pragma unroll 1
    for (int i1 = -n1; i1 <= n1; ++i1) {
        const double f1 = -(double)i1;
        const double X1 = fma(f1, aX, X0), Z1 = fma(f1, aZ, Z0), H1 = fma(f1, aH, H0);
        const bool cut = HOLE && abs(i1) <= hole;
#pragma unroll 1
        for (int seg = 0; seg <= (int)cut; ++seg) {
            const int i2a = seg == 0 ? -n2 : hole + 1;
            const int i2b = (cut && seg == 0) ? -hole - 1 : n2;
#pragma unroll 1
            for (int i2 = i2a; i2 <= i2b; ++i2) {
                const double f2 = -(double)i2;
                const double X = fma(f2, bX, X1), Z = fma(f2, bZ, Z1);
                const double H = fma(f2, bH, H1);
                const double r0sq = fma(X, X, fma(Z, Z, H * H));
                Kern k1, k2;
                if (r0sq >= vfar2) {  // far forms return the potentials added to the sums
                    rtri_pair_far<true>(X, H, Z, a, b, c, e.hyp, f.hyp, r0sq, s1[0], s2[0], k1, k2);
                } else if (r0sq >= far2) {
                    rtri_pair_far<false>(X, H, Z, a, b, c, e.hyp, f.hyp, r0sq, s1[0], s2[0], k1, k2);
                } else {
                    k1 = rtri_fp64(X, H, Z, a, c, e.hyp, e.ihyp, r0sq);
                    k2 = rtri_fp64(Z, H, -X, c, b, f.hyp, f.ihyp, r0sq);
                    k1.phi += s1[0];
                    k2.phi += s2[0];
                }
                s1[0] = k1.phi;
                s1[1] += k1.ex;
                s1[2] += k1.ez;
                s1[3] += k1.en;
                s2[0] = k2.phi;
                s2[1] += k2.ex;
                s2[2] += k2.ez;
                s2[3] += k2.en;
            }
        }
    }
}

// phi', E' (global frame) of both triangles of a pair with all their copies
// at P: o1 for the first, o2 for the second.
template <bool HOLE>
__device__ __forceinline__ void element_pair_copies(const Elem &e, const PairB &f, const ImgArgs &img, double Px,
                                                    double Py, double Pz, double (&o1)[4], double (&o2)[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) o1[c] = o2[c] = 0.0;
    for (int r = 0; r < img.nref; ++r) {
        const int ax = img.axes[r];
        const double Qx = (ax & 1) ? 2.0 * img.mpos[0] - Px : Px;
        const double Qy = (ax & 2) ? 2.0 * img.mpos[1] - Py : Py;
        const double Qz = (ax & 4) ? 2.0 * img.mpos[2] - Pz : Pz;
        const double rx = Qx - e.ox, ry = Qy - e.oy, rz = Qz - e.oz;
        const double X0 = rx * e.e1x + ry * e.e1y + rz * e.e1z;
        const double Z0 = rx * e.e2x + ry * e.e2y + rz * e.e2z;
        const double H0 = rx * e.e3x + ry * e.e3y + rz * e.e3z;
        const double *a = img.a1[r], *b = img.a2[r];
        const double aX = a[0] * e.e1x + a[1] * e.e1y + a[2] * e.e1z;
        const double aZ = a[0] * e.e2x + a[1] * e.e2y + a[2] * e.e2z;
        const double aH = a[0] * e.e3x + a[1] * e.e3y + a[2] * e.e3z;
        const double bX = b[0] * e.e1x + b[1] * e.e1y + b[2] * e.e1z;
        const double bZ = b[0] * e.e2x + b[1] * e.e2y + b[2] * e.e2z;
        const double bH = b[0] * e.e3x + b[1] * e.e3y + b[2] * e.e3z;
        double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
        sum_translations_pair<HOLE>(e, f, img.n1, img.n2, img.hole, X0, Z0, H0, aX, aZ, aH, bX, bZ, bH, s1, s2);
        // first triangle: frame (e1, e2, e3); second: (e2, -e1, e3)
        double g1x = s1[1] * e.e1x + s1[2] * e.e2x + s1[3] * e.e3x;
        double g1y = s1[1] * e.e1y + s1[2] * e.e2y + s1[3] * e.e3y;
        double g1z = s1[1] * e.e1z + s1[2] * e.e2z + s1[3] * e.e3z;
        double g2x = s2[1] * e.e2x - s2[2] * e.e1x + s2[3] * e.e3x;
        double g2y = s2[1] * e.e2y - s2[2] * e.e1y + s2[3] * e.e3y;
        double g2z = s2[1] * e.e2z - s2[2] * e.e1z + s2[3] * e.e3z;
        g1x = (ax & 1) ? -g1x : g1x;
        g1y = (ax & 2) ? -g1y : g1y;
        g1z = (ax & 4) ? -g1z : g1z;
        g2x = (ax & 1) ? -g2x : g2x;
        g2y = (ax & 2) ? -g2y : g2y;
        g2z = (ax & 4) ? -g2z : g2z;
        const double par = img.parity[r];
        o1[0] += par * s1[0];
        o1[1] += par * g1x;
        o1[2] += par * g1y;
        o1[3] += par * g1z;
        o2[0] += par * s2[0];
        o2[1] += par * g2x;
        o2[2] += par * g2y;
        o2[3] += par * g2z;
    }
}

// ----------------------------------------------------- mixed-path pairs
// In the mixed path a triangle pair far enough away is taken as one charge
// distribution: the sigma-weighted monopole (FP64), dipole and second
// moments (FP32) of both triangles about the centroid c0 of the whole
// triangle they came from.  In the first triangle's frame the pair has
// vertices o, A = o + a e1, C = o + c e2, B = o - b e1; its triangles'
// centroids lie (b/3, 0) and (-a/3, 0) from c0 = o + ((a - b)/3, c/3), so
// with charges w1 = sigma1 A1, w2 = sigma2 A2 the dipole is
// ((w1 b - w2 a)/3, 0) and the second moments are the triangles' central
// ones (right triangle per unit area: lx^2/18, lz^2/18, -lx lz/36 in its
// own frame; the second triangle's frame is (e2, -e1)) moved to c0.  The
// expansion is the multipole series of the single-triangle quadrupole tier
// (farfield_mixed.hpp) with the dipole term added; it is used from 96
// diameters of the whole triangle (a + b, which bounds every vertex's
// distance from c0 by (a + b) 2/3), where the truncation error relative to
// |w1| + |w2| is at most the single triangle's at 96 of its own diameters.
// Nearer copies take each triangle's own mixed tiers.  One such copy costs
// about what one triangle's quadrupole copy costs.
// The FP32 moments are carried in units of sc = |w1| + |w2| (so that their
// range does not depend on the densities' scale), and the FP32 corrections
// are multiplied by sc once, in FP64, after the copies.
template <int K>
struct PairMoments {
    double q[K], sc[K];                   // w1 + w2; |w1| + |w2|
    float dx[K], mxx[K], mzz[K], mxz[K];  // dipole (along e1), second moments, in units of sc
};

template <int K>
__device__ __forceinline__ PairMoments<K> pair_moments(double a, double b, double c, double area1, double area2,
                                                       const double (&sg1)[K], const double (&sg2)[K])
{
    PairMoments<K> m;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double v1 = sg1[k] * area1, v2 = sg2[k] * area2;
        m.q[k] = v1 + v2;
        const double sc = fabs(v1) + fabs(v2);
        m.sc[k] = sc > 0.0 ? sc : 1.0;
        const double w1 = v1 / m.sc[k], w2 = v2 / m.sc[k];
        m.dx[k] = (float)((w1 * b - w2 * a) * (1.0 / 3.0));
        m.mxx[k] = (float)(w1 * (a * a * (1.0 / 18.0) + b * b * (1.0 / 9.0)) +
                           w2 * (b * b * (1.0 / 18.0) + a * a * (1.0 / 9.0)));
        m.mzz[k] = (float)((w1 + w2) * (c * c * (1.0 / 18.0)));
        m.mxz[k] = (float)((w2 * b - w1 * a) * (c * (1.0 / 36.0)));
    }
    return m;
}

// One copy of the pair as one distribution at p = P - c0 (FP64, the first
// triangle's frame), rc2 = |p|^2: sigma-weighted monopole into s[k] (FP64),
// dipole + quadrupole corrections, in units of m.sc[k], into fc[k] (FP32).
template <int K>
__device__ __forceinline__ void pair_far_moments(double px, double pz, double ph, double rc2,
                                                 const PairMoments<K> &m, double (&s)[K][4], FarCorr (&fc)[K])
{
    const float fx = (float)px, fz = (float)pz, fh = (float)ph;
    const float frc2 = (float)rc2;
    const float fic = __builtin_amdgcn_rsqf(frc2);
    const float fic2 = fic * fic;
    const float fic3 = fic2 * fic;
    const float fic5 = fic3 * fic2;
    double ir = (double)fic;
    ir = ir * (1.5 - 0.5 * rc2 * ir * ir);
    const double ir2 = ir * ir;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double air = m.q[k] * ir;
        const double air3 = air * ir2;
        s[k][0] += air;
        s[k][1] = fma(air3, px, s[k][1]);
        s[k][2] = fma(air3, pz, s[k][2]);
        s[k][3] = fma(air3, ph, s[k][3]);
        const float mpx = fmaf(m.mxx[k], fx, m.mxz[k] * fz);
        const float mpz = fmaf(m.mxz[k], fx, m.mzz[k] * fz);
        const float t = m.mxx[k] + m.mzz[k];
        const float u = fmaf(3.0f, fmaf(fx, mpx, fz * mpz), -frc2 * t);  // 3q - R^2 t
        const float dpx = m.dx[k] * fx;                                   // d.p
        const float G = fmaf(3.0f, dpx, fmaf(2.5f * u, fic2, t));  // p coefficient (x fic5): quadrupole g + dipole 3 d.p
        fc[k].p += fmaf(0.5f * u, fic5, dpx * fic3);
        fc[k].x += fmaf(fic5, fmaf(G, fx, -3.0f * mpx), -m.dx[k] * fic3);
        fc[k].z = fmaf(fic5, fmaf(G, fz, -3.0f * mpz), fc[k].z);
        fc[k].n = fmaf(fic5, G * fh, fc[k].n);
    }
}

// One copy of one right triangle in the mixed path, unit density, at
// centroid-relative (Xc, Zc, H) in its own frame: the tiers of
// sum_translations<1, true>.
__device__ __forceinline__ void tri_copy_mixed(double Xc, double Zc, double H, double lx, double lz, double hyp,
                                               double ihyp, double area, const MixParams &mp, double far2,
                                               double vfar2, double (&s)[4], FarCorr &fc)
{
    const double rc2 = fma(Xc, Xc, fma(Zc, Zc, H * H));
    if (rc2 >= mp.quad2) {
        far_quadrupole<1>(Xc, Zc, H, rc2, lx, lz, area, s[0], s[1], s[2], s[3], fc);
        return;
    }
    if (rc2 >= mp.low2) {
        far_mixed<1>(Xc, Zc, H, rc2, lx, lz, area, s[0], s[1], s[2], s[3], fc);
        return;
    }
    const double X = Xc + lx * (1.0 / 3.0), Z = Zc + lz * (1.0 / 3.0);
    const double r0sq = fma(X, X, fma(Z, Z, H * H));
    Kern k;
    if (r0sq >= vfar2) {
        k = rtri_far<true>(X, H, Z, lx, lz, hyp, r0sq, s[0]);
    } else if (r0sq >= far2) {
        k = rtri_far<false>(X, H, Z, lx, lz, hyp, r0sq, s[0]);
    } else {
        k = rtri_fp64(X, H, Z, lx, lz, hyp, ihyp, r0sq);
        k.phi += s[0];
    }
    s[0] = k.phi;
    s[1] += k.ex;
    s[2] += k.ez;
    s[3] += k.en;
}

__device__ __forceinline__ MixParams mix_params(double near_factor, double diam, double low_d, double quad_d)
{
    MixParams mp;
    const double nd = near_factor * diam;
    const double ld = fmax(nd, low_d * diam), qd = fmax(nd, quad_d * diam);
    mp.low2 = ld * ld;
    mp.quad2 = qd * qd;
    return mp;
}

// phi', E' (global frame) of a triangle pair with all its copies at P in the
// mixed path, weighted by each column's densities (sg1, sg2): out[k].
template <int K, bool HOLE>
__device__ __forceinline__ void element_pair_copies_mixed(const Elem &e, const PairB &f, const double (&sg1)[K],
                                                          const double (&sg2)[K], const ImgArgs &img,
                                                          double near_factor, double Px, double Py, double Pz,
                                                          double (&out)[K][4])
{
    const double a = e.lx, c = e.lz, b = f.lz;
    const PairMoments<K> pm = pair_moments<K>(a, b, c, e.area, f.area, sg1, sg2);
    const MixParams mp1 = mix_params(near_factor, e.diam, 48.0, 96.0);
    const MixParams mp2 = mix_params(near_factor, f.diam, 48.0, 96.0);
    const MixParams mpp = mix_params(near_factor, a + b, 48.0, 96.0);
    const double far1 = (kFarDiam * kFarDiam) * (e.diam * e.diam), vfar1 = (kVeryFarDiam * kVeryFarDiam) * (e.diam * e.diam);
    const double far2 = (kFarDiam * kFarDiam) * (f.diam * f.diam), vfar2 = (kVeryFarDiam * kVeryFarDiam) * (f.diam * f.diam);
    const double c0x = (a - b) * (1.0 / 3.0), c0z = c * (1.0 / 3.0);
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) out[k][q] = 0.0;
    for (int r = 0; r < img.nref; ++r) {
        const int ax = img.axes[r];
        const double Qx = (ax & 1) ? 2.0 * img.mpos[0] - Px : Px;
        const double Qy = (ax & 2) ? 2.0 * img.mpos[1] - Py : Py;
        const double Qz = (ax & 4) ? 2.0 * img.mpos[2] - Pz : Pz;
        const double rx = Qx - e.ox, ry = Qy - e.oy, rz = Qz - e.oz;
        // coordinates relative to c0
        const double X0 = rx * e.e1x + ry * e.e1y + rz * e.e1z - c0x;
        const double Z0 = rx * e.e2x + ry * e.e2y + rz * e.e2z - c0z;
        const double H0 = rx * e.e3x + ry * e.e3y + rz * e.e3z;
        const double *av = img.a1[r], *bv = img.a2[r];
        const double aX = av[0] * e.e1x + av[1] * e.e1y + av[2] * e.e1z;
        const double aZ = av[0] * e.e2x + av[1] * e.e2y + av[2] * e.e2z;
        const double aH = av[0] * e.e3x + av[1] * e.e3y + av[2] * e.e3z;
        const double bX = bv[0] * e.e1x + bv[1] * e.e1y + bv[2] * e.e1z;
        const double bZ = bv[0] * e.e2x + bv[1] * e.e2y + bv[2] * e.e2z;
        const double bH = bv[0] * e.e3x + bv[1] * e.e3y + bv[2] * e.e3z;
        double sp[K][4];  // sigma-weighted, first triangle's frame
        FarCorr fp[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            sp[k][0] = sp[k][1] = sp[k][2] = sp[k][3] = 0.0;
            fp[k] = {0.0f, 0.0f, 0.0f, 0.0f};
        }
        double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};  // unit density, own frames
        FarCorr f1 = {0.0f, 0.0f, 0.0f, 0.0f}, f2 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int i1 = -img.n1; i1 <= img.n1; ++i1) {
            const double g1 = -(double)i1;
            const double X1 = fma(g1, aX, X0), Z1 = fma(g1, aZ, Z0), H1 = fma(g1, aH, H0);
            const bool cut = HOLE && abs(i1) <= img.hole;
#pragma unroll 1
            for (int seg = 0; seg <= (int)cut; ++seg) {
                const int i2a = seg == 0 ? -img.n2 : img.hole + 1;
                const int i2b = (cut && seg == 0) ? -img.hole - 1 : img.n2;
#pragma unroll 1
                for (int i2 = i2a; i2 <= i2b; ++i2) {
                    const double g2 = -(double)i2;
                    const double X = fma(g2, bX, X1), Z = fma(g2, bZ, Z1), H = fma(g2, bH, H1);
                    const double rc2 = fma(X, X, fma(Z, Z, H * H));
                    if (rc2 >= mpp.quad2) {
                        pair_far_moments<K>(X, Z, H, rc2, pm, sp, fp);
                        continue;
                    }
                    // each triangle on its own: corner-relative (X + c0x, Z + c0z);
                    // the second one's frame (e2, -e1): (Z + c0z, -(X + c0x))
                    const double Xo = X + c0x, Zo = Z + c0z;
                    tri_copy_mixed(Xo - a * (1.0 / 3.0), Zo - c * (1.0 / 3.0), H, a, c, e.hyp, e.ihyp, e.area, mp1,
                                   far1, vfar1, s1, f1);
                    tri_copy_mixed(Zo - c * (1.0 / 3.0), -Xo - b * (1.0 / 3.0), H, c, b, f.hyp, f.ihyp, f.area, mp2,
                                   far2, vfar2, s2, f2);
                }
            }
        }
        // unit-density sums with their FP32 corrections, the second
        // triangle's turned into the first one's frame (e1 = -e2', e2 = e1')
        const double u1[4] = {fma(e.area, (double)f1.p, s1[0]), fma(e.area, (double)f1.x, s1[1]),
                              fma(e.area, (double)f1.z, s1[2]), fma(e.area, (double)f1.n, s1[3])};
        const double u2[4] = {fma(f.area, (double)f2.p, s2[0]), -fma(f.area, (double)f2.z, s2[2]),
                              fma(f.area, (double)f2.x, s2[1]), fma(f.area, (double)f2.n, s2[3])};
        const double par = img.parity[r];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double l[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) l[q] = fma(sg2[k], u2[q], fma(sg1[k], u1[q], sp[k][q]));
            l[0] = fma(pm.sc[k], (double)fp[k].p, l[0]);
            l[1] = fma(pm.sc[k], (double)fp[k].x, l[1]);
            l[2] = fma(pm.sc[k], (double)fp[k].z, l[2]);
            l[3] = fma(pm.sc[k], (double)fp[k].n, l[3]);
            double gx = l[1] * e.e1x + l[2] * e.e2x + l[3] * e.e3x;
            double gy = l[1] * e.e1y + l[2] * e.e2y + l[3] * e.e3y;
            double gz = l[1] * e.e1z + l[2] * e.e2z + l[3] * e.e3z;
            gx = (ax & 1) ? -gx : gx;
            gy = (ax & 2) ? -gy : gy;
            gz = (ax & 4) ? -gz : gz;
            out[k][0] += par * l[0];
            out[k][1] += par * gx;
            out[k][2] += par * gy;
            out[k][3] += par * gz;
        }
    }
}

// -------------------------------------------------------------- evaluation
// The elements of a tile that an evaluation starts work on: all but the second
// triangles of pairs.  Pairs are taken greedily from the tile's start, as a
// walk through the whole tile takes them, so that a walk through any part of it
// agrees.  first / second: bits of the pairs' elements.
__device__ __forceinline__ void tile_pairs(bool flag, uint64_t &first, uint64_t &second)
{
    uint64_t rem = __ballot(flag);
    first = 0;
    while (rem) {
        const uint64_t b = rem & (0 - rem);
        first |= b;
        rem &= ~(b | (b << 1));
    }
    second = first << 1;
}

// The first element at or after s0 that a walk through the tile (records rec,
// cnt of them) starts work on: s0, or s0 + 1 if s0 ends a pair.
__device__ __forceinline__ int first_start(cdouble_p rec, int cnt, int s0)
{
    if (s0 == 0) return 0;
    const int lane = threadIdx.x & 63;
    uint64_t first, second;
    tile_pairs(lane + 1 < cnt && rec[min(lane, cnt - 1) * R_STRIDE + R_KIND] >= 2.0, first, second);
    return s0 + (int)((second >> s0) & 1);
}

// One wave's share of an evaluation: its lanes' points of the m points, elements
// [p0, p1) of the n (records drec, densities sigma; p0 a multiple of kSubElems)
// and their copies, FP64 sums per lane; outputs scaled by `scale`.  Runs of
// kSubElems elements are summed on their own and then added up in order, so
// that launches which give every run its own wave (split evaluations)
// reproduce the same bits: 100 points between two plates of 256 elements, which
// two waves of 512 elements took 1.06 ms for, take 81 us as 64 waves.  With the
// records staged in LDS the runs made 10^6 points at 1152 elements 5 % slower
// (17.6 ms); from scalar loads it is 16.8 ms, as without runs.
template <bool MIXED, bool HOLE = false>
__device__ __forceinline__ void eval_block(const double *__restrict__ drec, const double *__restrict__ sigma, int n,
                                           int p0, int p1, const ImgArgs &img, double near_factor,
                                           const double *__restrict__ px, const double *__restrict__ py,
                                           const double *__restrict__ pz, int m, int i, double scale,
                                           double *__restrict__ phi, double *__restrict__ ex,
                                           double *__restrict__ ey, double *__restrict__ ez)
{
    const int j = min(i, m - 1);  // lanes past the last point repeat it
    const double Px = px[j], Py = py[j], Pz = pz[j];
    const cdouble_p recs = uniform_ptr(drec), sg = uniform_ptr(sigma);
    double aphi = 0.0, aex = 0.0, aey = 0.0, aez = 0.0;
    for (int base = p0 & ~(kTileE - 1); base < p1; base += kTileE) {
        const int cnt = min(kTileE, n - base), hi = min(cnt, p1 - base);
        const cdouble_p tile = recs + (int64_t)base * R_STRIDE, tsg = sg + base;
        int p = first_start(tile, cnt, max(0, p0 - base));
        for (int s0 = max(0, p0 - base); s0 < hi; s0 += kSubElems) {
            double sphi = 0.0, sex = 0.0, sey = 0.0, sez = 0.0;
            const int s1 = min(s0 + kSubElems, hi);
            while (p < s1) {
                const int kind = uni((int)tile[p * R_STRIDE + R_KIND]);
                if (kind >= 2 && p + 1 < cnt) {
                    // a triangle pair inside this tile, both in one pass (q1 is the pair's first)
                    const int q1 = kind == 2 ? p : p + 1, q2 = kind == 2 ? p + 1 : p;
                    const Elem e = load_elem_c(tile + q1 * R_STRIDE);
                    const PairB f = load_pair_b_c(tile + q2 * R_STRIDE);
                    if (MIXED) {  // sigma-weighted
                        const double sg1[1] = {tsg[q1]}, sg2[1] = {tsg[q2]};
                        double c[1][4];
                        element_pair_copies_mixed<1, HOLE>(e, f, sg1, sg2, img, near_factor, Px, Py, Pz, c);
                        sphi += c[0][0];
                        sex += c[0][1];
                        sey += c[0][2];
                        sez += c[0][3];
                    } else {  // c[0] for element p, c[1] for p + 1
                        double c[2][4];
                        element_pair_copies<HOLE>(e, f, img, Px, Py, Pz, c[q1 - p], c[q2 - p]);
                        const double g1 = tsg[p], g2 = tsg[p + 1];
                        sphi = fma(g2, c[1][0], fma(g1, c[0][0], sphi));
                        sex = fma(g2, c[1][1], fma(g1, c[0][1], sex));
                        sey = fma(g2, c[1][2], fma(g1, c[0][2], sey));
                        sez = fma(g2, c[1][3], fma(g1, c[0][3], sez));
                    }
                    p += 2;
                    continue;
                }
                double cp, cx, cy, cz;
                element_copies<MIXED, HOLE>(load_elem_c(tile + p * R_STRIDE), img, Px, Py, Pz, false, near_factor, cp,
                                            cx, cy, cz);
                const double g = tsg[p];
                sphi = fma(g, cp, sphi);
                sex = fma(g, cx, sex);
                sey = fma(g, cy, sey);
                sez = fma(g, cz, sez);
                ++p;
            }
            aphi += sphi;
            aex += sex;
            aey += sey;
            aez += sez;
        }
    }
    if (i < m) {
        if (phi) phi[i] = scale * aphi;
        if (ex) ex[i] = scale * aex;
        if (ey) ey[i] = scale * aey;
        if (ez) ez[i] = scale * aez;
    }
}

int64_t img_copies(const ImgArgs &img)
{
    int64_t t = (int64_t)(2 * img.n1 + 1) * (2 * img.n2 + 1);
    if (img.hole >= 0) {
        const int64_t h1 = img.hole < img.n1 ? img.hole : img.n1;
        const int64_t h2 = img.hole < img.n2 ? img.hole : img.n2;
        t -= (2 * h1 + 1) * (2 * h2 + 1);
    }
    return (int64_t)img.nref * t;
}

SegPlan seg_plan(int64_t n, const ImgArgs &img) { return seg_plan(n, img_copies(img)); }

// FP64: the default allocation (about 250 VGPRs, two waves per SIMD) keeps every
// value in registers; a three-wave target made the allocator spill part of
// the per-element setup to scratch (10.6 GB of HBM writes per 10^6-point
// launch) for no measurable gain.  HOLE: img.hole is honoured (a separate
// instantiation, so the plain launch carries no test for it).
// Grid: x over blocks of BS points, y over units -- element segments of segsz
// elements (units 1), or `units` runs of kSubElems elements per segment; unit y
// writes its sums (times `scale`) at outputs + y * seg_stride.
template <bool HOLE, int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_eval_fp64(
    const double *__restrict__ drec, const double *__restrict__ sigma, int n, int segsz, int units, ImgArgs img,
    double near_factor, const double *__restrict__ px, const double *__restrict__ py, const double *__restrict__ pz,
    int m, double scale, double *__restrict__ phi, double *__restrict__ ex, double *__restrict__ ey,
    double *__restrict__ ez, int64_t seg_stride)
{
    const int per = units, seg = blockIdx.y / per, e0 = seg * segsz;
    const int ns = min(segsz, n - e0), p0 = per > 1 ? (blockIdx.y % per) * kSubElems : 0;
    const size_t so = (size_t)blockIdx.y * (size_t)seg_stride;
    eval_block<false, HOLE>(drec + (size_t)e0 * R_STRIDE, sigma + e0, ns, p0, per > 1 ? min(p0 + kSubElems, ns) : ns,
                                img, near_factor, px, py, pz, m, blockIdx.x * BS + threadIdx.x, scale, phi ? phi + so : nullptr,
                                ex ? ex + so : nullptr, ey ? ey + so : nullptr, ez ? ez + so : nullptr);
}

// Mixed: two waves per SIMD (the triangle-pair path holds two triangles'
// unit-density sums and the pair's weighted ones at once; at three waves it
// spilled inside the copy loop).
template <bool HOLE, int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_eval_mixed(
    const double *__restrict__ drec, const double *__restrict__ sigma, int n, int segsz, int units, ImgArgs img,
    double near_factor, const double *__restrict__ px, const double *__restrict__ py, const double *__restrict__ pz,
    int m, double scale, double *__restrict__ phi, double *__restrict__ ex, double *__restrict__ ey,
    double *__restrict__ ez, int64_t seg_stride)
{
    const int per = units, seg = blockIdx.y / per, e0 = seg * segsz;
    const int ns = min(segsz, n - e0), p0 = per > 1 ? (blockIdx.y % per) * kSubElems : 0;
    const size_t so = (size_t)blockIdx.y * (size_t)seg_stride;
    eval_block<true, HOLE>(drec + (size_t)e0 * R_STRIDE, sigma + e0, ns, p0, per > 1 ? min(p0 + kSubElems, ns) : ns,
                                img, near_factor, px, py, pz, m, blockIdx.x * BS + threadIdx.x, scale, phi ? phi + so : nullptr,
                                ex ? ex + so : nullptr, ey ? ey + so : nullptr, ez ? ez + so : nullptr);
}

template <int BS>
static void launch_eval_bs(const double *drec, const double *sigma, int64_t n, const SegPlan &sp, const ImgArgs &img,
                           int mixed, double near_factor, int units, const double *px, const double *py,
                           const double *pz, int64_t m, double scale, double *phi, double *ex, double *ey, double *ez,
                           int64_t seg_stride, hipStream_t s)
{
    const dim3 g((unsigned)((m + BS - 1) / BS), (unsigned)(sp.nseg * units));
    const bool hole = img.hole >= 0;
    auto k = mixed ? (hole ? k_eval_mixed<true, BS> : k_eval_mixed<false, BS>)
                   : (hole ? k_eval_fp64<true, BS> : k_eval_fp64<false, BS>);
    hipLaunchKernelGGL(k, g, dim3(BS), 0, s, drec, sigma, (int)n, sp.segsz, units, img, near_factor, px, py, pz,
                       (int)m, scale, phi, ex, ey, ez, seg_stride);
}

void launch_eval_seg(const double *drec, const double *sigma, int64_t n, const SegPlan &sp, const ImgArgs &img,
                     int mixed, double near_factor, bool split, const double *px, const double *py, const double *pz,
                     int64_t m, double scale, double *phi, double *ex, double *ey, double *ez, int64_t seg_stride,
                     hipStream_t s)
{
    if (m <= 0 || n <= 0) return;
    if (split)
        launch_eval_bs<64>(drec, sigma, n, sp, img, mixed, near_factor, eval_subunits(sp), px, py, pz, m, scale, phi,
                           ex, ey, ez, seg_stride, s);
    else
        launch_eval_bs<kBlock>(drec, sigma, n, sp, img, mixed, near_factor, 1, px, py, pz, m, scale, phi, ex, ey, ez,
                               seg_stride, s);
}

// out[c][i] += add[c m + i] for the non-null outputs
__global__ __launch_bounds__(kBlock) void k_add4(const double *__restrict__ add, int m, double *__restrict__ o0,
                                                 double *__restrict__ o1, double *__restrict__ o2,
                                                 double *__restrict__ o3)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= m) return;
    const size_t mm = (size_t)m;
    if (o0) o0[i] += add[i];
    if (o1) o1[i] += add[mm + i];
    if (o2) o2[i] += add[2 * mm + i];
    if (o3) o3[i] += add[3 * mm + i];
}

void launch_add4(const double *add, int64_t m, double *o0, double *o1, double *o2, double *o3, hipStream_t s)
{
    if (m <= 0) return;
    hipLaunchKernelGGL(k_add4, dim3((unsigned)((m + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, add, (int)m, o0, o1,
                       o2, o3);
}

// Primitive-averaged densities (Adaptive Modelling): sbar[p] = (sum of
// sigma_j A_j over the elements j with map[j] == p, in element order) / A_p.
// The elements are first sorted by primitive (stable radix sort of
// (map[j], j)); then one lane per primitive finds its run by binary search
// and sums it in order -- O(n log n) work instead of every lane scanning all
// n elements, the same sums bit for bit.  *bad is set when a map entry is
// outside [0, np) (such an element is sorted past every primitive).
__global__ __launch_bounds__(kBlock) void k_prim_keys(const int32_t *__restrict__ map, int n, int np,
                                                      unsigned *__restrict__ key, int *__restrict__ idx,
                                                      int *__restrict__ bad)
{
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= n) return;
    const int mj = map[j];
    const bool ok = mj >= 0 && mj < np;
    if (!ok) bad[0] = 1;
    key[j] = ok ? (unsigned)mj : (unsigned)np;
    idx[j] = j;
}

__device__ __forceinline__ int lower_bound_u(const unsigned *__restrict__ a, int n, unsigned v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(kBlock) void k_prim_density(const double *__restrict__ drec,
                                                         const double *__restrict__ sigma,
                                                         const unsigned *__restrict__ key,
                                                         const int *__restrict__ idx, int n,
                                                         const double *__restrict__ prec, int np,
                                                         double *__restrict__ sbar)
{
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= np) return;
    const int s0 = lower_bound_u(key, n, (unsigned)p), s1 = lower_bound_u(key, n, (unsigned)p + 1u);
    double q = 0.0;
    for (int s = s0; s < s1; ++s) {
        const int j = idx[s];
        q = fma(sigma[j], drec[(size_t)j * R_STRIDE + R_AREA], q);
    }
    sbar[p] = q / prec[(size_t)p * R_STRIDE + R_AREA];
}

size_t prim_density_workspace(int64_t n)
{
    size_t sort_b = 0;
    if (rocprim::radix_sort_pairs(nullptr, sort_b, (unsigned *)nullptr, (unsigned *)nullptr, (int *)nullptr,
                                  (int *)nullptr, (int)n, 0u, 32u) != hipSuccess)
        return 0;
    const size_t a = ((size_t)(n > 0 ? n : 1) * 4 + 255) & ~(size_t)255;
    return 4 * a + sort_b;
}

hipError_t launch_prim_density(const double *drec, const double *sigma, const int32_t *map, int64_t n,
                               const double *prec, int64_t np, double *sbar, int *bad, void *ws, size_t ws_bytes,
                               hipStream_t s)
{
    if (np <= 0 || n <= 0) return hipSuccess;
    const size_t need = prim_density_workspace(n);
    if (!need || !ws || ws_bytes < need) return hipErrorInvalidValue;
    const size_t a = ((size_t)n * 4 + 255) & ~(size_t)255;
    char *w = static_cast<char *>(ws);
    unsigned *kin = reinterpret_cast<unsigned *>(w), *kout = reinterpret_cast<unsigned *>(w + a);
    int *iin = reinterpret_cast<int *>(w + 2 * a), *iout = reinterpret_cast<int *>(w + 3 * a);
    const unsigned gn = (unsigned)((n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_prim_keys, dim3(gn), dim3(kBlock), 0, s, map, (int)n, (int)np, kin, iin, bad);
    size_t sort_b = need - 4 * a;
    hipError_t e = rocprim::radix_sort_pairs(w + 4 * a, sort_b, kin, kout, iin, iout, (int)n, 0u, 32u, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_prim_density, dim3((unsigned)((np + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, drec, sigma,
                       kout, iout, (int)n, prec, (int)np, sbar);
    return hipGetLastError();
}

// ------------------------------------------------- several sigma columns
// Weighting fields: K density columns over the same elements and points
// (column k of sigma at sigma + k n).  Each element's copies are summed once
// per point (the closed forms do not depend on sigma) and the K columns take
// their own FP64 sums in the same fixed order as eval_block, so column k's
// results equal a single-column evaluation with that column bit for bit.
// Output (component c, column k) goes to out[c] + k * ostride (out[c] may be
// null: that component is not stored).
template <bool MIXED, int K, int BS>
__device__ __forceinline__ void eval_block_multi(const double *__restrict__ drec, const double *__restrict__ sigma,
                                                 int n, int p0, int p1, int64_t sig_stride, const ImgArgs &img,
                                                 double near_factor, const double *__restrict__ px,
                                                 const double *__restrict__ py, const double *__restrict__ pz, int m,
                                                 int i, double scale, OutCols out)
{
    __shared__ double t_acc[K][4][BS];  // each lane's sums over runs: touched once per run
    const int j = min(i, m - 1);
    const double Px = px[j], Py = py[j], Pz = pz[j];
    const cdouble_p recs = uniform_ptr(drec), sg = uniform_ptr(sigma);
    for (int k = 0; k < K; ++k)
        for (int q = 0; q < 4; ++q) t_acc[k][q][threadIdx.x] = 0.0;
    for (int base = p0 & ~(kTileE - 1); base < p1; base += kTileE) {
        const int cnt = min(kTileE, n - base), hi = min(cnt, p1 - base);
        const cdouble_p tile = recs + (int64_t)base * R_STRIDE, tsg = sg + base;
        int p = first_start(tile, cnt, max(0, p0 - base));
        for (int s0 = max(0, p0 - base); s0 < hi; s0 += kSubElems) {
            double sub[K][4];
#pragma unroll
            for (int k = 0; k < K; ++k) sub[k][0] = sub[k][1] = sub[k][2] = sub[k][3] = 0.0;
            const int s1 = min(s0 + kSubElems, hi);
            while (p < s1) {
                const int kind = uni((int)tile[p * R_STRIDE + R_KIND]);
                if (kind >= 2 && p + 1 < cnt) {
                    // a triangle pair inside this tile, as in eval_block
                    const int q1 = kind == 2 ? p : p + 1, q2 = kind == 2 ? p + 1 : p;
                    const Elem e = load_elem_c(tile + q1 * R_STRIDE);
                    const PairB f = load_pair_b_c(tile + q2 * R_STRIDE);
                    if (MIXED) {
                        double sg1[K], sg2[K], c[K][4];
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            sg1[k] = tsg[k * sig_stride + q1];
                            sg2[k] = tsg[k * sig_stride + q2];
                        }
                        element_pair_copies_mixed<K, false>(e, f, sg1, sg2, img, near_factor, Px, Py, Pz, c);
#pragma unroll
                        for (int k = 0; k < K; ++k)
#pragma unroll
                            for (int q = 0; q < 4; ++q) sub[k][q] += c[k][q];
                    } else {
                        double c[2][4];
                        element_pair_copies<false>(e, f, img, Px, Py, Pz, c[q1 - p], c[q2 - p]);
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            const double g1 = tsg[k * sig_stride + p], g2 = tsg[k * sig_stride + p + 1];
#pragma unroll
                            for (int q = 0; q < 4; ++q) sub[k][q] = fma(g2, c[1][q], fma(g1, c[0][q], sub[k][q]));
                        }
                    }
                    p += 2;
                    continue;
                }
                double cc[4];
                element_copies<MIXED>(load_elem_c(tile + p * R_STRIDE), img, Px, Py, Pz, false, near_factor, cc[0],
                                      cc[1], cc[2], cc[3]);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const double g = tsg[k * sig_stride + p];
#pragma unroll
                    for (int q = 0; q < 4; ++q) sub[k][q] = fma(g, cc[q], sub[k][q]);
                }
                ++p;
            }
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int q = 0; q < 4; ++q) t_acc[k][q][threadIdx.x] += sub[k][q];
        }
    }
    if (i < m) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const size_t o = (size_t)k * out.stride + i;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (out.c[q]) out.c[q][o] = scale * t_acc[k][q][threadIdx.x];
        }
    }
}

// outputs of segment `seg`: every stored component moved by seg * seg_stride
__device__ __forceinline__ OutCols seg_out(OutCols o, int seg, int64_t seg_stride)
{
    const size_t so = (size_t)seg * (size_t)seg_stride;
#pragma unroll
    for (int c = 0; c < 4; ++c) o.c[c] = o.c[c] ? o.c[c] + so : nullptr;
    return o;
}

// grid as k_eval_fp64: x over point blocks, y over units
template <int K, int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_eval_multi_fp64(const double *__restrict__ drec,
                                                        const double *__restrict__ sigma, int n, int64_t sig_stride,
                                                        int segsz, int units, ImgArgs img, double near_factor,
                                                        const double *__restrict__ px, const double *__restrict__ py,
                                                        const double *__restrict__ pz, int m, double scale,
                                                        OutCols out, int64_t seg_stride)
{
    const int per = units, e0 = (blockIdx.y / per) * segsz;
    const int ns = min(segsz, n - e0), p0 = per > 1 ? (blockIdx.y % per) * kSubElems : 0;
    eval_block_multi<false, K, BS>(drec + (size_t)e0 * R_STRIDE, sigma + e0, ns, p0,
                                   per > 1 ? min(p0 + kSubElems, ns) : ns, sig_stride, img, near_factor, px, py, pz, m,
                                   blockIdx.x * BS + threadIdx.x, scale, seg_out(out, blockIdx.y, seg_stride));
}

// at most 256 VGPRs so that two waves share a SIMD (unbounded, K = 3 and 4
// would take 258 and 266)
template <int K, int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_eval_multi_mixed(
    const double *__restrict__ drec, const double *__restrict__ sigma, int n, int64_t sig_stride, int segsz, int units,
    ImgArgs img, double near_factor, const double *__restrict__ px, const double *__restrict__ py,
    const double *__restrict__ pz, int m, double scale, OutCols out, int64_t seg_stride)
{
    const int per = units, e0 = (blockIdx.y / per) * segsz;
    const int ns = min(segsz, n - e0), p0 = per > 1 ? (blockIdx.y % per) * kSubElems : 0;
    eval_block_multi<true, K, BS>(drec + (size_t)e0 * R_STRIDE, sigma + e0, ns, p0,
                                  per > 1 ? min(p0 + kSubElems, ns) : ns, sig_stride, img, near_factor, px, py, pz, m,
                                  blockIdx.x * BS + threadIdx.x, scale, seg_out(out, blockIdx.y, seg_stride));
}

template <int K, int BS>
static void launch_multi_k(const double *drec, const double *sigma, int n, int64_t sig_stride, const SegPlan &sp,
                           const ImgArgs &img, int mixed, double near_factor, int units, const double *px,
                           const double *py, const double *pz, int m, double scale, const OutCols &out,
                           int64_t seg_stride, hipStream_t s)
{
    const dim3 g((unsigned)((m + BS - 1) / BS), (unsigned)(sp.nseg * units));
    if (mixed)
        hipLaunchKernelGGL((k_eval_multi_mixed<K, BS>), g, dim3(BS), 0, s, drec, sigma, n, sig_stride, sp.segsz, units,
                           img, near_factor, px, py, pz, m, scale, out, seg_stride);
    else
        hipLaunchKernelGGL((k_eval_multi_fp64<K, BS>), g, dim3(BS), 0, s, drec, sigma, n, sig_stride, sp.segsz, units,
                           img, near_factor, px, py, pz, m, scale, out, seg_stride);
}

template <int BS>
static void launch_multi_bs(const double *drec, const double *sigma, int n, int64_t sig_stride, int ncol,
                            const SegPlan &sp, const ImgArgs &img, int mixed, double near_factor, int units,
                            const double *px, const double *py, const double *pz, int m, double scale,
                            const OutCols &out, int64_t seg_stride, hipStream_t s)
{
#define MULTI_ARGS drec, sigma, n, sig_stride, sp, img, mixed, near_factor, units, px, py, pz, m, scale, out, seg_stride, s
    switch (ncol) {
    case 1: launch_multi_k<1, BS>(MULTI_ARGS); break;
    case 2: launch_multi_k<2, BS>(MULTI_ARGS); break;
    case 3: launch_multi_k<3, BS>(MULTI_ARGS); break;
    default: launch_multi_k<4, BS>(MULTI_ARGS); break;
    }
#undef MULTI_ARGS
}

void launch_eval_multi_seg(const double *drec, const double *sigma, int64_t n, int64_t sig_stride, int ncol,
                           const SegPlan &sp, const ImgArgs &img, int mixed, double near_factor, bool split,
                           const double *px, const double *py, const double *pz, int64_t m, double scale,
                           const OutCols &out, int64_t seg_stride, hipStream_t s)
{
    if (m <= 0 || ncol <= 0 || n <= 0) return;
    if (split)
        launch_multi_bs<64>(drec, sigma, (int)n, sig_stride, ncol, sp, img, mixed, near_factor, eval_subunits(sp), px,
                            py, pz, (int)m, scale, out, seg_stride, s);
    else
        launch_multi_bs<kBlock>(drec, sigma, (int)n, sig_stride, ncol, sp, img, mixed, near_factor, 1, px, py, pz,
                                (int)m, scale, out, seg_stride, s);
}

// Segment partial sums -> results: for column k < ncol and component c,
// out.c[c][k * out.stride + i] = k_e (0 + sum over s = 0 .. nseg-1, in that
// order, of part[s * seg_stride + (4 k + c) m + i]); null components skipped.
__global__ __launch_bounds__(kBlock) void k_reduce_segments(const double *__restrict__ part, int nseg, int ncol,
                                                             int m, int64_t seg_stride, OutCols out)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= m) return;
    for (int k = 0; k < ncol; ++k)
        for (int c = 0; c < 4; ++c) {
            if (!out.c[c]) continue;
            const double *p = part + (size_t)(4 * k + c) * m + i;
            double acc = 0.0;
            for (int s = 0; s < nseg; ++s) acc += p[(size_t)s * (size_t)seg_stride];
            out.c[c][(size_t)k * out.stride + i] = kKe * acc;
        }
}

void launch_reduce_segments(const double *part, int nseg, int ncol, int64_t m, int64_t seg_stride,
                            const OutCols &out, hipStream_t s)
{
    if (m <= 0) return;
    hipLaunchKernelGGL(k_reduce_segments, dim3((unsigned)((m + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, part, nseg,
                       ncol, (int)m, seg_stride, out);
}

// ------------------------------------------------- grouped FP64: near part
// The copies of a group that are nearer to a point than the expansion's
// range (group_far.hpp), element by element with the closed forms.  Per wave,
// group and chunk of copies: a first loop tests every copy with the far
// pass's own arithmetic and lists those that are near for any lane, with the
// mask of the lanes they are near for; then each element (or triangle pair)
// of the group walks the listed copies only.  The list is the wave's own (LDS,
// no workgroup barrier), and the records come through scalar loads: with a
// few copies per element, staging them in LDS and moving them to scalar
// registers would cost as much as the closed forms.
constexpr int kNearCopies = 128;  // copies per list, 3 KB a wave

// one copy by the closed forms (tiers of sum_translations), added to s
template <int KIND>
__device__ __forceinline__ void copy_fp64(const Elem &e, double X, double Z, double H, double far2, double vfar2,
                                          double (&s)[4])
{
    Kern k;
    const double r0sq = fma(X, X, fma(Z, Z, H * H));
    if (r0sq >= vfar2) {
        k = KIND == 0 ? rect_far<true>(X, H, Z, e.lx, e.lz, r0sq, s[0])
                      : rtri_far<true>(X, H, Z, e.lx, e.lz, e.hyp, r0sq, s[0]);
    } else if (r0sq >= far2) {
        k = KIND == 0 ? rect_far<false>(X, H, Z, e.lx, e.lz, r0sq, s[0])
                      : rtri_far<false>(X, H, Z, e.lx, e.lz, e.hyp, r0sq, s[0]);
    } else {
        k = KIND == 0 ? rect_fp64(X, H, Z, e.lx, e.lz, r0sq)
                      : rtri_fp64(X, H, Z, e.lx, e.lz, e.hyp, e.ihyp, r0sq);
        k.phi += s[0];
    }
    s[0] = k.phi;
    s[1] += k.ex;
    s[2] += k.ez;
    s[3] += k.en;
}

// the same for both triangles of a pair, in the first one's frame
__device__ __forceinline__ void pair_copy_fp64(const Elem &e, const PairB &f, double X, double Z, double H,
                                               double far2, double vfar2, double (&s1)[4], double (&s2)[4])
{
    const double r0sq = fma(X, X, fma(Z, Z, H * H));
    Kern k1, k2;
    if (r0sq >= vfar2) {
        rtri_pair_far<true>(X, H, Z, e.lx, f.lz, e.lz, e.hyp, f.hyp, r0sq, s1[0], s2[0], k1, k2);
    } else if (r0sq >= far2) {
        rtri_pair_far<false>(X, H, Z, e.lx, f.lz, e.lz, e.hyp, f.hyp, r0sq, s1[0], s2[0], k1, k2);
    } else {
        k1 = rtri_fp64(X, H, Z, e.lx, e.lz, e.hyp, e.ihyp, r0sq);
        k2 = rtri_fp64(Z, H, -X, e.lz, f.lz, f.hyp, f.ihyp, r0sq);
        k1.phi += s1[0];
        k2.phi += s2[0];
    }
    s1[0] = k1.phi;
    s1[1] += k1.ex;
    s1[2] += k1.ez;
    s1[3] += k1.en;
    s2[0] = k2.phi;
    s2[1] += k2.ex;
    s2[2] += k2.ez;
    s2[3] += k2.en;
}

// A wave's list of near copies: translations as the factors of a1, a2, the
// lanes they are near for, and where each reflection's entries begin.
struct NearList {
    double f1[kNearCopies], f2[kNearCopies];
    uint64_t lanes[kNearCopies];
    int begin[9];
};

// copies [c0, c1) (reflection-major, then i1, i2) of the group with header h
__device__ __forceinline__ int list_near(NearList &nl, cdouble_p h, const ImgArgs &img, int c0, int c1, double Px,
                                         double Py, double Pz)
{
    const int w2 = 2 * img.n2 + 1, per = (2 * img.n1 + 1) * w2;
    int cnt = 0;
    for (int r = 0; r < img.nref; ++r) {
        nl.begin[r] = cnt;
        const int lo = max(c0 - r * per, 0), hi = min(c1 - r * per, per);
        if (lo >= hi) continue;
        const GroupVec v0 = group_origin(img, img.axes[r], Px, Py, Pz, h);
        int i1 = lo / w2 - img.n1, i2 = lo % w2 - img.n2;
        GroupVec v1 = group_step(v0, -(double)i1, img.a1[r]);
#pragma unroll 1
        for (int q = lo; q < hi; ++q) {
            const double r2 = group_r2(group_step(v1, -(double)i2, img.a2[r]));
            uint64_t b = __ballot(!(r2 >= h[kHeadTier]));
            if (b) b &= ~__ballot(super_far(img, r, i1, i2, Px, Py, Pz, h));
            if (b) {
                nl.f1[cnt] = -(double)i1;
                nl.f2[cnt] = -(double)i2;
                nl.lanes[cnt] = b;
                ++cnt;
            }
            if (++i2 > img.n2) {
                i2 = -img.n2;
                ++i1;
                v1 = group_step(v0, -(double)i1, img.a1[r]);
            }
        }
    }
    nl.begin[img.nref] = cnt;
    return cnt;
}

// The 64ths of a lattice of more copies than a list holds, in whole chunks of
// kNearCopies, that have near copies of the group with header h: the lists are made
// anew for each run of its elements, but only where there is something to list.
// 16 641 copies (1648 elements, 40 000 points): 768 ms with every list made for every
// run, 591 with these alone; 441 copies (20 000 points) 18.3, 16.6.  (One list of 256
// for all chunks: 608 ms, and calls of fewer than 128 copies 1 to 3 % longer.)
__device__ __forceinline__ int chunk_bit(int c, int ncopy)
{
    return (int)((unsigned)(c / kNearCopies) * 64u / (unsigned)((ncopy + kNearCopies - 1) / kNearCopies));
}
__device__ __forceinline__ uint64_t near_chunks(cdouble_p h, const ImgArgs &img, int ncopy, double Px, double Py,
                                                double Pz)
{
    const int w2 = 2 * img.n2 + 1;
    uint64_t have = 0;
    int c = 0;
    for (int r = 0; r < img.nref; ++r) {
        const GroupVec v0 = group_origin(img, img.axes[r], Px, Py, Pz, h);
#pragma unroll 1
        for (int i1 = -img.n1; i1 <= img.n1; ++i1, c += w2) {
            const GroupVec v1 = group_step(v0, -(double)i1, img.a1[r]);
            int lo = w2, hi = -1;  // the row's near copies
#pragma unroll 1
            for (int q = 0; q < w2; ++q)
                if (__ballot(!(group_r2(group_step(v1, -(double)(q - img.n2), img.a2[r])) >= h[kHeadTier]))) {
                    lo = min(lo, q);
                    hi = q;
                }
            if (hi < 0) continue;
            const int b0 = chunk_bit(c + lo, ncopy), b1 = chunk_bit(c + hi, ncopy);
            have |= (~(uint64_t)0 << b0) & (~(uint64_t)0 >> (63 - b1));
        }
    }
    return have;
}

// One element, or pair of triangles, over the listed copies: adds
// sum_k density x (phi', E') to acc.
template <int K, bool PAIR>
__device__ __forceinline__ void near_element(const NearList &nl, const Elem &e, const PairB &f, const double (&sg1)[K],
                                             const double (&sg2)[K], const ImgArgs &img, double Px, double Py,
                                             double Pz, double (&acc)[K][4])
{
    const double dp = PAIR ? fmax(e.diam, f.diam) : e.diam;
    const double far2 = (kFarDiam * kFarDiam) * (dp * dp), vfar2 = (kVeryFarDiam * kVeryFarDiam) * (dp * dp);
#pragma unroll 1
    for (int r = 0; r < img.nref; ++r) {
        const int lo = uni(nl.begin[r]), hi = uni(nl.begin[r + 1]);
        if (lo >= hi) continue;
        const int ax = img.axes[r];
        const double Qx = (ax & 1) ? 2.0 * img.mpos[0] - Px : Px;
        const double Qy = (ax & 2) ? 2.0 * img.mpos[1] - Py : Py;
        const double Qz = (ax & 4) ? 2.0 * img.mpos[2] - Pz : Pz;
        const double rx = Qx - e.ox, ry = Qy - e.oy, rz = Qz - e.oz;
        const double X0 = rx * e.e1x + ry * e.e1y + rz * e.e1z;
        const double Z0 = rx * e.e2x + ry * e.e2y + rz * e.e2z;
        const double H0 = rx * e.e3x + ry * e.e3y + rz * e.e3z;
        const double *a = img.a1[r], *b = img.a2[r];
        const double aX = a[0] * e.e1x + a[1] * e.e1y + a[2] * e.e1z;
        const double aZ = a[0] * e.e2x + a[1] * e.e2y + a[2] * e.e2z;
        const double aH = a[0] * e.e3x + a[1] * e.e3y + a[2] * e.e3z;
        const double bX = b[0] * e.e1x + b[1] * e.e1y + b[2] * e.e1z;
        const double bZ = b[0] * e.e2x + b[1] * e.e2y + b[2] * e.e2z;
        const double bH = b[0] * e.e3x + b[1] * e.e3y + b[2] * e.e3z;
        double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int l = lo; l < hi; ++l) {
            const double f1 = nl.f1[l], f2 = nl.f2[l];
            // the mask itself as the branch's lanes, no test in each: on a mesh in random order,
            // where all groups are wide and all copies near, the lists took 249.5 ms where
            // closed forms without them take 247.1, now 246.7 (THGEM, 9 copies, 200 000 points)
            const uint64_t lanes = nl.lanes[l];
            if (__builtin_amdgcn_inverse_ballot_w64(((uint64_t)(unsigned)uni((int)(lanes >> 32)) << 32) |
                                                    (unsigned)uni((int)lanes))) {
                const double X = fma(f2, bX, fma(f1, aX, X0)), Z = fma(f2, bZ, fma(f1, aZ, Z0)),
                             H = fma(f2, bH, fma(f1, aH, H0));
                if (PAIR)
                    pair_copy_fp64(e, f, X, Z, H, far2, vfar2, s1, s2);
                else if (e.kind == 0)
                    copy_fp64<0>(e, X, Z, H, far2, vfar2, s1);
                else
                    copy_fp64<1>(e, X, Z, H, far2, vfar2, s1);
            }
        }
        const double par = img.parity[r];
        const double px = (ax & 1) ? -par : par, py = (ax & 2) ? -par : par, pz = (ax & 4) ? -par : par;
        const double p1 = par * s1[0];
        const double x1 = px * fma(s1[1], e.e1x, fma(s1[2], e.e2x, s1[3] * e.e3x));
        const double y1 = py * fma(s1[1], e.e1y, fma(s1[2], e.e2y, s1[3] * e.e3y));
        const double z1 = pz * fma(s1[1], e.e1z, fma(s1[2], e.e2z, s1[3] * e.e3z));
#pragma unroll
        for (int k = 0; k < K; ++k) {
            acc[k][0] = fma(sg1[k], p1, acc[k][0]);
            acc[k][1] = fma(sg1[k], x1, acc[k][1]);
            acc[k][2] = fma(sg1[k], y1, acc[k][2]);
            acc[k][3] = fma(sg1[k], z1, acc[k][3]);
        }
        if (PAIR) {  // second triangle: frame (e2, -e1, e3)
            const double p2 = par * s2[0];
            const double x2 = px * fma(s2[1], e.e2x, fma(-s2[2], e.e1x, s2[3] * e.e3x));
            const double y2 = py * fma(s2[1], e.e2y, fma(-s2[2], e.e1y, s2[3] * e.e3y));
            const double z2 = pz * fma(s2[1], e.e2z, fma(-s2[2], e.e1z, s2[3] * e.e3z));
#pragma unroll
            for (int k = 0; k < K; ++k) {
                acc[k][0] = fma(sg2[k], p2, acc[k][0]);
                acc[k][1] = fma(sg2[k], x2, acc[k][1]);
                acc[k][2] = fma(sg2[k], y2, acc[k][2]);
                acc[k][3] = fma(sg2[k], z2, acc[k][3]);
            }
        }
    }
}

// Near copies of groups [g0, g1) of one segment (records drec, densities
// sigma of the segment's n elements), runs [u0, u1) of each group:
// runs added into the group's sum, groups into acc, in that order.
template <int K>
__device__ __forceinline__ void near_unit(NearList &nl, cdouble_p drec, cdouble_p sigma, int64_t sig_stride,
                                          cdouble_p gd, int n, const ImgArgs &img, double Px, double Py, double Pz,
                                          int g0, int g1, int u0, int u1, double (&acc)[K][4])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[k][c] = 0.0;
    const int ncopy = img.nref * (2 * img.n1 + 1) * (2 * img.n2 + 1);
#pragma unroll 1
    for (int g = g0; g < g1; ++g) {
        cdouble_p h = gd + (int64_t)g * kGroupStride;
        const int e0 = g * kGroupElems, cnt = min(kGroupElems, n - e0);
        int listed = -1;
        uint64_t chunks = ~(uint64_t)0;  // which 64ths of a lattice of several lists have near copies
        if (ncopy <= kNearCopies) {
            listed = list_near(nl, h, img, 0, ncopy, Px, Py, Pz);
            if (listed == 0) continue;
        } else if (u1 - u0 > 1) {
            chunks = near_chunks(h, img, ncopy, Px, Py, Pz);
            if (chunks == 0) continue;
        }
        uint64_t first, second;
        tile_pairs(lane + 1 < cnt && drec[(int64_t)(e0 + min(lane, cnt - 1)) * R_STRIDE + R_KIND] >= 2.0, first,
                   second);
        double grp[K][4];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) grp[k][c] = 0.0;
#pragma unroll 1
        for (int u = u0; u < u1; ++u) {
            double sub[K][4];
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int c = 0; c < 4; ++c) sub[k][c] = 0.0;
#pragma unroll 1
            for (int c0 = 0; c0 < ncopy; c0 += kNearCopies) {
                if (ncopy > kNearCopies)
                    listed = (chunks >> chunk_bit(c0, ncopy)) & 1
                                 ? list_near(nl, h, img, c0, min(c0 + kNearCopies, ncopy), Px, Py, Pz)
                                 : 0;
                if (listed == 0) continue;
                const int i1 = min((u + 1) * kRunElems, cnt);
#pragma unroll 1
                for (int i = u * kRunElems; i < i1; ++i) {
                    if ((second >> i) & 1) continue;
                    cdouble_p p = drec + (int64_t)(e0 + i) * R_STRIDE;
                    const bool pair = (first >> i) & 1;
                    double sg1[K], sg2[K];
                    if (pair) {
                        const bool fst = uni((int)p[R_KIND]) == 2;  // the pair's first triangle is element i
                        cdouble_p pf = p + (fst ? 0 : R_STRIDE), ps = p + (fst ? R_STRIDE : 0);
                        const PairB f = {ps[R_LZ], ps[R_HYP], ps[R_IHYP], ps[R_DIAM], ps[R_AREA]};
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            sg1[k] = sigma[k * sig_stride + e0 + i + (fst ? 0 : 1)];
                            sg2[k] = sigma[k * sig_stride + e0 + i + (fst ? 1 : 0)];
                        }
                        near_element<K, true>(nl, load_elem_c(pf), f, sg1, sg2, img, Px, Py, Pz, sub);
                    } else {
#pragma unroll
                        for (int k = 0; k < K; ++k) sg1[k] = sg2[k] = sigma[k * sig_stride + e0 + i];
                        near_element<K, false>(nl, load_elem_c(p), PairB{}, sg1, sg2, img, Px, Py, Pz, sub);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int c = 0; c < 4; ++c) grp[k][c] += sub[k][c];
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k][c] += grp[k][c];
    }
}

// Unit y of a near pass: groups [g0, g1) and runs [u0, u1) of a segment.
struct NearRange {
    int seg, ns, g0, g1, u0, u1;
};
__device__ __forceinline__ NearRange near_range(int y, int n, int segsz, int gps, int split, const int *order)
{
    NearRange r = {0, 0, 0, 0, 0, kNearRuns};
    if (split == 2) {
        r.u0 = y % kNearRuns;
        r.u1 = r.u0 + 1;
        y /= kNearRuns;
    }
    r.seg = split ? y / gps : order[y];
    r.ns = min(segsz, n - r.seg * segsz);
    const int ng = (r.ns + kGroupElems - 1) / kGroupElems;
    r.g0 = split ? y % gps : 0;
    r.g1 = split ? min(r.g0 + 1, ng) : ng;
    return r;
}
__device__ __forceinline__ bool columns_differ(cdouble_p gd, const NearRange &r)
{
    bool d = false;
    for (int g = r.g0; g < r.g1; ++g) d = d || gd[(int64_t)g * kGroupStride + kHeadDiffer] != 0.0;
    return d;
}

// Grid: x over points, y over units -- segments (split 0: added to the far
// pass's sums), groups (split 1) or runs of 8 of their elements (split
// 2: with runs of 16 the near pass of 64 points took 505 us, with 8 280, with 4 158, but
// 2003 points 1.34, 1.30 and 1.45 ms: each unit scans the lattice anew).
// The columns share column 0's walk through the near copies, unless a density is not
// finite in some of them only, and with it what is near differs (kHeadDiffer):
// then the others are left to k_near_columns.
template <int K>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_group_near(const double *__restrict__ drec,
                                                       const double *__restrict__ sigma,
                                                       const double *__restrict__ gdata, int n, int64_t sig_stride,
                                                       int segsz, int gps, int rps, ImgArgs img, int split,
                                                       const int *__restrict__ order,
                                                       const double *__restrict__ px, const double *__restrict__ py,
                                                       const double *__restrict__ pz, int m, OutCols out,
                                                       int64_t unit_stride)
{
    __shared__ NearList list;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = min(i, m - 1);
    const NearRange r = near_range(blockIdx.y, n, segsz, gps, split, order);
    const cdouble_p gd = uniform_ptr(gdata + (int64_t)r.seg * rps * kGroupStride);
    double acc[K][4];
    near_unit<K>(list, uniform_ptr(drec + (int64_t)r.seg * segsz * R_STRIDE),
                 uniform_ptr(sigma + (int64_t)r.seg * segsz), sig_stride, gd, r.ns, img, px[j], py[j], pz[j], r.g0, r.g1,
                 r.u0, r.u1, acc);
    const bool only0 = K > 1 && columns_differ(gd, r);
    if (i >= m) return;
    const int64_t o = (int64_t)(split ? (int)blockIdx.y : r.seg) * unit_stride + i;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (out.c[c] && !(k > 0 && only0)) {
                double *d = out.c[c] + o + k * out.stride;
                *d = split ? acc[k][c] : *d + acc[k][c];
            }
}

// Columns 1 .. ncol - 1 of the units in which they differ from column 0, by
// their own records (column k's at gdata + k gstride).  Mostly there are none, and the
// launch ends with the scan of the groups' flags: 4.6 us of the 4.0 ms of three columns
// at 4507 points.  (With this in k_group_near, as a loop or as workgroups of their
// own, that call took 1 to 2 % longer.)
__global__ __launch_bounds__(64) void k_near_columns(const double *__restrict__ drec, const double *__restrict__ sigma,
                                                     const double *__restrict__ gdata, int64_t gstride, int n,
                                                     int64_t sig_stride, int ncol, int nseg, int segsz, int gps, int rps,
                                                     ImgArgs img, int split, int units, const int *__restrict__ order,
                                                     const double *__restrict__ px, const double *__restrict__ py,
                                                     const double *__restrict__ pz, int m, OutCols out,
                                                     int64_t unit_stride)
{
    __shared__ NearList list;
    bool any = false;
    for (int g = threadIdx.x; g < nseg * gps; g += 64) {
        const int seg = g / gps, q = g % gps;
        if (seg * segsz + q * kGroupElems < min(n, (seg + 1) * segsz))
            any = any || gdata[((int64_t)seg * rps + q) * kGroupStride + kHeadDiffer] != 0.0;
    }
    if (__ballot(any) == 0) return;
    const int blocks = (m + 63) / 64;
    const int64_t items = (int64_t)units * blocks * (ncol - 1);
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int k = 1 + (int)(it % (ncol - 1));
        const int64_t v = it / (ncol - 1);
        const int y = (int)(v / blocks), i = (int)(v % blocks) * 64 + (int)threadIdx.x, j = min(i, m - 1);
        const NearRange r = near_range(y, n, segsz, gps, split, order);
        const double *g = gdata + (int64_t)r.seg * rps * kGroupStride;
        if (!columns_differ(uniform_ptr(g), r)) continue;
        double acc[1][4];
        near_unit<1>(list, uniform_ptr(drec + (int64_t)r.seg * segsz * R_STRIDE),
                     uniform_ptr(sigma + k * sig_stride + (int64_t)r.seg * segsz), 0, uniform_ptr(g + k * gstride), r.ns,
                     img, px[j], py[j], pz[j], r.g0, r.g1, r.u0, r.u1, acc);
        if (i >= m) continue;
        const int64_t o = (int64_t)(split ? y : r.seg) * unit_stride + k * out.stride + i;
        for (int c = 0; c < 4; ++c)
            if (out.c[c]) out.c[c][o] = split ? acc[0][c] : out.c[c][o] + acc[0][c];
    }
}

template <int K>
static void launch_near_k(const double *drec, const double *sigma, const double *gdata, int64_t n, int64_t sig_stride,
                          const SegPlan &sp, const ImgArgs &img, int split, const int *order, const double *px, const double *py,
                          const double *pz, int64_t m, const OutCols &out, int64_t unit_stride, hipStream_t s)
{
    const int gps = groups_per_seg(sp), rps = records_per_seg(sp);
    const int64_t ng = (int64_t)sp.nseg * gps;
    const int64_t units = split == 0 ? sp.nseg : split == 1 ? ng : ng * kNearRuns;
    const unsigned blocks = (unsigned)((m + 63) / 64);
    hipLaunchKernelGGL(k_group_near<K>, dim3(blocks, (unsigned)units), dim3(64), 0, s, drec, sigma, gdata, (int)n,
                       sig_stride, sp.segsz, gps, rps, img, split, order, px, py, pz, (int)m, out, unit_stride);
    if (K > 1) {  // two waves per SIMD
        const unsigned waves = (unsigned)std::min<int64_t>(2048, units * blocks * (K - 1));
        hipLaunchKernelGGL(k_near_columns, dim3(waves), dim3(64), 0, s, drec, sigma, gdata,
                           (int64_t)sp.nseg * rps * kGroupStride, (int)n, sig_stride, K, sp.nseg, sp.segsz, gps, rps, img,
                           split, (int)units, order, px, py, pz, (int)m, out, unit_stride);
    }
}

void launch_group_near(const double *drec, const double *sigma, const double *gdata, int64_t n, int64_t sig_stride,
                       int ncol, const SegPlan &sp, const ImgArgs &img, int split, const int *order, const double *px, const double *py,
                       const double *pz, int64_t m, const OutCols &out, int64_t unit_stride, hipStream_t s)
{
    if (m <= 0 || n <= 0) return;
#define NEAR_ARGS drec, sigma, gdata, n, sig_stride, sp, img, split, order, px, py, pz, m, out, unit_stride, s
    switch (ncol) {
    case 1: launch_near_k<1>(NEAR_ARGS); break;
    case 2: launch_near_k<2>(NEAR_ARGS); break;
    case 3: launch_near_k<3>(NEAR_ARGS); break;
    default: launch_near_k<4>(NEAR_ARGS); break;
    }
#undef NEAR_ARGS
}

// Continuous-batching evaluation: workgroup (one wave) b takes work item b --
// up to 64 points of one request against one segment of the elements of one
// resident geometry -- and writes the segment's unscaled partial sums; or, with
// `units`, unit y of it (8 elements of a group, or 16 elements), whose sums go to
// units[b][y][component][lane].  The per-point arithmetic does not depend on which
// other items share the launch, nor on the split.
template <bool MIXED>
__device__ __forceinline__ void eval_item(const WorkItem &w, const ImgArgs &img, double near_factor, double *units)
{
    double *phi = w.phi, *ex = w.ex, *ey = w.ey, *ez = w.ez;
    int p0 = 0, p1 = w.n;
    if (units) {
        p0 = blockIdx.y * kSubElems;
        p1 = min(p0 + kSubElems, w.n);
        if (p0 >= w.n) return;
        phi = units + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kUnitDoubles;
        ex = phi + 64;
        ey = phi + 128;
        ez = phi + 192;
    }
    eval_block<MIXED>(w.drec, w.sigma, w.n, p0, p1, img, near_factor, w.px, w.py, w.pz, w.count, threadIdx.x, 1.0, phi,
                      ex, ey, ez);
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_eval_items_fp64(
    const WorkItem *__restrict__ items, const ImgArgs *__restrict__ imgs, double near_factor,
    double *__restrict__ units)
{
    __shared__ NearList list;
    const WorkItem &w = items[blockIdx.x];
    if (!w.gdata) {
        eval_item<false>(w, imgs[w.geom], near_factor, units);
        return;
    }
    // grouped geometry: the near part, added to k_items_far's
    const int j = min((int)threadIdx.x, w.count - 1);
    const int ng = (w.n + kGroupElems - 1) / kGroupElems;
    const int g0 = units ? (int)blockIdx.y / kNearRuns : 0, g1 = units ? g0 + 1 : ng;
    const int u0 = units ? (int)blockIdx.y % kNearRuns : 0, u1 = units ? u0 + 1 : kNearRuns;
    if (g0 >= ng) return;
    double acc[1][4];
    near_unit<1>(list, uniform_ptr(w.drec), uniform_ptr(w.sigma), 0, uniform_ptr(w.gdata), w.n, imgs[w.geom], w.px[j],
                 w.py[j], w.pz[j], g0, g1, u0, u1, acc);
    if ((int)threadIdx.x >= w.count) return;
    if (units) {
        double *u = units + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kUnitDoubles + threadIdx.x;
        for (int c = 0; c < 4; ++c) u[64 * c] = acc[0][c];
        return;
    }
    w.phi[threadIdx.x] += acc[0][0];
    w.ex[threadIdx.x] += acc[0][1];
    w.ey[threadIdx.x] += acc[0][2];
    w.ez[threadIdx.x] += acc[0][3];
}

// two waves per SIMD, as k_eval_mixed
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_eval_items_mixed(
    const WorkItem *__restrict__ items, const ImgArgs *__restrict__ imgs, double near_factor,
    double *__restrict__ units)
{
    eval_item<true>(items[blockIdx.x], imgs[items[blockIdx.x].geom], near_factor, units);
}

int eval_items_slots(int mixed)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 1;
    const hipError_t e = mixed ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_eval_items_mixed, 64, 0)
                               : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_eval_items_fp64, 64, 0);
    return (e == hipSuccess && per_cu > 0) ? cus * per_cu : 1;
}

void launch_eval_items(const WorkItem *items, int nitems, const ImgArgs *imgs, int mixed, double near_factor,
                       const ItemUnits &u, hipStream_t s)
{
    // whole items, or as many at a time as have their units in the scratch
    int64_t batch = u.sums && u.per > 0 ? u.cap / u.per : 0;
    if (u.far_per > 0 && u.far_cap / u.far_per < batch) batch = u.far_cap / u.far_per;
    const int step = batch > 0 ? (int)(batch < nitems ? batch : nitems) : nitems;
    double *near = batch > 0 ? u.sums : nullptr, *far = near ? u.sums + u.cap * kUnitDoubles : nullptr;
    for (int i = 0; i < nitems; i += step) {
        const int c = nitems - i < step ? nitems - i : step;
        const WorkItem *it = items + i;
        const dim3 g(c, near ? u.per : 1);
        if (mixed) {
            hipLaunchKernelGGL(k_eval_items_mixed, g, dim3(64), 0, s, it, imgs, near_factor, near);
        } else {
            if (!near || u.far_per > 0) launch_items_far(it, c, imgs, far, u.far_per, s);
            hipLaunchKernelGGL(k_eval_items_fp64, g, dim3(64), 0, s, it, imgs, near_factor, near);
        }
        if (near) launch_items_fold(it, c, far, near, u.far_per, u.per, s);
    }
}

// ---------------------------------------------------------------- assembly
// Grid: x over blocks of 256 rows, y over blocks of kTileA columns.  Each
// lane writes A[i + j n] for its row i and the block's columns j: the 256
// lanes of a workgroup store 256 consecutive doubles of a column (2 KB).
// The matrix is assembled in FP64 to the same accuracy in both precision
// modes: it is a small share of a step's interactions, and an error in its entries
// carries into sigma through the solve, times the condition.  So the mixed path's
// far field (1e-7 of an element's) stays out of it, and the far copies' lattice sums
// (k_assemble_grouped) are truncated below the closed forms' own rounding.  Against
// 64-bit entries (closed forms near, Gauss rules far; GEM cells of 1736 x 121, 1648 x
// 49 and 2576 x 121 copies, THGEM of 5792 x 49), rms error over rms entry: potential
// rows 1.1, 1.4, 1.1, 1.5e-15 by lattice sums and 1.8, 1.6, 2.0, 2.7e-15 direct,
// interface rows 3.1, 3.0, 3.4, 3.1e-16 and 3.3, 3.0, 3.7, 3.3e-16; sigma's 2-norm error
// 3.9, 1.6, 5.1, 6.6e-13 and 4.1, 1.5, 4.9, 6.5e-13.
__global__ __launch_bounds__(kBlock) void k_assemble(const double *__restrict__ drec, int n, ImgArgs img,
                                                      const double *__restrict__ cx, const double *__restrict__ cy,
                                                      const double *__restrict__ cz, double *__restrict__ A)
{
    __shared__ double t_rec[kTileA * R_STRIDE];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int j0 = blockIdx.y * kTileA;
    const int cnt = min(kTileA, n - j0);
    for (int k = threadIdx.x; k < cnt * R_STRIDE; k += kBlock) t_rec[k] = drec[(size_t)j0 * R_STRIDE + k];
    __syncthreads();
    if (i >= n) return;
    const double *ri = drec + (size_t)i * R_STRIDE;
    const double Px = cx ? cx[i] : ri[R_CX];
    const double Py = cy ? cy[i] : ri[R_CY];
    const double Pz = cz ? cz[i] : ri[R_CZ];
    const bool diel = ri[R_BC] != 0.0;
    const double nx = ri[R_E3X], ny = ri[R_E3Y], nz = ri[R_E3Z];
    const double jump = ri[R_JUMP];
    for (int p = 0; p < cnt; ++p) {
        const int j = j0 + p;
        const Elem e = load_elem(t_rec + p * R_STRIDE);
        double cp, gx, gy, gz;
        element_copies<false>(e, img, Px, Py, Pz, i == j, 0.0, cp, gx, gy, gz);
        double a = diel ? kKe * (nx * gx + ny * gy + nz * gz) : kKe * cp;
        a += (diel && i == j) ? jump : 0.0;
        A[(size_t)j * n + i] = a;
    }
}

// The same with the far copies of each group of 64 elements by lattice sums of
// harmonics (lattice_far.hpp): 64 rows, one per lane, x one group per workgroup.
//   1. The waves scan the lattice for the copies near any of the rows (closer
//      than ~7 group radii) and keep the range of i2 they span in each row (r,
//      i1) of the lattice: the near copies, all others are far.
//   2. Each wave sums its orders' harmonics over the far copies in registers,
//      at the degree that the farthest tier of all lanes allows; dielectric
//      rows exchange orders through LDS for the normal component.
//   3. The sums times the moments of the 64 elements (uniform: scalar loads, an
//      SGPR operand per product), added over the waves through LDS.
//   4. The near copies by closed forms, element by element.
// FP64 VALU bound.  Direct: C x 64 closed forms of ~75 instructions per row and
// group, C = 121; here ~1000 per far copy at degree 14, ~400 at degree 6, ~15 000
// for the products, and the near copies' closed forms.  n = 8064 (GEM cell, 121
// copies): 22.9 ms direct; now 4.4 ms for the far copies, of which the products take
// 1.8, and 3.1 ms for the near ones (k_assemble_near).
constexpr int kLatticeRows = 512;  // lattice rows (reflection, i1) that the lists hold
struct NearRow {
    int row;  // r (2 n1 + 1) + i1 + n1
    int lo, hi;
};

__device__ const NormalFactors kNormalFactors = make_normal_factors();

template <int W>
__device__ __forceinline__ void assemble_far(cdouble_p h, cdouble_p coef, int cnt, const ImgArgs &img,
                                             const int2 *range, const GroupVec &P, const double *__restrict__ ri,
                                             double *x, double *__restrict__ A, int n, int i)
{
    const bool diel = ri[R_BC] != 0.0;
    const int lane = threadIdx.x & 63, nrow = 2 * img.n1 + 1;
    const bool any = __ballot(diel) != 0;
    const double a = h[3];
    const double scale = diel ? kKe / (a * a) : kKe / a;
    int buf = 0;
#pragma unroll 1
    for (int r = 0; r < img.nref; ++r) {
        LatticeSums<W> F;
        F.clear();
        const int ax = img.axes[r];
        const double par = img.parity[r];
        const GroupVec v0 = group_origin(img, ax, P.x, P.y, P.z, h);
#pragma unroll 1
        for (int i1 = -img.n1; i1 <= img.n1; ++i1) {
            const GroupVec v1 = group_step(v0, -(double)i1, img.a1[r]);
            const int2 near = range[r * nrow + i1 + img.n1];
            const int lo = uni(near.x), hi = uni(near.y);
#pragma unroll 1
            for (int i2 = -img.n2; i2 <= img.n2; ++i2) {
                if (i2 == lo) {
                    i2 = hi;
                    continue;
                }
                const GroupVec d = group_step(v1, -(double)i2, img.a2[r]);
                const double r2 = group_r2(d);
                const int deg = __ballot(!(r2 >= h[kHeadTier + 4])) == 0   ? 7
                                : __ballot(!(r2 >= h[kHeadTier + 2])) == 0 ? 11
                                                                           : kGroupL;
                F.add(d, r2, a, par, deg);
            }
        }
        if (any) {
            __syncthreads();  // the products' buffers of the last reflection are read
            F.put_exchange(x);
            __syncthreads();
            const double Nx = ri[R_E3X], Ny = ri[R_E3Y], Nz = ri[R_E3Z];
            F.normal_component(x, in_loop(uniform_ptr(kNormalFactors.f)), diel,
                               (ax & 1) ? -Nx : Nx, (ax & 2) ? -Ny : Ny, (ax & 4) ? -Nz : Nz);
            __syncthreads();
        }
#pragma unroll 1
        for (int j0 = 0; j0 < cnt; j0 += 8) {
            double *red = x + buf * (kSets * 8 * 64);
            buf ^= 1;
#pragma unroll 1
            for (int q = 0; q < 8; ++q)
                red[(W * 8 + q) * 64 + lane] =
                    F.dot(in_loop(coef + (int64_t)min(j0 + q, cnt - 1) * kElemCoefs + set_offset(W)));
            __syncthreads();
#pragma unroll
            for (int q = W; q < 8; q += kSets) {
                if (j0 + q >= cnt || i >= n) continue;
                double s = red[q * 64 + lane];
#pragma unroll
                for (int w = 1; w < kSets; ++w) s += red[(w * 8 + q) * 64 + lane];
                double *e = A + (size_t)(j0 + q) * n + i;
                *e = r == 0 ? scale * s : fma(scale, s, *e);
            }
        }
    }
}

// What both kernels below derive from their block: one row per lane, the group
// of columns, the range of near i2 in each row of the lattice, and whether there are far
// copies at all.  A group as wide as the lattice has none (in meshes whose elements
// come in random order all are like that): no harmonics and no products then.  In random
// order, n = 8064 x 121 copies: 24.6 ms direct, 27.0 with empty sums multiplied, 25.1
// so; n = 10 848 x 49: 21.7, 28.4, 23.1.  (k_assemble's own loops in k_assemble_near for
// such groups take 24.6 and 22.2, and 1 to 3 % longer for meshes in order.)
struct AsmBlock {
    int i, e0, cnt;
    bool far;
    GroupVec P;
    cdouble_p head;
};
__device__ __forceinline__ AsmBlock assemble_block(const double *__restrict__ drec, const double *__restrict__ heads,
                                                   int n, const ImgArgs &img, int2 *range)
{
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    AsmBlock b;
    b.i = blockIdx.x * 64 + lane;
    b.e0 = blockIdx.y * kGroupElems;
    b.cnt = min(kGroupElems, n - b.e0);
    const double *ri = drec + (size_t)min(b.i, n - 1) * R_STRIDE;
    b.P = {ri[R_CX], ri[R_CY], ri[R_CZ]};
    b.head = uniform_ptr(heads + (size_t)blockIdx.y * kGroupHead);
    const int nrow = 2 * img.n1 + 1, rows = img.nref * nrow;
    bool far = false;
#pragma unroll 1
    for (int q = wave; q < rows; q += 4) {
        const int r = q / nrow, i1 = q % nrow - img.n1;
        const GroupVec v1 =
            group_step(group_origin(img, img.axes[r], b.P.x, b.P.y, b.P.z, b.head), -(double)i1, img.a1[r]);
        int lo = img.n2 + 1, hi = img.n2;
#pragma unroll 1
        for (int i2 = -img.n2; i2 <= img.n2; ++i2)
            if (__ballot(!(group_r2(group_step(v1, -(double)i2, img.a2[r])) >= b.head[kHeadTier]))) {
                lo = min(lo, i2);
                hi = i2;
            }
        if (lane == 0) range[q] = make_int2(lo, hi);
        far = far || lo > -img.n2 || hi < img.n2;
    }
    b.far = __syncthreads_or(far);
    return b;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_assemble_grouped(
    const double *__restrict__ drec, const double *__restrict__ heads, const double *__restrict__ coef, int n,
    ImgArgs img, double *__restrict__ A)
{
    __shared__ double x[kExchange * 128];  // exchanged orders, then two buffers of 8 columns' products
    __shared__ int2 range[kLatticeRows];
    const AsmBlock b = assemble_block(drec, heads, n, img, range);
    double *const Ag = A + (size_t)b.e0 * n;
    if (!b.far) return;  // k_assemble_near stores all there is
    const cdouble_p cg = uniform_ptr(coef + (size_t)b.e0 * kElemCoefs);
    const double *ri = drec + (size_t)min(b.i, n - 1) * R_STRIDE;
    switch (uni((int)(threadIdx.x >> 6))) {
    case 0: assemble_far<0>(b.head, cg, b.cnt, img, range, b.P, ri, x, Ag, n, b.i); break;
    case 1: assemble_far<1>(b.head, cg, b.cnt, img, range, b.P, ri, x, Ag, n, b.i); break;
    case 2: assemble_far<2>(b.head, cg, b.cnt, img, range, b.P, ri, x, Ag, n, b.i); break;
    default: assemble_far<3>(b.head, cg, b.cnt, img, range, b.P, ri, x, Ag, n, b.i); break;
    }
}

// The near copies by closed forms, added to what k_assemble_grouped stored, if
// anything.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_assemble_near(
    const double *__restrict__ drec, const double *__restrict__ heads, int n, ImgArgs img, double *__restrict__ A)
{
    __shared__ int2 range[kLatticeRows];
    __shared__ NearRow list[kLatticeRows];
    __shared__ int s_count;
    const AsmBlock blk = assemble_block(drec, heads, n, img, range);
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const int i = blk.i, e0 = blk.e0, cnt = blk.cnt;
    const bool in = i < n;
    const GroupVec P = blk.P;
    const double *ri = drec + (size_t)min(i, n - 1) * R_STRIDE;
    const GroupVec N = {ri[R_E3X], ri[R_E3Y], ri[R_E3Z]};
    const bool diel = ri[R_BC] != 0.0;
    const double jump = ri[R_JUMP];
    const int nrow = 2 * img.n1 + 1, rows = img.nref * nrow;
    if (wave == 0) {  // the lattice rows with near copies, in order
        int count = 0;
        for (int q0 = 0; q0 < rows; q0 += 64) {
            const int q = q0 + lane;
            const int2 e = range[min(q, rows - 1)];
            const bool has = q < rows && e.x <= e.y;
            const uint64_t m = __ballot(has);
            if (has) list[count + __popcll(m & ((1ull << lane) - 1))] = {q, e.x, e.y};
            count += __popcll(m);
        }
        if (lane == 0) s_count = count;
    }
    __syncthreads();
    double *const Ag = A + (size_t)e0 * n;
    const int count = uni(s_count);
    if (count == 0) return;
#pragma unroll 1
    for (int j = wave + kSets * blockIdx.z; j < cnt; j += kSets * gridDim.z) {
        const Elem e = load_elem_c(uniform_ptr(drec + (size_t)(e0 + j) * R_STRIDE));
        const double far2 = (kFarDiam * kFarDiam) * (e.diam * e.diam);
        const double vfar2 = (kVeryFarDiam * kVeryFarDiam) * (e.diam * e.diam);
        const bool self = i == e0 + j;
        double sum = 0.0;
        for (int l = 0; l < count;) {
            const int r = uni(list[l].row) / nrow, ax = img.axes[r];
            const double Qx = (ax & 1) ? 2.0 * img.mpos[0] - P.x : P.x;
            const double Qy = (ax & 2) ? 2.0 * img.mpos[1] - P.y : P.y;
            const double Qz = (ax & 4) ? 2.0 * img.mpos[2] - P.z : P.z;
            const double rx = Qx - e.ox, ry = Qy - e.oy, rz = Qz - e.oz;
            const double X0 = rx * e.e1x + ry * e.e1y + rz * e.e1z;
            const double Z0 = rx * e.e2x + ry * e.e2y + rz * e.e2z;
            const double H0 = rx * e.e3x + ry * e.e3y + rz * e.e3z;
            const double *a = img.a1[r], *b = img.a2[r];
            const double aX = a[0] * e.e1x + a[1] * e.e1y + a[2] * e.e1z;
            const double aZ = a[0] * e.e2x + a[1] * e.e2y + a[2] * e.e2z;
            const double aH = a[0] * e.e3x + a[1] * e.e3y + a[2] * e.e3z;
            const double bX = b[0] * e.e1x + b[1] * e.e1y + b[2] * e.e1z;
            const double bZ = b[0] * e.e2x + b[1] * e.e2y + b[2] * e.e2z;
            const double bH = b[0] * e.e3x + b[1] * e.e3y + b[2] * e.e3z;
            double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
            for (; l < count; ++l) {
                const int row = uni(list[l].row) - r * nrow;
                if (row >= nrow) break;
                const int i1 = row - img.n1, hi = uni(list[l].hi);
                const double f1 = -(double)i1;
                const double X1 = fma(f1, aX, X0), Z1 = fma(f1, aZ, Z0), H1 = fma(f1, aH, H0);
#pragma unroll 1
                for (int i2 = uni(list[l].lo); i2 <= hi; ++i2) {
                    const double f2 = -(double)i2;
                    const double X = fma(f2, bX, X1), Z = fma(f2, bZ, Z1);
                    double H = fma(f2, bH, H1);
                    H = (self && r == 0 && i1 == 0 && i2 == 0) ? 0.0 : H;
                    if (e.kind == 0)
                        copy_fp64<0>(e, X, Z, H, far2, vfar2, s);
                    else
                        copy_fp64<1>(e, X, Z, H, far2, vfar2, s);
                }
            }
            const double gx = s[1] * e.e1x + s[2] * e.e2x + s[3] * e.e3x;
            const double gy = s[1] * e.e1y + s[2] * e.e2y + s[3] * e.e3y;
            const double gz = s[1] * e.e1z + s[2] * e.e2z + s[3] * e.e3z;
            const double field =
                N.x * ((ax & 1) ? -gx : gx) + N.y * ((ax & 2) ? -gy : gy) + N.z * ((ax & 4) ? -gz : gz);
            sum = fma(img.parity[r], diel ? field : s[0], sum);
        }
        if (in) {
            double *p = Ag + (size_t)j * n + i;
            const double v = kKe * sum + (diel && self ? jump : 0.0);
            *p = blk.far ? *p + v : v;
        }
    }
}

// With 25 copies per element the two ways take the same time (n = 8064 5.7 and 5.8
// ms, n = 1242 0.58 and 0.53), with 121 7.5 and 22.9 ms.  The direct kernel also takes
// lattices with more rows than the lists hold, and collocation points of the
// caller's own, which need not lie on their elements.
bool assemble_grouped(int64_t n, const ImgArgs &img)
{
    return n >= 2 * kGroupElems && img_copies(img) >= 36 && (int64_t)img.nref * (2 * img.n1 + 1) <= kLatticeRows;
}

void launch_assemble(const double *drec, int64_t n, const ImgArgs &img, const double *cx, const double *cy,
                     const double *cz, double *A, double *scratch, hipStream_t s)
{
    if (n <= 0) return;
    if (scratch && !cx && assemble_grouped(n, img)) {
        const int ng = (int)((n + kGroupElems - 1) / kGroupElems);
        double *heads = scratch, *coef = scratch + (size_t)ng * kGroupHead;
        launch_element_moments(drec, n, heads, coef, s);
        const dim3 g((unsigned)((n + 63) / 64), (unsigned)ng);
        hipLaunchKernelGGL(k_assemble_grouped, g, dim3(256), 0, s, drec, heads, coef, (int)n, img, A);
        // elements of a group over several workgroups where there are few groups
        const unsigned parts = (uint64_t)g.x * g.y >= 2048 ? 1u : 4u;
        hipLaunchKernelGGL(k_assemble_near, dim3(g.x, g.y, parts), dim3(256), 0, s, drec, heads, (int)n, img, A);
        return;
    }
    const dim3 g((unsigned)((n + kBlock - 1) / kBlock), (unsigned)((n + kTileA - 1) / kTileA));
    hipLaunchKernelGGL(k_assemble, g, dim3(kBlock), 0, s, drec, (int)n, img, cx, cy, cz, A);
}

}  // namespace nebem
