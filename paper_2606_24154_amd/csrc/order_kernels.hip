// order_kernels.hip -- evaluation in spatial (Morton) order of the points.
//
// The field kernels give every lane one point and walk the elements in the
// same order for all lanes; a point's arithmetic does not depend on the other
// points of its wave, so the order in which points are packed into waves
// changes no bit of any result.  It does change how much work a wave does:
// the per-lane choice between the near and the far evaluation of an element
// copy (and, on the mixed path, among the far-field tiers) is a divergent
// branch, and a wave whose 64 points are scattered over the cell executes
// several of them for the same copy.  Sorting the points along a Morton curve
// of their bounding box packs neighbours into a wave, whose lanes then agree
// on the branch for nearly every copy.  Results are scattered back to the
// caller's order.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "nebem_internal.hpp"

namespace nebem {

constexpr int kOB = 256;         // threads per block of the helper kernels
constexpr int kBoxParts = 256;   // partial bounding boxes (first reduction pass)

// per-block bounding box of a strided share of the points (min / max are
// exact, so the result does not depend on the reduction order)
__global__ __launch_bounds__(kOB) void k_bbox_part(const double *__restrict__ px, const double *__restrict__ py,
                                                   const double *__restrict__ pz, int m, double *__restrict__ part)
{
    __shared__ double red[6][kOB];
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int i = blockIdx.x * kOB + threadIdx.x; i < m; i += gridDim.x * kOB) {
        const double c[3] = {px[i], py[i], pz[i]};
        for (int k = 0; k < 3; ++k) {
            v[k] = fmin(v[k], c[k]);
            v[3 + k] = fmax(v[3 + k], c[k]);
        }
    }
    for (int k = 0; k < 6; ++k) red[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int h = kOB / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h)
            for (int k = 0; k < 6; ++k)
                red[k][threadIdx.x] = k < 3 ? fmin(red[k][threadIdx.x], red[k][threadIdx.x + h])
                                            : fmax(red[k][threadIdx.x], red[k][threadIdx.x + h]);
        __syncthreads();
    }
    if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = red[threadIdx.x][0];
}

// 10-bit coordinate -> bits spread to every third position
__device__ __forceinline__ unsigned spread3(unsigned x)
{
    x &= 0x3ffu;
    x = (x | (x << 16)) & 0x030000ffu;
    x = (x | (x << 8)) & 0x0300f00fu;
    x = (x | (x << 4)) & 0x030c30c3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

__device__ __forceinline__ unsigned quant10(double v, double lo, double sc)
{
    const double t = (v - lo) * sc;  // NaN coordinates fail both tests -> 0
    return t >= 1023.0 ? 1023u : (t > 0.0 ? (unsigned)t : 0u);
}

// Morton code of a point in the box (min x, y, z, max x, y, z).  cubes: the
// box's longest side sets the scale of all three axes, so that consecutive
// points fill cubes -- a wave of 64 stands as close together as it can (in a
// detector gap, many times longer than a cell is wide, the per-axis scale
// makes it as elongated as the gap).
__device__ __forceinline__ unsigned morton_key(double x, double y, double z, const double *box, int cubes)
{
    const double c[3] = {x, y, z};
    double ext[3] = {box[3] - box[0], box[4] - box[1], box[5] - box[2]};
    if (cubes) ext[0] = ext[1] = ext[2] = fmax(ext[0], fmax(ext[1], ext[2]));
    unsigned q[3];
    for (int k = 0; k < 3; ++k) {
        const double sc = (ext[k] > 0.0 && ext[k] < INFINITY) ? 1024.0 / ext[k] : 0.0;
        q[k] = quant10(c[k], box[k], sc);
    }
    return spread3(q[0]) | (spread3(q[1]) << 1) | (spread3(q[2]) << 2);
}

// keys[i] = Morton code of point i in the box (reduced from nparts partial
// boxes by every block: nparts x 6 doubles, L2-resident), idx[i] = i
__global__ __launch_bounds__(kOB) void k_keys(const double *__restrict__ px, const double *__restrict__ py,
                                              const double *__restrict__ pz, int m,
                                              const double *__restrict__ part, int nparts, int cubes,
                                              unsigned *__restrict__ keys, int *__restrict__ idx)
{
    __shared__ double box[6];
    if (threadIdx.x < 6) {
        const int k = threadIdx.x;
        double b = k < 3 ? INFINITY : -INFINITY;
        for (int p = 0; p < nparts; ++p) b = k < 3 ? fmin(b, part[p * 6 + k]) : fmax(b, part[p * 6 + k]);
        box[k] = b;
    }
    __syncthreads();
    const int i = blockIdx.x * kOB + threadIdx.x;
    if (i >= m) return;
    keys[i] = morton_key(px[i], py[i], pz[i], box, cubes);
    idx[i] = i;
}

// Up to kSmallOrder points by one workgroup: bounding box, keys, a bitonic
// sort of (key, index) in LDS (unique keys, so it is the stable order the
// radix sort gives) and the gather, in one launch (30 us at 2003 points, bound
// by the sort's ~66 barriers) where the radix sort takes ten.
constexpr int kSmallOrder = 4096;
constexpr int kSmallThreads = 1024;
__global__ __launch_bounds__(kSmallThreads) void k_order_small(const double *__restrict__ px,
                                                               const double *__restrict__ py,
                                                               const double *__restrict__ pz, int m, int len, int cubes,
                                                               double *__restrict__ sx, double *__restrict__ sy,
                                                               double *__restrict__ sz, int *__restrict__ perm)
{
    __shared__ unsigned long long key[kSmallOrder];
    __shared__ double red[6][kSmallThreads / 64];
    __shared__ double box[6];
    const int t = threadIdx.x;
    double v[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};  // min x, y, z, -x, -y, -z
    for (int i = t; i < m; i += kSmallThreads) {
        const double c[3] = {px[i], py[i], pz[i]};
        for (int k = 0; k < 3; ++k) {
            v[k] = fmin(v[k], c[k]);
            v[3 + k] = fmin(v[3 + k], -c[k]);
        }
    }
    for (int k = 0; k < 6; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[k] = fmin(v[k], __shfl_xor(v[k], off));
        if ((t & 63) == 0) red[k][t >> 6] = v[k];
    }
    __syncthreads();
    if (t < 6) {
        double b = red[t][0];
        for (int w = 1; w < kSmallThreads / 64; ++w) b = fmin(b, red[t][w]);
        box[t] = t < 3 ? b : -b;
    }
    __syncthreads();
    for (int i = t; i < len; i += kSmallThreads)
        key[i] = i < m ? ((unsigned long long)morton_key(px[i], py[i], pz[i], box, cubes) << 32) | (unsigned)i : ~0ull;
    __syncthreads();
    for (int k = 2; k <= len; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int p = t; p < len / 2; p += kSmallThreads) {
                const int lo = ((p & ~(j - 1)) << 1) | (p & (j - 1)), hi = lo | j;
                const unsigned long long a = key[lo], b = key[hi];
                if ((a > b) == ((lo & k) == 0)) {
                    key[lo] = b;
                    key[hi] = a;
                }
            }
            __syncthreads();
        }
    for (int i = t; i < m; i += kSmallThreads) {
        const int q = (int)(unsigned)key[i];
        perm[i] = q;
        sx[i] = px[q];
        sy[i] = py[q];
        sz[i] = pz[q];
    }
}

__global__ __launch_bounds__(kOB) void k_gather3(const double *__restrict__ px, const double *__restrict__ py,
                                                 const double *__restrict__ pz, const int *__restrict__ perm, int m,
                                                 double *__restrict__ sx, double *__restrict__ sy,
                                                 double *__restrict__ sz)
{
    const int k = blockIdx.x * kOB + threadIdx.x;
    if (k >= m) return;
    const int i = perm[k];
    sx[k] = px[i];
    sy[k] = py[i];
    sz[k] = pz[i];
}

// dst_j[perm[k]] = src[j * m + k] for every non-null destination j
__global__ __launch_bounds__(kOB) void k_scatter4(const double *__restrict__ src, const int *__restrict__ perm, int m,
                                                  double *__restrict__ d0, double *__restrict__ d1,
                                                  double *__restrict__ d2, double *__restrict__ d3)
{
    const int k = blockIdx.x * kOB + threadIdx.x;
    if (k >= m) return;
    const int i = perm[k];
    const size_t mm = (size_t)m;
    if (d0) d0[i] = src[k];
    if (d1) d1[i] = src[mm + k];
    if (d2) d2[i] = src[2 * mm + k];
    if (d3) d3[i] = src[3 * mm + k];
}

namespace {
// scratch of one sort: keys (in/out), identity indices, partial boxes, sort temp
struct SortLayout {
    size_t keys_in, keys_out, idx_in, part, sort, total;
    size_t sort_bytes;
};

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

hipError_t sort_layout(int64_t m, SortLayout &L)
{
    size_t sort_bytes = 0;
    hipError_t e = rocprim::radix_sort_pairs(nullptr, sort_bytes, (const unsigned *)nullptr, (unsigned *)nullptr,
                                             (const int *)nullptr, (int *)nullptr, (int)m, 0u, 30u);
    if (e != hipSuccess) return e;
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off += align256(b);
        return o;
    };
    L.keys_in = take(4 * (size_t)m);
    L.keys_out = take(4 * (size_t)m);
    L.idx_in = take(4 * (size_t)m);
    L.part = take(sizeof(double) * 6 * kBoxParts);
    L.sort = take(sort_bytes);
    L.sort_bytes = sort_bytes;
    L.total = off;
    return hipSuccess;
}
}  // namespace

bool eval_ordering_pays(int64_t m) { return m >= kOrderMin; }

size_t order_points_workspace(int64_t m)
{
    SortLayout L;
    if (sort_layout(m, L) != hipSuccess) return 0;
    return L.total;
}

hipError_t launch_order_points(const double *px, const double *py, const double *pz, int64_t m, double *sx,
                               double *sy, double *sz, int *perm, bool cubes, void *ws, size_t ws_bytes, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    if (m <= kSmallOrder) {
        int len = 2;
        while (len < m) len <<= 1;
        hipLaunchKernelGGL(k_order_small, dim3(1), dim3(kSmallThreads), 0, s, px, py, pz, (int)m, len, (int)cubes, sx,
                           sy, sz, perm);
        return hipGetLastError();
    }
    SortLayout L;
    hipError_t e = sort_layout(m, L);
    if (e != hipSuccess) return e;
    if (!ws || ws_bytes < L.total) return hipErrorInvalidValue;
    char *w = static_cast<char *>(ws);
    unsigned *keys_in = reinterpret_cast<unsigned *>(w + L.keys_in);
    unsigned *keys_out = reinterpret_cast<unsigned *>(w + L.keys_out);
    int *idx_in = reinterpret_cast<int *>(w + L.idx_in);
    double *part = reinterpret_cast<double *>(w + L.part);
    const int mi = (int)m;
    const unsigned g = (unsigned)((m + kOB - 1) / kOB);
    const int nparts = (int)std::min<int64_t>(kBoxParts, g);
    hipLaunchKernelGGL(k_bbox_part, dim3(nparts), dim3(kOB), 0, s, px, py, pz, mi, part);
    hipLaunchKernelGGL(k_keys, dim3(g), dim3(kOB), 0, s, px, py, pz, mi, part, nparts, (int)cubes, keys_in, idx_in);
    size_t sort_bytes = L.sort_bytes;
    e = rocprim::radix_sort_pairs(w + L.sort, sort_bytes, keys_in, keys_out, idx_in, perm, mi, 0u, 30u, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gather3, dim3(g), dim3(kOB), 0, s, px, py, pz, perm, mi, sx, sy, sz);
    return hipGetLastError();
}

void launch_unorder4(const double *src, const int *perm, int64_t m, double *d0, double *d1, double *d2, double *d3,
                     hipStream_t s)
{
    if (m <= 0) return;
    hipLaunchKernelGGL(k_scatter4, dim3((unsigned)((m + kOB - 1) / kOB)), dim3(kOB), 0, s, src, perm, (int)m, d0, d1,
                       d2, d3);
}

// ------------------------------------------------------- evaluation driver
namespace {
EvalShape shape_of(int64_t n, const ImgArgs &img, int ncol, int mixed)
{
    return eval_shape(seg_plan(n, img), !mixed && eval_grouped(n, img), (int64_t)img.nref * (2 * img.n1 + 1), ncol,
                      group_record_bytes());
}

// one column block of a grouped chunk: unscaled segment sums into part; `fresh`:
// the groups' records are not there yet
void eval_grouped_chunk(const double *drec, const double *sg, int64_t n, int k, const EvalShape &sh,
                        const ImgArgs &img, const double *px, const double *py, const double *pz, int64_t c,
                        const OutCols &pc, int64_t seg_stride, char *w, const ChunkLayout &L, bool fresh,
                        hipStream_t s)
{
    double *gd = reinterpret_cast<double *>(w + L.groups);
    if (fresh) launch_group_moments(drec, sg, n, n, k, sh.sp, gd, s);
    if (!L.fsplit) {
        int *order = segment_order(gd, k, sh.sp);
        launch_segment_order(gd, n, sh.sp, order, s);
        launch_group_far(gd, n, k, sh.sp, img, 0, order, px, py, pz, c, pc, seg_stride, s);
        launch_group_near(drec, sg, gd, n, n, k, sh.sp, img, 0, order, px, py, pz, c, pc, seg_stride, s);
        return;
    }
    double *far = reinterpret_cast<double *>(w + L.far), *near = reinterpret_cast<double *>(w + L.near);
    // components that are not wanted are not written, and their sums not read
    auto cols = [&](double *b) {
        OutCols o = pc;
        for (int q = 0; q < 4; ++q) o.c[q] = pc.c[q] ? b + (size_t)q * c : nullptr;
        return o;
    };
    launch_group_far(gd, n, k, sh.sp, img, L.fsplit, nullptr, px, py, pz, c, cols(far), seg_stride, s);
    launch_group_near(drec, sg, gd, n, n, k, sh.sp, img, L.nsplit, nullptr, px, py, pz, c, cols(near), seg_stride, s);
    if (L.fsplit == 2) {
        double *f = reinterpret_cast<double *>(w + L.ffold);
        launch_fold_units(far, sh.nrec, (int)sh.rows, seg_stride, f, s);
        far = f;
    }
    if (L.nsplit == 2) {
        double *f = reinterpret_cast<double *>(w + L.nfold);
        launch_fold_units(near, sh.ngroup, kNearRuns, seg_stride, f, s);
        near = f;
    }
    launch_fold_groups(far, near, sh.sp, seg_stride, reinterpret_cast<double *>(w + L.part), s);
}

// one chunk of c points (unsorted input px.., outputs o.c[comp] + col * ostride);
// first: the first one of the call
void eval_chunk(const double *drec, const double *sigma, int64_t n, int ncol, const EvalShape &sh,
                const ImgArgs &img, int mixed, double near_factor, const double *px, const double *py,
                const double *pz, int64_t c, const OutCols &o, char *w, const ChunkLayout &L, bool first,
                hipStream_t s)
{
    double *part = sh.part_pp ? reinterpret_cast<double *>(w + L.part) : nullptr;
    for (int c0 = 0; c0 < ncol; c0 += kMultiCols) {
        const int k = ncol - c0 < kMultiCols ? ncol - c0 : kMultiCols;
        const double *sg = sigma + (size_t)c0 * n;
        OutCols oc = o;
        for (int q = 0; q < 4; ++q) oc.c[q] = o.c[q] ? o.c[q] + (size_t)c0 * o.stride : nullptr;
        if (!sh.part_pp && !L.fsplit) {
            if (ncol == 1)
                launch_eval_seg(drec, sg, n, sh.sp, img, mixed, near_factor, false, px, py, pz, c, kKe, oc.c[0],
                                oc.c[1], oc.c[2], oc.c[3], 0, s);
            else
                launch_eval_multi_seg(drec, sg, n, n, k, sh.sp, img, mixed, near_factor, false, px, py, pz, c, kKe, oc,
                                      0, s);
            continue;
        }
        // partials: column j, component q of unit y at buf + y * 4 k c + (4 j + q) c
        const size_t cc = (size_t)c;
        const int64_t seg_stride = (int64_t)(4 * (size_t)k * cc);
        auto cols = [&](double *b) {
            return OutCols{{o.c[0] ? b : nullptr, o.c[1] ? b + cc : nullptr, o.c[2] ? b + 2 * cc : nullptr,
                            o.c[3] ? b + 3 * cc : nullptr},
                           (int64_t)(4 * cc)};
        };
        if (sh.grouped) {
            eval_grouped_chunk(drec, sg, n, k, sh, img, px, py, pz, c, cols(part), seg_stride, w, L, first, s);
        } else {
            const bool split = L.fsplit != 0;
            double *units = split ? reinterpret_cast<double *>(w + L.far) : part;
            const OutCols pc = cols(units);
            if (ncol == 1)
                launch_eval_seg(drec, sg, n, sh.sp, img, mixed, near_factor, split, px, py, pz, c, 1.0, pc.c[0],
                                pc.c[1], pc.c[2], pc.c[3], seg_stride, s);
            else
                launch_eval_multi_seg(drec, sg, n, n, k, sh.sp, img, mixed, near_factor, split, px, py, pz, c, 1.0, pc,
                                      seg_stride, s);
            if (split && sh.sp.nseg == 1) {  // one segment: its units are the reduction's own terms
                launch_reduce_segments(units, eval_subunits(sh.sp), k, c, seg_stride, oc, s);
                continue;
            }
            if (split) launch_fold_units(units, sh.sp.nseg, eval_subunits(sh.sp), seg_stride, part, s);
        }
        launch_reduce_segments(part, sh.sp.nseg, k, c, seg_stride, oc, s);
    }
}
}  // namespace

size_t eval_workspace(int64_t n, const ImgArgs &img, int64_t m, int ncol, int mixed)
{
    if (m <= 0 || ncol <= 0 || n <= 0) return 0;
    const EvalShape sh = shape_of(n, img, ncol, mixed);
    const int64_t c = chunk_points(sh, m, SIZE_MAX, order_points_workspace);
    ChunkLayout L;
    if (!c || !chunk_layout(sh, c, SIZE_MAX, order_points_workspace, L)) return 0;
    return L.total;
}

size_t eval_workspace_min(int64_t n, const ImgArgs &img, int64_t m, int ncol, int mixed)
{
    if (m <= 0 || ncol <= 0 || n <= 0) return 0;
    const EvalShape sh = shape_of(n, img, ncol, mixed);
    ChunkLayout L;
    if (!chunk_layout(sh, std::min<int64_t>(m, 256), 0, order_points_workspace, L)) return 0;
    return L.total;
}

hipError_t run_eval(const double *drec, const double *sigma, int64_t n, int ncol, const ImgArgs &img, int mixed,
                    double near_factor, const double *px, const double *py, const double *pz, int64_t m, double *phi,
                    double *ex, double *ey, double *ez, void *ws, size_t ws_bytes, hipStream_t s)
{
    if (m <= 0 || ncol <= 0) return hipSuccess;
    const size_t mm = (size_t)m;
    if (n <= 0) {  // no elements: zero fields
        for (double *o : {phi, ex, ey, ez})
            if (o) {
                hipError_t e = hipMemsetAsync(o, 0, mm * (size_t)ncol * sizeof(double), s);
                if (e != hipSuccess) return e;
            }
        return hipSuccess;
    }
    const EvalShape sh = shape_of(n, img, ncol, mixed);
    const int64_t c = chunk_points(sh, m, ws_bytes, order_points_workspace);
    if (!c || (!ws && ws_bytes)) return hipErrorInvalidValue;
    char *w = static_cast<char *>(ws);
    for (int64_t p0 = 0; p0 < m; p0 += c) {
        const int64_t cnt = std::min<int64_t>(c, m - p0);
        ChunkLayout Lc;
        if (!chunk_layout(sh, cnt, ws_bytes, order_points_workspace, Lc) || Lc.total > ws_bytes)
            return hipErrorInvalidValue;
        // one column block: its records serve all chunks
        const bool first = p0 == 0 || ncol > kMultiCols;
        if (!Lc.ordered) {
            OutCols o = {{phi ? phi + p0 : nullptr, ex ? ex + p0 : nullptr, ey ? ey + p0 : nullptr,
                          ez ? ez + p0 : nullptr},
                         m};
            eval_chunk(drec, sigma, n, ncol, sh, img, mixed, near_factor, px + p0, py + p0, pz + p0, cnt, o, w, Lc,
                       first, s);
            continue;
        }
        const size_t cc = (size_t)cnt;
        int *perm = reinterpret_cast<int *>(w + Lc.perm);
        double *sp = reinterpret_cast<double *>(w + Lc.pts);
        double *so = reinterpret_cast<double *>(w + Lc.res);
        hipError_t e = launch_order_points(px + p0, py + p0, pz + p0, cnt, sp, sp + cc, sp + 2 * cc, perm, true,
                                           w + Lc.sort, Lc.sort_ws, s);
        if (e != hipSuccess) return e;
        for (int c0 = 0; c0 < ncol; c0 += kMultiCols) {
            const int k = ncol - c0 < kMultiCols ? ncol - c0 : kMultiCols;
            // sorted results of column j of this column block: so + 4 j cnt (phi, ex, ey, ez)
            OutCols o = {{phi ? so : nullptr, ex ? so + cc : nullptr, ey ? so + 2 * cc : nullptr,
                          ez ? so + 3 * cc : nullptr},
                         (int64_t)(4 * cc)};
            eval_chunk(drec, sigma + (size_t)c0 * n, n, k, sh, img, mixed, near_factor, sp, sp + cc, sp + 2 * cc,
                       cnt, o, w, Lc, first, s);
            for (int j = 0; j < k; ++j) {
                const size_t col = (size_t)(c0 + j) * mm + (size_t)p0;
                launch_unorder4(so + 4 * (size_t)j * cc, perm, cnt, phi ? phi + col : nullptr,
                                ex ? ex + col : nullptr, ey ? ey + col : nullptr, ez ? ez + col : nullptr, s);
            }
        }
    }
    return hipGetLastError();
}

}  // namespace nebem
