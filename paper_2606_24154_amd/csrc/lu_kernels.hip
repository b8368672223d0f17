// lu_kernels.hip -- dense LU factorisation with row pivoting and triangular
// solves on gfx950 (paper Eq. Matrix, K sigma = phi, and Algorithm 1's LU
// factorisation; the inverse is never formed, new right-hand sides use the
// resident factors).
//
// Blocked right-looking factorisation, column-major A with leading
// dimension n, in two levels: outer blocks of kOuterNB columns, each
// factored by panels of kNB columns whose updates stay inside the outer
// block, followed by one update of the rest of the matrix with the whole
// outer block (K = kOuterNB), so the trailing matrix is read and written
// once per outer block instead of once per panel:
//   for each outer block [K0, K1):
//     for each panel [k, k+kb) of it:
//       1. panel factorisation: every workgroup owns 64 or 256 consecutive rows.
//          Normally one cooperative launch for the whole panel, the rows kept
//          in LDS and the pivots agreed on through memory (k_panel_fused);
//          if the device cannot hold all of the panel's workgroups at once,
//          one launch per column: a launch eliminates column c on its rows
//          (scale by the pivot, rank-1 update of the rest of the panel) and
//          then finds the largest |a| of column c+1 among its rows; the last
//          workgroup to finish (atomic counter, no spinning) reduces the
//          per-workgroup maxima, records the pivot (first index among equal
//          maxima) and swaps the two rows inside the panel;
//       2. the same row swaps applied to every column outside the panel;
//       3. U = L11^-1 A for the columns [k+kb, K1) (unit lower solve, LDS);
//       4. A -= L21 U on rows [k+kb, n) x columns [k+kb, K1) (MFMA);
//     5. U12 = L11^-1 A12 for the columns [K1, n), panel by panel (step 3 and
//        an MFMA update of the outer block's lower rows);
//     6. A22 -= L21 U12 on rows and columns [K1, n), K = K1 - K0 (MFMA).
// T = double uses v_mfma_f64_16x16x4_f64, T = float v_mfma_f32_16x16x4_f32.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>
#include <cstdint>
#include <cstdlib>
#include <cmath>

#include "lu_internal.hpp"

namespace nebem {


// Lane i's value broadcast to the wave (i uniform): v_readlane, no LDS.
__device__ __forceinline__ double lane_bcast(double v, int i)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), i);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), i);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_bcast(float v, int i)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
}

// ------------------------------------------------------------- panel step
// c: column eliminated by this launch (c == k - 1: none, pivot search only).
template <typename T>
__global__ __launch_bounds__(kPB) void k_panel(T *__restrict__ A, int n, int k, int kb, int c,
                                               int *__restrict__ ipiv, T *__restrict__ pval,
                                               int *__restrict__ pidx, int *__restrict__ counter,
                                               int *__restrict__ info)
{
    __shared__ T urow[kNB];
    __shared__ T red_v[kPB];
    __shared__ int red_i[kPB];
    __shared__ int am_last;
    const int tid = threadIdx.x;
    const int r = k + blockIdx.x * kPB + tid;
    const int kend = k + kb;
    const int cn = c + 1;  // column whose pivot is searched
    T vnext = T(0);
    if (c >= k) {
        if (tid < kend - c) urow[tid] = A[(size_t)(c + tid) * n + c];
        __syncthreads();
        const T piv = urow[0];
        if (r > c && r < n) {
            // the row's entries in columns c .. kend-1 are loaded 32 at a time
            // and all in flight together
            T l = A[(size_t)c * n + r];
            for (int c0 = c + 1; c0 < kend; c0 += 32) {
                T v[32];
#pragma unroll
                for (int t = 0; t < 32; ++t) v[t] = (c0 + t < kend) ? A[(size_t)(c0 + t) * n + r] : T(0);
                if (c0 == c + 1) {
                    l = (piv != T(0)) ? l / piv : l;
                    A[(size_t)c * n + r] = l;
                }
#pragma unroll
                for (int t = 0; t < 32; ++t)
                    if (c0 + t < kend) {
                        const T w = v[t] - l * urow[c0 + t - c];
                        A[(size_t)(c0 + t) * n + r] = w;
                        if (c0 + t == cn) vnext = w;
                    }
            }
            if (c + 1 >= kend) {
                l = (piv != T(0)) ? l / piv : l;
                A[(size_t)c * n + r] = l;
            }
        }
    } else if (r < n && cn < kend) {
        vnext = A[(size_t)cn * n + r];
    }
    if (cn >= kend) return;  // last column of the panel: nothing to search
    // block argmax of |A[r, cn]| over r >= cn (first index among equal maxima)
    const bool valid = r >= cn && r < n;
    red_v[tid] = valid ? fabs(vnext) : T(-1);
    red_i[tid] = valid ? r : 0x7fffffff;
    __syncthreads();
    for (int s = kPB / 2; s > 0; s >>= 1) {
        if (tid < s) {
            const T a = red_v[tid], b = red_v[tid + s];
            const int ia = red_i[tid], ib = red_i[tid + s];
            if (b > a || (b == a && ib < ia)) {
                red_v[tid] = b;
                red_i[tid] = ib;
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        pval[blockIdx.x] = red_v[0];
        pidx[blockIdx.x] = red_i[0];
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) am_last = (atomicAdd(counter, 1) == (int)gridDim.x - 1);
    __syncthreads();
    if (!am_last) return;
    __threadfence();
    // last workgroup: reduce the per-workgroup maxima
    T bv = T(-1);
    int bi = 0x7fffffff;
    for (int b = tid; b < (int)gridDim.x; b += kPB) {
        const T v = pval[b];
        const int i = pidx[b];
        if (v > bv || (v == bv && i < bi)) {
            bv = v;
            bi = i;
        }
    }
    red_v[tid] = bv;
    red_i[tid] = bi;
    __syncthreads();
    for (int s = kPB / 2; s > 0; s >>= 1) {
        if (tid < s) {
            const T a = red_v[tid], b = red_v[tid + s];
            const int ia = red_i[tid], ib = red_i[tid + s];
            if (b > a || (b == a && ib < ia)) {
                red_v[tid] = b;
                red_i[tid] = ib;
            }
        }
        __syncthreads();
    }
    int p = red_i[0];
    const T pv = red_v[0];
    if (p < cn || p >= n) p = cn;  // no usable pivot (column all NaN): no swap, flagged below
    if (tid == 0) {
        ipiv[cn] = p;
        if (!(pv > T(0))) atomicMin(info, cn);
        *counter = 0;
    }
    if (p != cn && tid < kb) {
        const size_t col = (size_t)(k + tid) * n;
        const T a = A[col + cn], b = A[col + p];
        A[col + cn] = b;
        A[col + p] = a;
    }
}

// --------------------------------------------- values passed between workgroups
// Values that workgroups of one launch pass to each other are published as
// 64-bit words with a tag in the low half -- the two halves of a double, or a
// float -- so that a reader knows from the words themselves that they are the
// ones it waits for, with no flag to order after the data and no fence.  Every
// wait is bounded (kSpinLimit polls, seconds): one that gives up sets *timeout,
// every wait that then sees the flag returns, the launches run to their end and
// the host reports an error instead of the device hanging.
constexpr unsigned kSpinLimit = 1u << 22;
template <typename T>
struct Words {
    static constexpr int N = sizeof(T) / 4;
};
__device__ __forceinline__ void put_words(uint64_t *w, int64_t stride, double v, unsigned tag)
{
    __hip_atomic_store(w, ((uint64_t)(unsigned)__double2hiint(v) << 32) | tag, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + stride, ((uint64_t)(unsigned)__double2loint(v) << 32) | tag, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_words(uint64_t *w, int64_t, float v, unsigned tag)
{
    __hip_atomic_store(w, ((uint64_t)(unsigned)__float_as_int(v) << 32) | tag, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
// words of one value, and whether they carry the tag
template <typename T>
struct Taken {
    uint64_t w[Words<T>::N];
    __device__ __forceinline__ void load(const uint64_t *p, int64_t stride)
    {
#pragma unroll
        for (int k = 0; k < Words<T>::N; ++k)
            w[k] = __hip_atomic_load(p + k * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ bool is(unsigned tag) const
    {
        bool ok = true;
#pragma unroll
        for (int k = 0; k < Words<T>::N; ++k) ok = ok && (unsigned)w[k] == tag;
        return ok;
    }
    __device__ __forceinline__ T value() const;
};
template <>
__device__ __forceinline__ double Taken<double>::value() const
{
    return __hiloint2double((int)(w[0] >> 32), (int)(w[1] >> 32));
}
template <>
__device__ __forceinline__ float Taken<float>::value() const
{
    return __int_as_float((int)(w[0] >> 32));
}
// after a failed poll: whether to give up
__device__ __forceinline__ bool gives_up(unsigned polls, int *timeout)
{
    if (polls < kSpinLimit &&
        !((polls & 63) == 63 && __hip_atomic_load(timeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
        return false;
    atomicExch(timeout, 1);
    return true;
}

// Largest value over the wave (no NaN among them), by DPP: rows of 16, then
// the rows' last lanes broadcast; lane 63 holds the result.
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <typename T>
__device__ __forceinline__ T wave_max(T v)
{
    v = fmax(v, dpp<0x111>(v));  // row_shr 1, 2, 4, 8
    v = fmax(v, dpp<0x112>(v));
    v = fmax(v, dpp<0x114>(v));
    v = fmax(v, dpp<0x118>(v));
    v = fmax(v, dpp<0x142>(v));  // row_bcast 15, 31
    v = fmax(v, dpp<0x143>(v));
    return lane_bcast(v, 63);
}

// --------------------------------------------- single-launch panel
// The whole panel [k, k+kb) x rows [k, n) factored by one cooperative launch
// (all G workgroups resident at once): workgroup b keeps its 64 NW rows of the
// panel in LDS for all kb columns.  Per column c:
//   1. each workgroup finds its candidate (largest |a_rc|, r >= c, first
//      index among equal maxima) and publishes it; then the previous column's
//      update of the columns past c is made up for, and the candidate's row
//      is published, and row c by the workgroup that owns it;
//   2. every wave reads the G candidates and reduces them in the same total
//      order, so all agree on the pivot row p, and takes p's row;
//   3. it swaps rows c and p if it owns either, divides, and eliminates column
//      c from column c + 1 alone: the next candidates need no more.
// What bounds it is the chain of a write and two dependent reads through memory
// per column, ~1.5 us of 2.2 us at n = 8064 (panels 18.2 ms; with a fenced grid
// barrier, a reduction over the workgroup and the whole update inside the chain
// 5.8 us, 47 ms).  NW = 1 has no workgroup barrier at all and spreads the rows over
// the most CUs: 144 us a panel at n = 8064 where NW = 4 takes 163.  It is taken
// while G stays at most kLoneWaves, the four candidates that a lane reads at once
// (panel_rule.hpp).
// A wave of its own for the reads was slower (two barriers a column: 204 us).
// Slots are double-buffered by column parity: a slot is written again two
// columns later, when the writer has read the next column's candidates of all
// workgroups, and each published those after its last read of the slot.  Tags are
// column numbers, so the words are cleared once per factorisation.
constexpr int kPanelPad = 8;

// s[u stride] -= l u[u] for N columns of a row
template <int N, typename T>
__device__ __forceinline__ void update_columns(T *s, int stride, const T *u, T l)
{
    T v[N], w[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        v[q] = s[q * stride];
        w[q] = u[q];
    }
#pragma unroll
    for (int q = 0; q < N; ++q) s[q * stride] = fma(-l, w[q], v[q]);
}

template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void k_panel_fused(T *__restrict__ A, int n, int k, int kb,
                                                         int *__restrict__ ipiv, int *__restrict__ info,
                                                         uint64_t *__restrict__ words, int *__restrict__ timeout)
{
    constexpr int kKeySets = panel_key_sets(NW, sizeof(T));
    constexpr int W = Words<T>::N, R = 64 * NW, LD = R + 1;  // odd: a row's entries lie in different banks
    // this workgroup's rows of the panel, S[col * LD + row]; an update's last batch
    // may reach past the panel's columns, into slots that nothing else uses
    __shared__ T S[(kNB + kPanelPad) * LD];
    __shared__ T urow[NW][kNB + kPanelPad];
    __shared__ T sv[2][NW];
    __shared__ int si[2][NW];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, b = blockIdx.x, G = gridDim.x;
    const int r = k + b * R + t;
    const bool live = r < n;
    uint64_t *const keys = words, *const rows = words + (size_t)2 * (W + 1) * G;
    uint64_t *const tops = rows + (size_t)2 * G * W * kNB;
    const T *Ar = A + (size_t)k * n + min(r, n - 1);
    for (int j0 = 0; j0 < kb; j0 += 32) {  // 32 loads in flight per thread
        T v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = Ar[(size_t)min(j0 + u, kb - 1) * n];
#pragma unroll
        for (int u = 0; u < 32; ++u) S[(j0 + u) * LD + t] = live ? v[u] : T(0);
    }
    T cur = S[t], l = T(0);
    bool act = false;  // the last column's elimination reaches this row
    for (int j = 0; j < kb; ++j) {
        const int c = k + j, sl = j & 1;
        const unsigned tag = (unsigned)c + 1;
        // 1. this workgroup's candidate (a NaN entry never wins)
        const T x0 = fabs(cur);
        const T x = (live && r >= c && x0 == x0) ? x0 : T(-1);
        T mx = wave_max(x);
        int il = 64 * wave + __ffsll((unsigned long long)__ballot(x == mx)) - 1;
        if constexpr (NW > 1) {
            if (lane == 0) {
                sv[sl][wave] = mx;
                si[sl][wave] = il;
            }
            __syncthreads();
            mx = sv[sl][0];
            il = si[sl][0];
#pragma unroll
            for (int q = 1; q < NW; ++q)
                if (sv[sl][q] > mx) {
                    mx = sv[sl][q];
                    il = si[sl][q];
                }
        }
        il = __builtin_amdgcn_readfirstlane(il);
        if (wave == 0) {
            if (lane == 0) put_words(keys + (size_t)sl * (W + 1) * G + b, G, mx, tag);
            if (lane == 1)
                __hip_atomic_store(keys + ((size_t)sl * (W + 1) + W) * G + b,
                                   ((uint64_t)(unsigned)(k + b * R + il) << 32) | tag, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        if (act) {
            const T *up = urow[wave];
            int j0 = j + 1;
            for (; j0 + 8 < kb; j0 += 16) update_columns<16>(S + j0 * LD + t, LD, up + j0, l);
            if (j0 < kb) update_columns<8>(S + j0 * LD + t, LD, up + j0, l);
        }
        if (wave == il >> 6 && lane < kb)
            put_words(rows + (((size_t)sl * G + b) * W) * kNB + lane, kNB, S[lane * LD + il], tag);
        if (b == 0 && wave == 0 && lane < kb) put_words(tops + (size_t)sl * W * kNB + lane, kNB, S[lane * LD + j], tag);
        // 2. the pivot
        T kv[kKeySets];
        int ki[kKeySets];
        for (unsigned polls = 0;; ++polls) {
            Taken<T> q[kKeySets];
            uint64_t qi[kKeySets];
#pragma unroll
            for (int u = 0; u < kKeySets; ++u)
                if (64 * u < G) {
                    const uint64_t *key = keys + (size_t)sl * (W + 1) * G + min(64 * u + lane, G - 1);
                    q[u].load(key, G);
                    qi[u] = __hip_atomic_load(key + (size_t)W * G, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            bool ok = true;
#pragma unroll
            for (int u = 0; u < kKeySets; ++u) {
                kv[u] = T(-1);
                ki[u] = INT_MAX;
                if (64 * u < G) {
                    ok = ok && q[u].is(tag) && (unsigned)qi[u] == tag;
                    kv[u] = q[u].value();
                    ki[u] = (int)(qi[u] >> 32);
                }
            }
            if (__ballot(!ok) == 0 || gives_up(polls, timeout)) break;
        }
        T pv = kv[0];
#pragma unroll
        for (int u = 1; u < kKeySets; ++u) pv = fmax(pv, kv[u]);
        pv = wave_max(pv);
        int p = c;  // no usable pivot (column all NaN): no swap, flagged below
#pragma unroll
        for (int u = kKeySets - 1; u >= 0; --u) {
            const unsigned long long m = __ballot(kv[u] == pv);
            if (m) p = __builtin_amdgcn_readlane(ki[u], __ffsll(m) - 1);
        }
        if (pv < T(0) || p < c || p >= n) p = c;
        // its row, and row c where that goes
        const int bw = (p - k) / R;
        const bool mine = p != c && (p - k) >> 6 == b * NW + wave;
        const uint64_t *top = tops + (size_t)sl * W * kNB + min(lane, kb - 1);
        const uint64_t *win = p == c ? top : rows + (((size_t)sl * G + bw) * W) * kNB + min(lane, kb - 1);
        Taken<T> uw, tw;
        for (unsigned polls = 0;; ++polls) {
            uw.load(win, kNB);
            bool ok = true;
            if (mine) {
                tw.load(top, kNB);
                ok = tw.is(tag);
            }
            ok = ok && uw.is(tag);
            if (__ballot(!ok) == 0 || gives_up(polls, timeout)) break;
        }
        const T u = uw.value();
        if (lane < kb) {
            urow[wave][lane] = u;
            if (p != c && b == 0 && wave == 0) S[lane * LD + j] = u;
            if (mine) S[lane * LD + (p - k - b * R)] = tw.value();
        }
        if (b == 0 && t == 0) {
            ipiv[c] = p;
            if (!(pv > T(0))) atomicMin(info, c);
        }
        // 3. elimination from the next column
        const T piv = lane_bcast(u, j), un = lane_bcast(u, min(j + 1, kb - 1));
        act = live && r > c;
        if (act) {
            const T s = S[j * LD + t];
            l = (piv != T(0)) ? s / piv : s;
            S[j * LD + t] = l;
            if (j + 1 < kb) {
                cur = fma(-l, un, S[(j + 1) * LD + t]);
                S[(j + 1) * LD + t] = cur;
            }
        }
    }
    if (live)
        for (int jj = 0; jj < kb; ++jj) A[(size_t)(k + jj) * n + r] = S[jj * LD + t];
}

// Row swaps of panel [k, k+kb) applied to every column outside the panel.  Each
// wave first works out, one row per lane, where the kb swaps together bring the
// panel's rows from (src) and what goes to the rows below that they touch (osrc, in
// the lane of the first swap with that row), then moves kSwapCols columns, one at a
// time per lane and row: all loads, then all stores.  One column per lane and
// its swaps one after the other, as LAPACK has it, read 64 cache lines per
// instruction in a chain of 64: 40 us for 8000 FP64 columns (n = 8064), now 14; FP32
// columns of a matrix of normal entries 79 us, now 22.  Panels in which no row moves
// (diagonally dominant systems) took 5.8 us and 6.4 with the permutation worked out for
// nothing, 2.7 now.
constexpr int kSwapCols = 8;
template <typename T>
__global__ __launch_bounds__(256) void k_laswp(T *__restrict__ A, int n, int k, int kb,
                                               const int *__restrict__ ipiv)
{
    const int lane = threadIdx.x & 63;
    const int j0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * kSwapCols;
    const int ncol = n - kb;
    if (j0 >= ncol) return;
    const bool top = lane < kb;
    const int p = top ? ipiv[k + lane] - k : lane;
    if (__ballot(p != lane) == 0) return;  // no row moves
    int src = lane, osrc = p;
    bool first = false;  // this lane's swap is the first with a row below the panel
    for (int t = 0; t < kb; ++t) {
        const int pt = __builtin_amdgcn_readlane(p, t);
        if (pt == t) continue;
        const int a = __builtin_amdgcn_readlane(src, t);
        if (pt < kb) {
            const int b = __builtin_amdgcn_readlane(src, pt);
            src = lane == t ? b : lane == pt ? a : src;
        } else {
            const int s = __ffsll((unsigned long long)__ballot(top && p == pt)) - 1;
            const int b = __builtin_amdgcn_readlane(osrc, s);
            src = lane == t ? b : src;
            osrc = lane == s ? a : osrc;
            first = first || lane == s;
        }
    }
    const bool mv = top && src != lane, ov = first && osrc != p;
    T v[kSwapCols], w[kSwapCols];
#pragma unroll
    for (int c = 0; c < kSwapCols; ++c) {
        const int j = min(j0 + c, ncol - 1);
        const T *col = A + (size_t)(j >= k ? j + kb : j) * n + k;
        if (mv) v[c] = col[src];
        if (ov) w[c] = col[osrc];
    }
    // no store before the last load: rows are sources and targets of different lanes
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int c = 0; c < kSwapCols; ++c) {
        const int j = j0 + c;
        if (j >= ncol) break;
        T *col = A + (size_t)(j >= k ? j + kb : j) * n + k;
        if (mv) col[lane] = v[c];
        if (ov) col[p] = w[c];
    }
}

// U = L11^-1 A[k:k+kb, j] for the columns j in [jb, je), 4 kTrsmCols per workgroup
// (unit lower L11 = A[k:k+kb, k:k+kb], kb <= 64).  Wave w solves kTrsmCols columns with
// lane r holding row r of each: the entry solved at step i reaches the other lanes
// by readlane, so the waves run without barriers; every subtraction comes in the
// order of plain forward substitution.  VALU bound on few workgroups: 16 columns a
// wave took 22 us for 4000 FP64 columns (63 workgroups), 4 columns 10 us, 8 columns 17.
// More columns, which read L11 less often, do not pay at large sizes either: 38 000 FP64
// columns 46.5 us at 16 a wave, 39.7 at 4; 68 000 FP32 columns 45.5, 40.7.
constexpr int kTrsmCols = 4;
template <typename T>
__global__ __launch_bounds__(256) void k_trsm(T *__restrict__ A, int n, int k, int kb, int jb, int je)
{
    constexpr int NC = kTrsmCols;
    __shared__ T L[kNB][kNB + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int j0 = jb + blockIdx.x * (4 * NC);
    const int ncol = min(4 * NC, je - j0);
    T x[NC];
    {
        // 16 + NC loads per thread, all issued before the first is used
        T lv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = tid + 256 * u, rr = e & 63, cc = e >> 6;
            lv[u] = (rr < kb && cc < kb) ? A[(size_t)(k + cc) * n + k + rr] : T(0);
        }
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int xc = NC * w + u;
            x[u] = (lane < kb && xc < ncol) ? A[(size_t)(j0 + xc) * n + k + lane] : T(0);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = tid + 256 * u;
            L[e & 63][e >> 6] = lv[u];
        }
    }
    __syncthreads();
    const bool row_in = lane < kb;
    for (int i = 0; i < kb - 1; ++i) {
        const T l = L[lane][i];
        const bool upd = row_in && lane > i;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const T xi = lane_bcast(x[q], i);
            const T u = x[q] - l * xi;
            x[q] = upd ? u : x[q];
        }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        const int xc = NC * w + q;
        if (row_in && xc < ncol) A[(size_t)(j0 + xc) * n + k + lane] = x[q];
    }
}

// ------------------------------------------------------------------ GEMM
// C -= L21 U12 over the trailing matrix rows/cols [k+kb, n), K = kb <= 64.
// Workgroup tile 64 x 64, four waves each 32 x 32 (2 x 2 MFMA tiles).  The
// MFMA computes the transposed tile, D'[i][j] = C[row j][col i], so that the
// 16 lanes holding one output column walk 16 consecutive rows (contiguous in
// the column-major matrix).  MFMA 16x16x4 operand layout (wave64, checked
// on gfx950): A operand (16 x 4) element [i][kk] in lane i + 16 kk; B operand
// (4 x 16) element [kk][j] in lane j + 16 kk; result element [i][j] in lane
// j + 16 (i / 4), register i % 4 for f32, but lane j + 16 (i % 4), register
// i / 4 for f64.
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma16(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// result row i held by (lane group g = lane / 16, register v)
template <typename T>
struct Acc;
template <>
struct Acc<double> {
    typedef d4 type;
    static __device__ __forceinline__ int row(int g, int v) { return 4 * v + g; }
};
template <>
struct Acc<float> {
    typedef f4 type;
    static __device__ __forceinline__ int row(int g, int v) { return 4 * g + v; }
};

constexpr int kGT = 64;     // trailing-update workgroup tile (rows and columns)
constexpr int kKC = 32;     // K chunk staged in LDS at a time (keeps several workgroups per CU)
constexpr int kXCD = 8;     // accelerator complex dies; workgroups are dealt to them round-robin
constexpr int kGroupR = 8;  // tile rows per group of the tile order

// C[r0:r1, c0:c1] -= A[r0:r1, k:k+kb] A[k:k+kb, c0:c1] for any kb.  1-D grid
// of kXCD * per_xcd workgroups: workgroup b works on linear tile
// (b % kXCD) * per_xcd + b / kXCD, so each die takes one contiguous range of
// the tile order, and that order walks groups of kGroupR tile rows column by
// column -- the workgroups a die runs at one time share their L21 and U12
// tiles in its L2.
template <typename T>
__global__ __launch_bounds__(256) void k_gemm_update(T *__restrict__ A, int n, int k, int kb, int r0, int r1, int c0,
                                                     int c1, int per_xcd)
{
    typedef typename Acc<T>::type V4;
    // One K chunk of the operands.  Strides chosen so that the 32 lanes of
    // each half-wave hit distinct LDS banks on the staging stores and on the
    // MFMA operand loads: -L21 row-major in k (rows contiguous, as in A),
    // U12 column-major (k contiguous, as in A).
    __shared__ T sL[kKC][kGT + 16];  // sL[kk][row] = -L21
    __shared__ T sU[kGT][kKC + 2];   // sU[col][kk] =  U12
    const int nt_r = (r1 - r0 + kGT - 1) / kGT, nt_c = (c1 - c0 + kGT - 1) / kGT;
    const int lin = (int)(blockIdx.x % kXCD) * per_xcd + (int)(blockIdx.x / kXCD);
    if (lin >= nt_r * nt_c) return;  // whole workgroup: padding of the last die's range
    const int gsz = kGroupR * nt_c;
    const int first = (lin / gsz) * kGroupR;
    const int rows_in = min(kGroupR, nt_r - first);
    const int within = lin % gsz;
    const int row0 = r0 + (first + within % rows_in) * kGT;
    const int col0 = c0 + (within / rows_in) * kGT;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wr = (wave & 1) * 32, wc = (wave >> 1) * 32;  // wave's 32x32 sub-tile
    const int li = lane & 15, lk = lane >> 4;
    // The accumulators start from C itself (loads issued before the operand
    // staging so that the two overlap); the MFMA chain then adds (-L21) U12.
    // Every global load is unconditional, from an index clamped into the
    // matrix, and out-of-range entries are replaced when they reach LDS (or
    // are never stored, for C): a load under a branch would have to complete
    // inside that branch, one memory latency per load.
    V4 acc[2][2];
#pragma unroll
    for (int tc = 0; tc < 2; ++tc)
#pragma unroll
        for (int tr = 0; tr < 2; ++tr)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gc = col0 + wc + 16 * tc + Acc<T>::row(lk, v);
                const int gr = row0 + wr + 16 * tr + li;
                acc[tc][tr][v] = A[(size_t)min(gc, c1 - 1) * n + min(gr, r1 - 1)];
            }
    // K in chunks of kKC; entries past kb are staged as zeros, so every chunk
    // has the same compile-time shape (index arithmetic by shifts, the MFMA
    // loop fully unrolled).  FP32: the next chunk's global loads are issued
    // into registers before the current chunk's MFMAs and stored to LDS
    // after them, so their latency hides behind the matrix-core work.  FP64:
    // the chunk's loads are issued together when it is needed (the prefetch
    // registers would halve the resident workgroups).
    constexpr bool kPrefetch = sizeof(T) == 4;
    constexpr int kPer = kKC * kGT / 256;  // staged entries per thread and operand
    T pl[kPer], pu[kPer];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = tid + 256 * u;
            const int rr = e % kGT, kl = e / kGT;
            pl[u] = A[(size_t)(k + min(k0 + kl, kb - 1)) * n + min(row0 + rr, r1 - 1)];
            const int ku = e % kKC, cc = e / kKC;
            pu[u] = A[(size_t)min(col0 + cc, c1 - 1) * n + k + min(k0 + ku, kb - 1)];
        }
    };
    auto stage = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = tid + 256 * u;
            const int rr = e % kGT, kl = e / kGT;
            sL[kl][rr] = (row0 + rr < r1 && k0 + kl < kb) ? -pl[u] : T(0);
            const int ku = e % kKC, cc = e / kKC;
            sU[cc][ku] = (col0 + cc < c1 && k0 + ku < kb) ? pu[u] : T(0);
        }
    };
    if constexpr (kPrefetch) fetch(0);
    for (int k0 = 0; k0 < kb; k0 += kKC) {
        if (k0) __syncthreads();  // every wave is done reading the previous chunk
        if constexpr (!kPrefetch) fetch(k0);
        stage(k0);
        __syncthreads();
        if constexpr (kPrefetch) {
            if (k0 + kKC < kb) fetch(k0 + kKC);
        }
#pragma unroll
        for (int kk = 0; kk < kKC; kk += 4) {
            // A operand: U12 columns (i index), B operand: -L21 rows (j index)
            const T u0 = sU[wc + li][kk + lk], u1 = sU[wc + 16 + li][kk + lk];
            const T l0 = sL[kk + lk][wr + li], l1 = sL[kk + lk][wr + 16 + li];
            acc[0][0] = mfma16(u0, l0, acc[0][0]);
            acc[0][1] = mfma16(u0, l1, acc[0][1]);
            acc[1][0] = mfma16(u1, l0, acc[1][0]);
            acc[1][1] = mfma16(u1, l1, acc[1][1]);
        }
    }
    // lane holds D'[i][j] for i = Acc::row(lk, v) (column offset), j = li (row offset)
#pragma unroll
    for (int tc = 0; tc < 2; ++tc)
#pragma unroll
        for (int tr = 0; tr < 2; ++tr)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gc = col0 + wc + 16 * tc + Acc<T>::row(lk, v);
                const int gr = row0 + wr + 16 * tr + li;
                if (gc < c1 && gr < r1) A[(size_t)gc * n + gr] = acc[tc][tr][v];
            }
}

// The same update with 128 x 128 workgroup tiles for large trailing
// matrices: four waves of 64 x 64 (4 x 4 MFMA tiles, 16 accumulators in the
// matrix-core registers), K in chunks of kBK staged through two LDS buffers,
// the next chunk's global loads held in registers while the current chunk's
// MFMAs run, one workgroup barrier per chunk.  Per output element the MFMA
// sequence (accumulator from C, K in steps of 4 in increasing order) is that
// of k_gemm_update, so both give bit-identical results; the larger tile
// halves the operand bytes staged per FLOP.
constexpr int kBT = 128;  // large-update workgroup tile (rows and columns)
constexpr int kBK = 16;   // its K chunk

template <typename T>
__global__ __launch_bounds__(256, 2) void k_gemm_update_big(T *__restrict__ A, int n, int k, int kb, int r0, int r1,
                                                            int c0, int c1, int per_xcd)
{
    typedef typename Acc<T>::type V4;
    // strides as in k_gemm_update: consecutive k of sL, and the 16 columns a
    // half-wave reads from sU, fall on distinct LDS banks
    __shared__ T sL[2][kBK][kBT + 16];  // sL[buf][kk][row] = -L21
    __shared__ T sU[2][kBT][kBK + 2];   // sU[buf][col][kk] =  U12
    const int nt_r = (r1 - r0 + kBT - 1) / kBT, nt_c = (c1 - c0 + kBT - 1) / kBT;
    const int lin = (int)(blockIdx.x % kXCD) * per_xcd + (int)(blockIdx.x / kXCD);
    if (lin >= nt_r * nt_c) return;  // whole workgroup: padding of the last die's range
    const int gsz = kGroupR * nt_c;
    const int first = (lin / gsz) * kGroupR;
    const int rows_in = min(kGroupR, nt_r - first);
    const int within = lin % gsz;
    const int row0 = r0 + (first + within % rows_in) * kBT;
    const int col0 = c0 + (within / rows_in) * kBT;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wr = (wave & 1) * 64, wc = (wave >> 1) * 64;  // wave's 64 x 64 sub-tile
    const int li = lane & 15, lk = lane >> 4;
    // Every global load is unconditional, from an index clamped into the
    // matrix, and out-of-range entries are replaced when they reach LDS or
    // the accumulators: a load under a branch would have to complete inside
    // that branch, one memory latency per load.
    V4 acc[4][4];
#pragma unroll
    for (int tc = 0; tc < 4; ++tc)
#pragma unroll
        for (int tr = 0; tr < 4; ++tr)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gc = col0 + wc + 16 * tc + Acc<T>::row(lk, v);
                const int gr = row0 + wr + 16 * tr + li;
                acc[tc][tr][v] = A[(size_t)min(gc, c1 - 1) * n + min(gr, r1 - 1)];
            }
    constexpr int kPer = kBK * kBT / 256;  // staged entries per thread and operand
    T pl[kPer], pu[kPer];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = tid + 256 * u;
            const int rr = e % kBT, kl = e / kBT;
            pl[u] = A[(size_t)(k + min(k0 + kl, kb - 1)) * n + min(row0 + rr, r1 - 1)];
            const int ku = e % kBK, cc = e / kBK;
            pu[u] = A[(size_t)min(col0 + cc, c1 - 1) * n + k + min(k0 + ku, kb - 1)];
        }
    };
    auto stage = [&](int b, int k0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = tid + 256 * u;
            const int rr = e % kBT, kl = e / kBT;
            sL[b][kl][rr] = (row0 + rr < r1 && k0 + kl < kb) ? -pl[u] : T(0);
            const int ku = e % kBK, cc = e / kBK;
            sU[b][cc][ku] = (col0 + cc < c1 && k0 + ku < kb) ? pu[u] : T(0);
        }
    };
    const int nch = (kb + kBK - 1) / kBK;
    fetch(0);
    stage(0, 0);
    if (nch > 1) fetch(kBK);
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
        const int b = c & 1;
#pragma unroll
        for (int kk = 0; kk < kBK; kk += 4) {
            T u[4], l[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u[t] = sU[b][wc + 16 * t + li][kk + lk];
                l[t] = sL[b][kk + lk][wr + 16 * t + li];
            }
#pragma unroll
            for (int tc = 0; tc < 4; ++tc)
#pragma unroll
                for (int tr = 0; tr < 4; ++tr) acc[tc][tr] = mfma16(u[tc], l[tr], acc[tc][tr]);
        }
        // the other buffer was last read in chunk c - 1, which every wave
        // finished before the previous barrier
        if (c + 1 < nch) {
            stage(b ^ 1, (c + 1) * kBK);
            if (c + 2 < nch) fetch((c + 2) * kBK);
        }
        __syncthreads();
    }
#pragma unroll
    for (int tc = 0; tc < 4; ++tc)
#pragma unroll
        for (int tr = 0; tr < 4; ++tr)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gc = col0 + wc + 16 * tc + Acc<T>::row(lk, v);
                const int gr = row0 + wr + 16 * tr + li;
                if (gc < c1 && gr < r1) A[(size_t)gc * n + gr] = acc[tc][tr][v];
            }
}

template <typename T>
static void gemm_update(T *A, int n, int k, int kb, int r0, int r1, int c0, int c1, hipStream_t s)
{
    if (r1 <= r0 || c1 <= c0 || kb <= 0) return;
    if (r1 - r0 >= 2 * kBT && c1 - c0 >= 2 * kBT) {
        const int tiles = ((r1 - r0 + kBT - 1) / kBT) * ((c1 - c0 + kBT - 1) / kBT);
        const int per_xcd = (tiles + kXCD - 1) / kXCD;
        hipLaunchKernelGGL(k_gemm_update_big<T>, dim3((unsigned)(per_xcd * kXCD)), dim3(256), 0, s, A, n, k, kb, r0,
                           r1, c0, c1, per_xcd);
        return;
    }
    const int tiles = ((r1 - r0 + kGT - 1) / kGT) * ((c1 - c0 + kGT - 1) / kGT);
    const int per_xcd = (tiles + kXCD - 1) / kXCD;
    hipLaunchKernelGGL(k_gemm_update<T>, dim3((unsigned)(per_xcd * kXCD)), dim3(256), 0, s, A, n, k, kb, r0, r1, c0,
                       c1, per_xcd);
}

template <typename T>
static void trsm(T *A, int n, int k, int kb, int jb, int je, hipStream_t s)
{
    if (je <= jb) return;
    hipLaunchKernelGGL(k_trsm<T>, dim3((unsigned)((je - jb + 4 * kTrsmCols - 1) / (4 * kTrsmCols))), dim3(256), 0, s, A,
                       n, k, kb, jb, je);
}

// ------------------------------------------------------ triangular solves
// L W = P B, then U X = W, each by one launch in which the 64-row blocks pass
// their solutions on as they have them: workgroup b sums its block row against
// the solved blocks in order (four waves, 16 columns of a block each, the next
// block's factor entries and solutions already loading), subtracts, solves its
// 64 x 64 diagonal block in one wave by substitution (lane = row, the entry
// solved at step i reaches the others by readlane) and publishes.  One launch
// per block, with a reload of the diagonal tile and a pass over the rows below
// in each, took 20 us per 64 rows; here a block adds one exchange and its own
// substitution to the chain, ~5 us, and the factors stream through beside it.
// Three solves and two residuals of n = 8064: 18.0 -> 4.4 ms.
//
// Tags are never reused within a workspace (SolveFlow), so it is cleared once.
// Workgroups take their blocks from a counter: a block only waits for blocks
// whose workgroups have started before its own, so the waits end whatever the
// device holds at once; each wait is bounded all the same.

// v / d from inv = 1/d with a residual correction, for d with |d| in a range
// whose reciprocals are exact to rounding (quotient_takes); an infinite or NaN
// product stays as it is.
__device__ __forceinline__ bool quotient_takes(double d) { return fabs(d) > 0x1p-1000 && fabs(d) < 0x1p1000; }
__device__ __forceinline__ bool quotient_takes(float d) { return fabsf(d) > 0x1p-100f && fabsf(d) < 0x1p100f; }
template <typename T>
__device__ __forceinline__ T quotient(T v, T d, T inv)
{
    const T q = v * inv, r = fma(fma(-q, d, v), inv, q);
    return isfinite(q) ? r : q;
}

// NR right-hand sides (columns of ld n).  LOWER: rhs row i is B[perm[i]] and
// the diagonal is 1; else rhs row i is B[i].
template <typename T, typename TB, int NR, bool LOWER>
__global__ __launch_bounds__(256) void k_trsv_flow(const T *__restrict__ LU, int n, const int *__restrict__ perm,
                                                   const TB *__restrict__ B, T *__restrict__ Y,
                                                   uint64_t *__restrict__ words, unsigned *__restrict__ ticket,
                                                   unsigned base, unsigned tag, int *__restrict__ timeout)
{
    __shared__ int s_block;
    __shared__ T red[4][NR][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_block = (int)(atomicAdd(ticket, 1u) - base);
    __syncthreads();
    const int nb = (n + 63) / 64;
    const int b = LOWER ? s_block : nb - 1 - s_block;
    const int r = 64 * b + lane, rc = min(r, n - 1);
    const bool in = r < n;
    // this wave's columns of block j, rows of this block row (the columns of a
    // short last block are clamped into the matrix; their solutions enter as 0)
    auto load_tile = [&](int j, T(&v)[16]) {
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = LU[(size_t)min(64 * j + 16 * wave + t, n - 1) * n + rc];
    };
    // the wave's 16 solutions of block j, one per lane < 16
    const int64_t wn = (int64_t)n * NR;
    auto load_x = [&](int j, Taken<T>(&x)[NR]) {
        const int c = min(64 * j + 16 * wave + (lane & 15), n - 1);
#pragma unroll
        for (int q = 0; q < NR; ++q) x[q].load(words + (int64_t)q * n + c, wn);
    };
    T acc[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) acc[q] = T(0);
    const int steps = LOWER ? b : nb - 1 - b;
    T v[16], vn[16];
    Taken<T> x[NR];
    if (steps > 0) {
        load_tile(LOWER ? 0 : nb - 1, v);
        load_x(LOWER ? 0 : nb - 1, x);
    }
    for (int k = 0; k < steps; ++k) {
        const int j = LOWER ? k : nb - 1 - k;
        if (k + 1 < steps) load_tile(LOWER ? j + 1 : j - 1, vn);
        for (unsigned polls = 0;; ++polls) {
            bool ok = true;
#pragma unroll
            for (int q = 0; q < NR; ++q) ok = ok && x[q].is(tag);
            if (__ballot(!ok) == 0 || gives_up(polls, timeout)) break;
            __builtin_amdgcn_s_sleep(1);
            load_x(j, x);
        }
        T xv[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) xv[q] = 64 * j + 16 * wave + (lane & 15) < n ? x[q].value() : T(0);
        if (k + 1 < steps) load_x(LOWER ? j + 1 : j - 1, x);
#pragma unroll
        for (int t = 0; t < 16; ++t)
#pragma unroll
            for (int q = 0; q < NR; ++q) acc[q] = fma(v[t], lane_bcast(xv[q], t), acc[q]);
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = vn[t];
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) red[wave][q][lane] = acc[q];
    // the diagonal block, before the barrier: entries that a row does not use,
    // those of columns past the last among them, are zeros, so the substitution
    // needs no tests
    T d[64], dd = T(1), inv = T(1), rhs = T(0);
    if (wave < NR) {
#pragma unroll
        for (int i = 0; i < 64; ++i) {
            const T e = LU[(size_t)min(64 * b + i, n - 1) * n + rc];
            d[i] = in && 64 * b + i < n && (LOWER ? i < lane : i > lane) ? e : T(0);
        }
        if (!LOWER) {
            dd = in ? LU[(size_t)rc * n + rc] : T(1);
            inv = T(1) / dd;
        }
        rhs = in ? (T)B[(size_t)wave * n + (LOWER ? perm[rc] : rc)] : T(0);
    }
    __syncthreads();
    if (wave >= NR) return;
    T y = rhs - (((red[0][wave][lane] + red[1][wave][lane]) + red[2][wave][lane]) + red[3][wave][lane]);
    // a row's value is taken at its own step: what the later steps' zeros make of
    // it (NaN, where a solution is infinite) is not used
    T out = y;
    if (LOWER) {
#pragma unroll
        for (int i = 0; i < 64; ++i) {
            out = lane == i ? y : out;
            y = fma(-d[i], lane_bcast(y, i), y);
        }
    } else if (__ballot(!quotient_takes(dd)) == 0) {
#pragma unroll
        for (int i = 63; i >= 0; --i) {
            const T qi = quotient(y, dd, inv);
            out = lane == i ? qi : out;
            y = fma(-d[i], lane_bcast(qi, i), y);
        }
    } else {
#pragma unroll
        for (int i = 63; i >= 0; --i) {
            const T qi = y / dd;
            out = lane == i ? qi : out;
            y = fma(-d[i], lane_bcast(qi, i), y);
        }
    }
    if (in) {
        put_words(words + (int64_t)wave * n + r, wn, out, tag);
        Y[(size_t)wave * n + r] = out;
    }
}

// Transposed solves with the same factors, one right-hand side, one launch
// per 64-row block: lower = 1 solves U^T w = v forward (U^T lower, diagonal
// of U), lower = 0 solves L^T v = w backward (unit diagonal).  Row r of a
// transposed factor is column r of LU, so the block's entries of row r are
// LU[r n + b0 .. b0 + 63], contiguous.  X is reduced in place on the
// unsolved side and the block's solution goes to Y: solved rows are never written to
// X, so no workgroup reads a half-updated block.
__global__ __launch_bounds__(256) void k_trsv_t_step(const double *__restrict__ LU, int n, double *__restrict__ X,
                                                     double *__restrict__ Y, int b0, int bsz, int lower)
{
    __shared__ double D[64][65];  // D[r][c] = (transposed factor)[b0 + r][b0 + c]
    __shared__ double y[64];
    const int tid = threadIdx.x;
    {
        double dv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = tid + 256 * u, c = e & 63, r = e >> 6;
            dv[u] = (r < bsz && c < bsz) ? LU[(size_t)(b0 + r) * n + b0 + c] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = tid + 256 * u;
            D[e >> 6][e & 63] = dv[u];
        }
        if (tid < 64) y[tid] = tid < bsz ? X[b0 + tid] : 0.0;
    }
    __syncthreads();
    if (tid < 64) {  // one wave: lane r holds row r
        const int lane = tid;
        const bool in = lane < bsz;
        double v = y[lane];
        if (lower) {
            for (int i = 0; i < bsz; ++i) {
                const double yi = lane_bcast(v, i) / D[i][i];
                const double u = v - D[lane][i] * yi;
                v = (lane == i) ? yi : ((in && lane > i) ? u : v);
            }
        } else {
            for (int i = bsz - 1; i >= 0; --i) {
                const double yi = lane_bcast(v, i);
                const double u = v - D[lane][i] * yi;
                v = (in && lane < i) ? u : v;
            }
        }
        if (in) y[lane] = v;
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid < bsz) Y[b0 + tid] = y[tid];
    const int lo = lower ? b0 + bsz : 0;
    const int hi = lower ? n : b0;
    const int r = lo + blockIdx.x * 256 + tid;
    if (r < hi) {
        double acc = X[r];
        const double *row = LU + (size_t)r * n + b0;
        for (int j0 = 0; j0 < bsz; j0 += 16) {
            double l[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) l[t] = (j0 + t < bsz) ? row[j0 + t] : 0.0;
#pragma unroll
            for (int t = 0; t < 16; ++t)
                if (j0 + t < bsz) acc -= l[t] * y[j0 + t];
        }
        X[r] = acc;
    }
}

// z[perm[i]] = v[i] (the inverse of the pivoting gather)
__global__ __launch_bounds__(256) void k_unpermute(const double *__restrict__ v, double *__restrict__ z,
                                                   const int *__restrict__ perm, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) z[perm[i]] = v[i];
}

// --------------------------------------------------------------- launchers
// Workgroups of k_panel_fused<T, NW> the device holds at once (0 if unknown).
template <typename T, int NW>
static int fused_capacity()
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    int coop = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_panel_fused<T, NW>, 64 * NW, 0) != hipSuccess) return 0;
    return per_cu * cus;
}

// NEBEM_PANEL_PER_COLUMN=1 in the environment selects the per-column panel
// launches everywhere (the path taken when a panel's workgroups do not fit
// on the device at once), so that tests can reach it at any size.
static bool per_column_forced()
{
    const char *e = std::getenv("NEBEM_PANEL_PER_COLUMN");
    return e && e[0] == '1';
}

template <typename T>
void lu_factor_launch(T *A, int n, int *ipiv, LUWork &w, hipStream_t s)
{
    const bool one_launch = w.words && !per_column_forced();
    const int cap1 = one_launch ? fused_capacity<T, 1>() : 0, cap4 = one_launch ? fused_capacity<T, 4>() : 0;
    bool fused_ok = cap4 > 0;
    for (int K0 = 0; K0 < n; K0 += kOuterNB) {
        const int K1 = (n - K0 < kOuterNB) ? n : K0 + kOuterNB;
        for (int k = K0; k < K1; k += kNB) {
            const int kb = (K1 - k < kNB) ? K1 - k : kNB;
            const unsigned gp = (unsigned)((n - k + kPB - 1) / kPB), g1 = (unsigned)((n - k + 63) / 64);
            const int nw = fused_ok ? panel_waves(n - k, sizeof(T), cap1, cap4) : 0;
            bool done = false;
            if (nw) {
                int a_n = n, a_k = k, a_kb = kb;
                void *args[] = {&A, &a_n, &a_k, &a_kb, &ipiv, &w.info, &w.words, &w.timeout};
                const hipError_t e =
                    nw == 1 ? hipLaunchCooperativeKernel((const void *)k_panel_fused<T, 1>, dim3(g1), dim3(64), args, 0, s)
                            : hipLaunchCooperativeKernel((const void *)k_panel_fused<T, 4>, dim3(gp), dim3(kPB), args, 0,
                                                         s);
                if (e == hipSuccess) {
                    done = true;
                } else {
                    (void)hipGetLastError();
                    fused_ok = false;  // per-column launches from here on
                }
            }
            if (!done)
                for (int c = k - 1; c < k + kb; ++c)
                    hipLaunchKernelGGL(k_panel<T>, dim3(gp), dim3(kPB), 0, s, A, n, k, kb, c, ipiv, (T *)w.pval,
                                       w.pidx, w.counter, w.info);
            if (n - kb > 0) {
                const unsigned gl = (unsigned)((n - kb + 4 * kSwapCols - 1) / (4 * kSwapCols));
                hipLaunchKernelGGL(k_laswp<T>, dim3(gl), dim3(256), 0, s, A, n, k, kb, ipiv);
            }
            trsm(A, n, k, kb, k + kb, K1, s);
            gemm_update(A, n, k, kb, k + kb, n, k + kb, K1, s);
        }
        if (K1 < n) {
            for (int b = K0; b < K1; b += kNB) {
                const int bb = (K1 - b < kNB) ? K1 - b : kNB;
                trsm(A, n, b, bb, K1, n, s);
                gemm_update(A, n, b, bb, b + bb, K1, K1, n, s);
            }
            gemm_update(A, n, K0, K1 - K0, K1, n, K1, n, s);
        }
    }
}

__global__ __launch_bounds__(256) void k_clear_words(uint64_t *__restrict__ w, int64_t len)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < len) w[i] = 0;
}

void clear_words(uint64_t *w, int64_t len, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear_words, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, w, len);
}

size_t solve_flow_bytes(int n) { return 256 + (size_t)n * kSolveCols * 2 * sizeof(uint64_t); }

void solve_flow_init(SolveFlow &f, void *mem, int n, hipStream_t s)
{
    f.ticket = (unsigned *)mem;
    f.timeout = (int *)mem + 1;
    f.words = (uint64_t *)((char *)mem + 256);
    f.launches = 0;
    clear_words((uint64_t *)mem, (int64_t)(solve_flow_bytes(n) / sizeof(uint64_t)), s);
}

template <typename T, typename TB, int NR, bool LOWER>
static void trsv_flow(const T *LU, int n, const int *perm, const TB *B, T *Y, SolveFlow &f, hipStream_t s)
{
    const unsigned nb = (unsigned)((n + 63) / 64);
    const unsigned base = f.launches * nb, tag = f.launches + 1;
    ++f.launches;
    hipLaunchKernelGGL((k_trsv_flow<T, TB, NR, LOWER>), dim3(nb), dim3(256), 0, s, LU, n, perm, B, Y, f.words,
                       f.ticket, base, tag, f.timeout);
}

// X = A^-1 P B, up to kSolveCols right-hand sides per pass over the factors.  W: n x
// nrhs workspace.  A pass is bound by the chain of blocks, so that 2 or 3 columns take
// little more than one: 3 columns of n = 200 0.15 ms (singly 0.21), 7 of n = 8064 3.2
// (the last three singly 5.4).
template <typename T, int NR>
static void lu_solve_columns(const T *LU, int n, const int *perm, const double *B, T *X, T *W, SolveFlow &f, hipStream_t s)
{
    trsv_flow<T, double, NR, true>(LU, n, perm, B, W, f, s);
    trsv_flow<T, T, NR, false>(LU, n, perm, W, X, f, s);
}
void lu_solve(const double *LU, int n, const int *perm, const double *B, double *X, double *W, int nrhs, SolveFlow &f,
              hipStream_t s)
{
    for (int q = 0; q < nrhs; q += kSolveCols) {
        const size_t o = (size_t)q * n;
        switch (nrhs - q) {
        case 1: lu_solve_columns<double, 1>(LU, n, perm, B + o, X + o, W + o, f, s); break;
        case 2: lu_solve_columns<double, 2>(LU, n, perm, B + o, X + o, W + o, f, s); break;
        case 3: lu_solve_columns<double, 3>(LU, n, perm, B + o, X + o, W + o, f, s); break;
        default: lu_solve_columns<double, kSolveCols>(LU, n, perm, B + o, X + o, W + o, f, s); break;
        }
    }
}

void lu_solve_transposed(const double *LU, int n, const int *perm, const double *b, double *z, double *W,
                         double *V, hipStream_t s)
{
    // U^T w = b: X = W (copy of b, reduced in place), solution in V
    (void)hipMemcpyAsync(W, b, (size_t)n * sizeof(double), hipMemcpyDeviceToDevice, s);
    for (int b0 = 0; b0 < n; b0 += 64) {
        const int bsz = (n - b0 < 64) ? n - b0 : 64;
        const int rows = n - b0 - bsz;
        const unsigned gb = rows > 0 ? (unsigned)((rows + 255) / 256) : 1u;
        hipLaunchKernelGGL(k_trsv_t_step, dim3(gb), dim3(256), 0, s, LU, n, W, V, b0, bsz, 1);
    }
    // L^T v = w: X = V, solution in W
    const int last = ((n - 1) / 64) * 64;
    for (int b0 = last; b0 >= 0; b0 -= 64) {
        const int bsz = (n - b0 < 64) ? n - b0 : 64;
        const unsigned gb = b0 > 0 ? (unsigned)((b0 + 255) / 256) : 1u;
        hipLaunchKernelGGL(k_trsv_t_step, dim3(gb), dim3(256), 0, s, LU, n, V, W, b0, bsz, 0);
    }
    hipLaunchKernelGGL(k_unpermute, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, W, z, perm, n);
}

void lu_factor(double *A, int n, int *ipiv, LUWork &w, hipStream_t s) { lu_factor_launch<double>(A, n, ipiv, w, s); }
void lu_factor(float *A, int n, int *ipiv, LUWork &w, hipStream_t s) { lu_factor_launch<float>(A, n, ipiv, w, s); }
void lu_solve(const float *LU, int n, const int *perm, const double *B, float *X, float *W, SolveFlow &f, hipStream_t s)
{
    lu_solve_columns<float, 1>(LU, n, perm, B, X, W, f, s);
}

}  // namespace nebem
