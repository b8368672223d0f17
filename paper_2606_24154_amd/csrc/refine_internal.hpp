// refine_internal.hpp -- launchers for the mixed-precision solve helpers.
#pragma once
#include <hip/hip_runtime.h>

namespace nebem {

// Column chunks of the two passes over the matrix (row maxima, residual): enough
// of them that row blocks x chunks give the device some 2048 workgroups, at most
// kMaxChunk columns each.  At n = 8064 four chunks of 2048 columns were 128
// workgroups: 0.81 ms for 0.52 GB.
constexpr int kMaxChunk = 2048;
inline int matrix_chunks(int n)
{
    const int rows = (n + 255) / 256, least = (n + kMaxChunk - 1) / kMaxChunk;
    const int want = (2048 + rows - 1) / rows, most = (n + 63) / 64;
    const int c = want > least ? want : least;
    return c < most ? c : (most > least ? most : least);
}

// s[i] = 1 / max_j |A_ij| (1 for an all-zero row); part: n * matrix_chunks(n) doubles
void row_scale(const double *A, int n, double *part, double *s, hipStream_t st);
// A32 = float(diag(s) A), column-major
void convert_scaled(const double *A, const double *s, int n, float *A32, hipStream_t st);
// rs = s .* (b - A x) in FP64; sq[k] = per-workgroup sums of (b - A x)^2 (ceil(n/256) entries);
// part: n * matrix_chunks(n) doubles
void residual(const double *A, int n, const double *x, const double *b, const double *s, double *part, double *rs,
              double *sq, hipStream_t st);
void sumsq(const double *v, int n, double *sq, hipStream_t st);
void add_f32(double *x, const float *d, int n, hipStream_t st);
void add_f64(double *x, const double *d, int n, hipStream_t st);
// cs[j] = sum_i |A_ij|, n entries
void column_abs_sums(const double *A, int n, double *cs, hipStream_t st);
void scale_vec(const double *s, const double *b, int n, double *out, hipStream_t st);
void fill(double *x, int n, double v, hipStream_t st);

}  // namespace nebem
