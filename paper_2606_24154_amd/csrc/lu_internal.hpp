// lu_internal.hpp -- dense LU factorisation / solve launchers.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "panel_rule.hpp"

namespace nebem {

constexpr int kOuterNB = 256;  // LU outer block width (multiple of kNB)

// Device scratch of one factorisation: per-workgroup pivot candidates
// (ceil(n/256) entries), a completion counter (must start at 0; every panel
// launch leaves it at 0) and `info` (must start at n; receives the first
// column with a zero pivot).
// The single-launch panel factorisation (taken when words is not null and
// the panel's workgroups fit on the device at once) also needs panel_words(n,
// sizeof(entry) / 4) words and a flag `timeout`, all starting at 0; `timeout` is
// set if a wait gave up.
struct LUWork {
    void *pval;
    int *pidx;
    int *counter;
    int *info;
    uint64_t *words = nullptr;
    int *timeout = nullptr;
};
void clear_words(uint64_t *w, int64_t len, hipStream_t s);

void lu_factor(double *A, int n, int *ipiv, LUWork &w, hipStream_t s);
void lu_factor(float *A, int n, int *ipiv, LUWork &w, hipStream_t s);
// Workspace of the triangular solves of one factorisation, on one stream:
// solve_flow_bytes(n) bytes at a 256-byte boundary, cleared by
// solve_flow_init.  *timeout (device) is set if a wait gave up: the results are
// then worthless, and the caller, which synchronises anyway, reports an error.
constexpr int kSolveCols = 4;  // right-hand sides solved together
struct SolveFlow {
    uint64_t *words;
    unsigned *ticket;
    int *timeout;
    unsigned launches;  // tags in use so far
};
size_t solve_flow_bytes(int n);
void solve_flow_init(SolveFlow &f, void *mem, int n, hipStream_t s);
// X = A^-1 B with the row permutation perm (X[i] = (P B)[i] = B[perm[i]]);
// W is an n x nrhs workspace of the solve's type.  X, W and B must be distinct.
void lu_solve(const double *LU, int n, const int *perm, const double *B, double *X, double *W, int nrhs,
              SolveFlow &f, hipStream_t s);
// the same with FP32 factors, one column
void lu_solve(const float *LU, int n, const int *perm, const double *B, float *X, float *W, SolveFlow &f,
              hipStream_t s);
// z = A^-T b with the FP64 factors of P A = L U (perm as in lu_solve); W, V:
// n-entry workspaces.  z must not alias b, W or V.
void lu_solve_transposed(const double *LU, int n, const int *perm, const double *b, double *z, double *W,
                         double *V, hipStream_t s);

}  // namespace nebem
