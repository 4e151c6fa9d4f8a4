// bk_chol.hpp - dense FP64 Cholesky factorisation, the inverse factor and the traces
// of the likelihood's gradient, on the matrix cores (bk_chol.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bk {

constexpr int kCholB = 128;                      // block size

struct CholWork {
    double* w;        // [nb][128 x 128] inverses of the diagonal blocks' factors
    double* wt;       // [nb][128 x 128] their transposes
    double* zrow;     // [n] right-hand side, reduced block by block
    double* u;        // [nb * 128] L^-1 z
    double* ypart;    // [nb][n] partial sums of a (with the inverse factor only)
    double* a;        // [n] Sigma^-1 z (with the inverse factor only)
    double* part;     // partial sums: nb log-determinants, nb quadratic forms, 4 per trace tile
    double* res;      // [6] log det L, |u|^2, then the four gradient sums
    int* info;        // nonzero: a pivot was not positive
};

inline int64_t chol_blocks(int64_t n) { return (n + kCholB - 1) / kCholB; }

// Factorises the lower triangle of S (n x n, column-major, leading dimension n) and
// reduces z: res[0] = log det L, res[1] = z^T Sigma^-1 z. dB, dN not NULL: also
// L^-T in S's strictly upper blocks, a = Sigma^-1 z, and
//   res[2] = a^T dB a, res[3] = tr(Sigma^-1 dB), res[4], res[5] the same of dN
// from the lower triangles of dB and dN. bk_status.
int chol_solve(double* S, const double* dB, const double* dN, const double* z, int64_t n, const CholWork& wk,
               hipStream_t stream);

}  // namespace bk
