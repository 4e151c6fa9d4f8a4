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

// Tiles of the trace sums: 128 x 128, or quarters of those below kTraceBlocks block rows,
// where whole ones are fewer than the workgroups the chip holds (likelihood with gradient:
// 1,024 sites 0.76 -> 0.62 ms, 4,096 sites (32 block rows) 3.59 -> 3.16, 5,625 (44) 6.02 ->
// 6.46).
constexpr int64_t kTraceBlocks = 38;
inline int64_t chol_trace_tiles(int64_t n)
{
    const int64_t nb = chol_blocks(n), t = nb >= kTraceBlocks ? nb : 2 * nb;
    return t * (t + 1) / 2;
}

// Factorises the lower triangle of S (n x n, column-major, leading dimension n; its scale
// within 2^-200 to 2^200) and reduces zscale z: res[0] = log det L, res[1] = zscale^2 z^T
// Sigma^-1 z. dB, dN not NULL: also L^-T in S's strictly upper blocks, a = zscale Sigma^-1 z, and
//   res[2] = a^T dB a, res[3] = tr(Sigma^-1 dB), res[4], res[5] the same of dN
// from the lower triangles of dB and dN. bk_status.
int chol_solve(double* S, const double* dB, const double* dN, const double* z, double zscale, int64_t n,
               const CholWork& wk, hipStream_t stream);

}  // namespace bk
