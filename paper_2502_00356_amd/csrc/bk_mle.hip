// bk_mle.hip - Gaussian log-likelihood of observations under the Matern
// covariance, and its gradient in (sigma2, beta, nu): the consumer of the
// generated matrix (Sec. III-A; the paper generates Matern matrices for
// likelihood maximisation).
//
//   l = -1/2 z^T Sigma^-1 z - 1/2 log det Sigma - n/2 log(2 pi)
//   dl/dtheta = 1/2 a^T dSigma a - 1/2 tr(Sigma^-1 dSigma),  a = Sigma^-1 z
//
// Sigma (and for the gradient dSigma/dbeta, dSigma/dnu) comes from this library's
// Matern kernels as one full column-major tile; the factorisation, the inverse factor and
// the traces are bk_chol.hip's (sums in a fixed order).
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "../../include/besselk.h"
#include "bk_chol.hpp"
#include "bk_internal.hpp"

namespace bk {

constexpr int64_t kMleMaxN = 46340;

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct MleLayout {
    size_t S, dB, dN, w, wt, zrow, u, a, ypart, part, res, info, mws, total;
};

struct MleResult {
    double sums[6];
    int info;
};

static MleLayout mle_layout(int64_t n, int with_grad)
{
    MleLayout L;
    const size_t mat = align256(sizeof(double) * (size_t)n * (size_t)n);
    const size_t nb = (size_t)chol_blocks(n), blocks = align256(sizeof(double) * nb * kCholB * kCholB);
    const size_t tiles = (size_t)chol_trace_tiles(n);
    size_t o = 0;
    L.S = o; o += mat;
    L.dB = o; o += with_grad ? mat : 0;
    L.dN = o; o += with_grad ? mat : 0;
    L.w = o; o += blocks;
    L.wt = o; o += blocks;
    L.zrow = o; o += align256(sizeof(double) * (size_t)n);
    L.u = o; o += align256(sizeof(double) * nb * kCholB);
    L.a = o; o += with_grad ? align256(sizeof(double) * (size_t)n) : 0;
    L.ypart = o; o += with_grad ? align256(sizeof(double) * nb * (size_t)n) : 0;
    L.part = o; o += align256(sizeof(double) * (with_grad ? 4 * tiles + 2 * nb : 2 * nb));
    L.res = o;                                       // six sums and the info word, read back together
    L.info = L.res + offsetof(MleResult, info); o += 256;
    L.mws = o; o += matern_learned_workspace_bytes(n, (int32_t)n, 0);   // for a learned-form Sigma
    L.total = o;
    return L;
}

}  // namespace bk

using namespace bk;

extern "C" size_t bk_matern_loglik_workspace_bytes(int64_t n, int32_t with_grad)
{
    if (n <= 0 || n > kMleMaxN) return 0;
    return mle_layout(n, with_grad ? 1 : 0).total;
}

extern "C" int bk_matern_loglik(const bk_locs* locs, const double* z, const bk_params* prm, int32_t with_grad,
                                double* result, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (!locs || !prm || !z || !result || !workspace) return BK_EINVAL;
    const int64_t n = locs->n;
    if (n <= 0 || n > kMleMaxN || !locs->x || !locs->y) return BK_EINVAL;
    if (with_grad && prm->mode != BK_PLAIN_F64) return BK_EINVAL;
    if (!(prm->beta > 0.0) || !(prm->nu > 0.0) || !(prm->sigma2 > 0.0)) return BK_EINVAL;
    const MleLayout L = mle_layout(n, with_grad ? 1 : 0);
    if (workspace_bytes < L.total) return BK_ENOMEM;
    char* ws = (char*)workspace;
    auto at = [&](size_t o) { return (double*)(ws + o); };
    double *S = at(L.S), *dB = with_grad ? at(L.dB) : nullptr, *dN = with_grad ? at(L.dN) : nullptr;
    const CholWork wk = {at(L.w), at(L.wt), at(L.zrow), at(L.u), at(L.ypart), at(L.a), at(L.part), at(L.res),
                         (int*)(ws + L.info)};

    // Sigma (and its derivatives) as one full column-major n x n tile, FP64
    bk_params p = *prm;
    p.out_dtype = BK_OUT_F64;
    p.workspace = ws + L.mws;
    p.workspace_bytes = L.total - L.mws;
    // Far from 1, sigma2 is taken as 4^k sigma2': Sigma / 4^k and z / 2^k have the same quadratic
    // forms and traces, and log det Sigma / 4^k is log det Sigma less 2 n k log 2
    int k = 0;
    if (!(prm->sigma2 >= 0x1p-200 && prm->sigma2 <= 0x1p200) && prm->sigma2 <= DBL_MAX) {
        k = ilogb(prm->sigma2) / 2;
        p.sigma2 = ldexp(prm->sigma2, -2 * k);
    }
    int st = with_grad ? bk_matern_grad_tiles(locs, &p, (int32_t)n, 0, S, dB, dN, stream)
                       : bk_matern_tiles(locs, &p, (int32_t)n, 0, S, stream);
    if (st != BK_OK) return st;

    st = chol_solve(S, dB, dN, z, ldexp(1.0, -k), n, wk, stream);
    if (st != BK_OK) return st;
    MleResult h = {};
    if (hipMemcpyAsync(&h, wk.res, sizeof(h), hipMemcpyDeviceToHost, stream) != hipSuccess) return BK_EHIP;
    if (hipStreamSynchronize(stream) != hipSuccess) return BK_EHIP;
    if (h.info != 0) return BK_ENOTPD;
    const double *hres = h.sums, logdet = 2.0 * hres[0] + (double)n * (2.0 * k * kLn2), quad = hres[1];
    result[0] = -0.5 * quad - 0.5 * logdet - 0.5 * (double)n * 1.8378770664093454836;   // log(2 pi)
    if (with_grad) {
        result[1] = 0.5 * (quad - (double)n) / prm->sigma2;
        result[2] = 0.5 * hres[2] - 0.5 * hres[3];
        result[3] = 0.5 * hres[4] - 0.5 * hres[5];
    }
    return BK_OK;
}
