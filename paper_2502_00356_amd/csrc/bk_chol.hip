// bk_chol.hip - right-looking blocked Cholesky Sigma = L L^T in FP64 on
// v_mfma_f64_16x16x4, with L^-T built in the same sweep.
//
// Every product here has the form X Y^T with both operands column-major, which is how a
// lane's matrix-core operands (one row of X or Y, one k) lie contiguous over 16 lanes:
//  - panel: L_ik = A_ik W_k^T, W_k = L_kk^-1 (128 x 128, from the diagonal kernel);
//  - trailing update: A_im -= L_ik L_mk^T;
//  - inverse factor: Y = L^-T is what the same two operations make of the rows of an
//    identity appended below Sigma; Y is upper triangular, so its blocks (j, m), j < m, take
//    the place of Sigma's upper half and its diagonal blocks are W_k^T;
//  - Sigma^-1 = Y Y^T, tile by tile, only to be multiplied into dSigma and summed.
// n^3 operations in all with the gradient (7.4 ms at the library product's rate for 8,100
// sites), n^3 / 3 for the value. rocSOLVER's potrf, potrs and potri took 76 ms and 41 (its
// 128-column unblocked kernel alone 64 x 171 us); this 18.0 and 9.9.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "bk_chol.hpp"
#include "bk_internal.hpp"

namespace bk {

typedef double chol4_t __attribute__((ext_vector_type(4)));
constexpr int kB = kCholB;
// Block columns a trailing update: 8,100 sites with gradient 19.3 ms with two, 18.0 with
// four, 17.5 with eight; value alone 10.3, 9.9, 10.4.
constexpr int kStep = 4;

// One operand block: rows contiguous, columns (k) ld apart; rows past lim repeat row lim.
struct Operand {
    const double* p;
    int64_t ld;
    int lim;
};

template <int NA, int NB>
struct Acc {
    chol4_t v[NB][NA];
    __device__ __forceinline__ Acc()
    {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int a = 0; a < NA; ++a) v[b][a] = chol4_t{0.0, 0.0, 0.0, 0.0};
    }
};

// acc.v[b][a] += (rows y0 + 16 b of Y) (rows x0 + 16 a of X)^T over cols columns, a wave's
// 16 NA x 16 NB part: lane holds X row 16 a + lane % 16 and Y rows 16 b + lane / 16 + 4 r of
// the product. The loads of D - 1 k steps (4 columns each) are in flight under the products.
// cols: a multiple of 4 D, or with kTail any number up to kB (columns past it count as 0).
template <int D, bool kTail, int NA, int NB>
__device__ __forceinline__ void nt_run(Acc<NA, NB>& acc, const Operand& X, const Operand& Y, int x0, int y0, int cols)
{
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int q0 = kTail ? min(q, cols - 1) : q;
    const double *px[NA], *py[NB];
#pragma unroll
    for (int a = 0; a < NA; ++a) px[a] = X.p + min(x0 + 16 * a + r, X.lim) + (int64_t)q0 * X.ld;
#pragma unroll
    for (int b = 0; b < NB; ++b) py[b] = Y.p + min(y0 + 16 * b + r, Y.lim) + (int64_t)q0 * Y.ld;
    double x[D][NA], y[D][NB];
    const int steps = kTail ? kB / 4 : cols >> 2;
    auto load = [&](int slot, int s) {
        const int k = 4 * s + q, step = kTail ? min(k, cols - 1) - q0 : 4 * s;
        const bool in = !kTail || k < cols;
#pragma unroll
        for (int a = 0; a < NA; ++a) x[slot][a] = in ? px[a][step * X.ld] : 0.0;
#pragma unroll
        for (int b = 0; b < NB; ++b) y[slot][b] = in ? py[b][step * Y.ld] : 0.0;
    };
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, d);
    for (int s = 0; s < steps; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (s + d + D - 1 < steps) load((d + D - 1) % D, s + d + D - 1);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    acc.v[b][a] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[d][b], x[d][a], acc.v[b][a], 0, 0, 0);
        }
    }
}

// Block (i, k) of S as an operand.
__device__ __forceinline__ Operand s_block(const double* S, int64_t n, int i, int k)
{
    return {S + (int64_t)i * kB + (int64_t)k * kB * n, n, (int)min((int64_t)(kB - 1), n - 1 - (int64_t)i * kB)};
}

// S's (or, for an upper block's first update, the identity's zero) minus the product.
template <int NA, int NB>
__device__ __forceinline__ void subtract(double* S, int64_t n, int64_t row0, int64_t col0, bool over, const Acc<NA, NB>& acc)
{
    const int lane = threadIdx.x & 63;
    row0 += lane & 15;
    col0 += lane >> 4;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t col = col0 + 16 * b + 4 * r;
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const int64_t row = row0 + 16 * a;
                if (row < n && col < n) {
                    double* c = S + row + col * n;
                    *c = (over ? 0.0 : *c) - acc.v[b][a][r];
                }
            }
        }
}

// Rows of block row i against block row m, block columns k0 .. k1 - 1 of L (lower i) or Y
// (upper i < k1, whose diagonal block is W^T).
template <int D, int NA, int NB>
__device__ __forceinline__ void panel_products(Acc<NA, NB>& acc, const double* S, int64_t n, const double* wt, int i, int m,
                                               int k0, int k1, int x0, int y0)
{
    if (i < m && i >= k0) {
        nt_run<D, false>(acc, Operand{wt + (int64_t)i * kB * kB, kB, kB - 1}, s_block(S, n, m, i), x0, y0, kB);
        k0 = i + 1;
    }
    if (k0 < k1) nt_run<D, false>(acc, s_block(S, n, i, k0), s_block(S, n, m, k0), x0, y0, kB * (k1 - k0));
}

// Trailing update of the block columns m >= m0 by the block columns k0 .. k1 - 1 (blockIdx.y:
// m - m0; blockIdx.x: lower blocks i = m ..., then with the inverse the upper ones i < k1).
// A tile is 128 x 128, a wave a quarter of it: 16 products of 2,048 operations a k step
// against 8 loads, so the matrix cores bound it (FP64: 78.6 TFLOP/s nominal, the library's
// product 71): 38 TFLOP/s over all steps of 8,100 sites, 8.6 ms of the 18.0; one block
// column a step reached 31.
__global__ __launch_bounds__(256, 2) void k_chol_update(double* S, int64_t n, int nb, const double* __restrict__ wt,
                                                        int k0, int k1, int m0, int inverse)
{
    const int m = m0 + (int)blockIdx.y, lower = nb - m;
    const int x = (int)blockIdx.x;
    const int i = x < lower ? m + x : x - lower;
    if (x >= lower && (!inverse || i >= k1)) return;
    const int wave = threadIdx.x >> 6, x0 = 64 * (wave & 1), y0 = 64 * (wave >> 1);
    Acc<4, 4> acc;
    panel_products<2>(acc, S, n, wt, i, m, k0, k1, x0, y0);
    subtract(S, n, (int64_t)i * kB + x0, (int64_t)m * kB + y0, i < m && i >= k0, acc);
}

// The same for one block column m, 32 rows a workgroup (a wave 32 x 32): four times the
// workgroups, for a column's few tiles (24 us a launch at 8,100 sites; 128-row tiles took
// 29 for the panels, 13 now).
__global__ __launch_bounds__(256) void k_chol_column(double* S, int64_t n, int nb, const double* __restrict__ wt, int k0,
                                                     int k1, int m)
{
    const int lower = nb - m, x = (int)blockIdx.x >> 2;
    const int i = x < lower ? m + x : x - lower;
    const int x0 = 32 * ((int)blockIdx.x & 3), y0 = 32 * (int)(threadIdx.x >> 6);
    Acc<2, 2> acc;
    panel_products<4>(acc, S, n, wt, i, m, k0, k1, x0, y0);
    subtract(S, n, (int64_t)i * kB + x0, (int64_t)m * kB + y0, i < m && i >= k0, acc);
}

// Panel k: S_ik <- S_ik W_k^T for every block i > k (and i < k with the inverse), 32 rows a
// workgroup (which alone reads and writes them), and for i > k the right-hand side's rows:
// zrow_i -= L_ik u_k.
__global__ __launch_bounds__(256) void k_chol_panel(double* S, int64_t n, int nb, const double* __restrict__ w,
                                                    const double* __restrict__ u, double* __restrict__ zrow, int k)
{
    __shared__ double red[4][32];
    const int below = nb - 1 - k, x = (int)blockIdx.x >> 2;
    const int i = x < below ? k + 1 + x : x - below;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int x0 = 32 * ((int)blockIdx.x & 3), y0 = 32 * wave;
    const Operand X = s_block(S, n, i, k), W = {w + (int64_t)k * kB * kB, kB, kB - 1};
    const int kw = (int)min((int64_t)kB, n - (int64_t)k * kB);     // the last block column may be narrow
    Acc<2, 2> acc;
    if (kw == kB) nt_run<4, false>(acc, X, W, x0, y0, kB);
    else nt_run<4, true>(acc, X, W, x0, y0, kw);
    __syncthreads();                 // the other waves have read these rows
    double* C = S + (int64_t)i * kB + (int64_t)k * kB * n;
    const int rows = (int)min((int64_t)kB, n - (int64_t)i * kB);
    const double* uk = u + (int64_t)k * kB;
    double dot[2] = {0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = y0 + 16 * b + 4 * r + q;
            const double uc = uk[col];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int row = x0 + 16 * a + r16;
                if (row < rows && col < kw) C[row + (int64_t)col * n] = acc.v[b][a][r];
                dot[a] = fma(acc.v[b][a][r], uc, dot[a]);
            }
        }
    if (i < k) return;               // uniform over the workgroup
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        dot[a] += __shfl_xor(dot[a], 16, 64);
        dot[a] += __shfl_xor(dot[a], 32, 64);
        if (q == 0) red[wave][16 * a + r16] = dot[a];
    }
    __syncthreads();
    const int t = (int)threadIdx.x;
    if (t < 32 && x0 + t < rows) zrow[(int64_t)i * kB + x0 + t] -= (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
}

__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// 1 / sqrt(d) from the hardware's estimate and two Newton steps.
__device__ __forceinline__ double rsqrt_newton(double d)
{
    double y = __builtin_amdgcn_rsq(d);
    y = fma(y * 0.5, fma(-d * y, y, 1.0), y);
    return fma(y * 0.5, fma(-d * y, y, 1.0), y);
}

// Diagonal block k: its factor, the factor's inverse W_k (and transpose), u_k = W_k zrow_k,
// and the block's share of log det L and |u|^2. One workgroup, the block in LDS, by
// 16 x 16 sub-blocks: one wave factors the sub-block in registers, a lane a row solves for
// the rows below, the matrix cores update the rest; then the sub-blocks' inverses, a lane a
// column, and the whole inverse, a block column a wave. Rows past n are the identity's. A
// serial chain, bound by latency: 136 us with each sub-block inverted before its panel, the
// logarithms and divisions on the chain and the block loaded a value at a time; 53 now.
__global__ __launch_bounds__(256) void k_chol_diag(const double* __restrict__ S, int64_t n, int nb, int k,
                                                   double* __restrict__ w, double* __restrict__ wt,
                                                   const double* __restrict__ zrow, double* __restrict__ u,
                                                   double* __restrict__ part, int* __restrict__ info)
{
    constexpr int LD = kB + 1, NS = kB / 16;
    __shared__ double A[kB * LD];
    __shared__ double G[NS][16 * 17];              // inverses of the diagonal sub-blocks
    __shared__ double zs[kB], ip[kB], red[2][4];   // ip: 1 / L_ii
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, r16 = lane & 15, q = lane >> 4;
    const int64_t g0 = (int64_t)k * kB;
    const int live = (int)min((int64_t)kB, n - g0);
    {
        const int r = t & (kB - 1), h = t >> 7, rr = min(r, live - 1);
        const double* src = S + g0 + rr + g0 * n;
        for (int c0 = h; c0 < kB; c0 += 32) {      // 16 loads in flight; columns past the row's own stay in the block
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = src[(int64_t)min(c0 + 2 * e, rr) * n];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = c0 + 2 * e;
                A[r * LD + c] = r < live && c <= r ? v[e] : (r == c ? 1.0 : 0.0);
            }
        }
    }
    if (t < kB) zs[t] = t < live ? zrow[g0 + t] : 0.0;
    __syncthreads();
    for (int s = 0; s < NS; ++s) {
        const int o = 16 * s;
        if (wave == 0) {
            double v[16], own = 0.0;
            bool bad = false;
#pragma unroll
            for (int c = 0; c < 16; ++c) v[c] = A[(o + r16) * LD + o + c];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const double d = lane_value(v[c], c);
                bad |= !(d > 0.0);
                const double y = rsqrt_newton(d);
                own = r16 == c ? y : own;
                v[c] *= y;                          // row c: d / sqrt(d)
#pragma unroll
                for (int c2 = c + 1; c2 < 16; ++c2) v[c2] = fma(-v[c], lane_value(v[c], c2), v[c2]);
            }
            if (lane < 16) {
                ip[o + r16] = own;
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (c <= r16) A[(o + r16) * LD + o + c] = v[c];
            }
            if (bad && lane == 0) *info = 1;
        }
        __syncthreads();
        // rows below: x L_ss^T = a by columns, a lane a row
        const int row = o + 16 + t;
        if (row < kB) {
            double x[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) x[c] = A[row * LD + o + c];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                x[c] *= ip[o + c];
#pragma unroll
                for (int c2 = c + 1; c2 < 16; ++c2) x[c2] = fma(-x[c], A[(o + c2) * LD + o + c], x[c2]);
            }
#pragma unroll
            for (int c = 0; c < 16; ++c) A[row * LD + o + c] = x[c];
        }
        __syncthreads();
        // the rest: A_IJ -= A_Is A_Js^T
        const int rem = NS - 1 - s, tiles = rem * (rem + 1) / 2;
        for (int f = wave; f < tiles; f += 4) {
            int I = 0, f0 = f;
            while (f0 > I) f0 -= ++I;
            const int ri = 16 * (s + 1 + I), rj = 16 * (s + 1 + f0);
            chol4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(ri + r16) * LD + o + 4 * c + q],
                                                           A[(rj + r16) * LD + o + 4 * c + q], acc, 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) A[(ri + q + 4 * c) * LD + rj + r16] -= acc[c];
        }
        __syncthreads();
    }
    if (t < kB) {                                   // column r16 of sub-block t / 16's inverse
        const int s = t >> 4, o = 16 * s;
        double x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = r16 == i ? 1.0 : 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            x[i] *= ip[o + i];
#pragma unroll
            for (int m = i + 1; m < 16; ++m) x[m] = fma(-A[(o + m) * LD + o + i], x[i], x[m]);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) G[s][i * 17 + r16] = x[i];
    }
    __syncthreads();
    // W_IJ = -G_I sum_{J <= K < I} L_IK W_KJ, kept transposed in the upper blocks (J, I)
    for (int pass = 0; pass < 2; ++pass) {
        const int J = pass == 0 ? wave : NS - 1 - wave;
        for (int I = J + 1; I < NS; ++I) {
            chol4_t acc = {0.0, 0.0, 0.0, 0.0};
            for (int K = J; K < I; ++K) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int m = 4 * c + q;
                    const double b = K == J ? G[J][m * 17 + r16] : A[(16 * J + r16) * LD + 16 * K + m];
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(16 * I + r16) * LD + 16 * K + m], b, acc, 0, 0, 0);
                }
            }
            chol4_t wij = {0.0, 0.0, 0.0, 0.0};
            // a product's registers hold rows lane / 16 + 4 c: the next product's operand
#pragma unroll
            for (int c = 0; c < 4; ++c)
                wij = __builtin_amdgcn_mfma_f64_16x16x4f64(G[I][r16 * 17 + 4 * c + q], acc[c], wij, 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) A[(16 * J + r16) * LD + 16 * I + q + 4 * c] = -wij[c];
        }
    }
    __syncthreads();
    // the diagonal blocks' lower parts, transposed into the upper half with the rest
    for (int e = t; e < NS * 256; e += 256) {
        const int s = e >> 8, i = (e >> 4) & 15, j = e & 15;
        if (i >= j) A[(16 * s + j) * LD + 16 * s + i] = G[s][i * 17 + j];
    }
    __syncthreads();
    double* wk = w + (int64_t)k * kB * kB;
    double* wtk = wt + (int64_t)k * kB * kB;
    {
        const int r = t & (kB - 1), h = t >> 7;
#pragma unroll 8
        for (int c = h; c < kB; c += 2) {
            wk[r + c * kB] = r >= c ? A[c * LD + r] : 0.0;
            wtk[r + c * kB] = c >= r ? A[r * LD + c] : 0.0;
        }
    }
    double sum = 0.0;
    const int ru = t >> 1, h = t & 1;
#pragma unroll 8
    for (int c = h; c <= ru; c += 2) sum = fma(A[c * LD + ru], zs[c], sum);
    sum += __shfl_xor(sum, 1, 64);
    if (h == 0) u[g0 + ru] = sum;
    double sq = h == 0 ? sum * sum : 0.0, logs = h == 0 ? -log(ip[ru]) : 0.0;
    for (int d = 32; d > 0; d >>= 1) {
        sq += __shfl_xor(sq, d, 64);
        logs += __shfl_xor(logs, d, 64);
    }
    if (lane == 0) {
        red[0][wave] = logs;
        red[1][wave] = sq;
    }
    __syncthreads();
    if (t == 0) {
        part[k] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        part[nb + k] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
}

// ypart[k][rows of block c] = Y_ck u_k (blockIdx.x: c, blockIdx.y: k >= c).
__global__ __launch_bounds__(256) void k_chol_yu(const double* __restrict__ S, int64_t n, const double* __restrict__ wt,
                                                 const double* __restrict__ u, double* __restrict__ ypart)
{
    __shared__ double red[kB];
    const int c = (int)blockIdx.x, k = (int)blockIdx.y;
    if (k < c) return;
    const int r = threadIdx.x & (kB - 1), h = threadIdx.x >> 7;
    const Operand Y = k == c ? Operand{wt + (int64_t)k * kB * kB, kB, kB - 1} : s_block(S, n, c, k);
    const int kw = (int)min((int64_t)kB, n - (int64_t)k * kB);
    const double* uk = u + (int64_t)k * kB;
    double sum = 0.0;
    for (int m = 64 * h; m < min(64 * h + 64, kw); ++m) sum = fma(Y.p[min(r, Y.lim) + (int64_t)m * Y.ld], uk[m], sum);
    if (h == 1) red[r] = sum;
    __syncthreads();
    const int64_t row = (int64_t)c * kB + r;
    if (h == 0 && row < n) ypart[(int64_t)k * n + row] = sum + red[r];
}

__global__ __launch_bounds__(256) void k_chol_ysum(const double* __restrict__ ypart, int64_t n, int nb,
                                                   double* __restrict__ a)
{
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= n) return;
    double s = 0.0;
    for (int k = (int)(row / kB); k < nb; ++k) s += ypart[(int64_t)k * n + row];
    a[row] = s;
}

// Tile (c, d), c >= d, of Sigma^-1 = Y Y^T, multiplied into dB and dN at once:
//   part[4 x ..] = sum w a_i a_j dB_ij, sum w Sinv_ij dB_ij, and the same of dN,
// over the tile's part of the lower triangle (w = 2 off the diagonal). Tiles with the
// longest sums (small c) come first. 177 GFLOP in 3.3 ms at 8,100 sites (54 TFLOP/s).
__global__ __launch_bounds__(256, 2) void k_chol_traces(const double* __restrict__ S, int64_t n, int nb,
                                                        const double* __restrict__ wt, const double* __restrict__ av,
                                                        const double* __restrict__ dB, const double* __restrict__ dN,
                                                        double* __restrict__ part)
{
    __shared__ double red[4][4];
    const int f = (int)blockIdx.x;
    int c = (int)((__builtin_amdgcn_sqrtf(8.0f * (float)f + 1.0f) - 1.0f) * 0.5f);
    while (c * (c + 1) / 2 > f) --c;
    while ((c + 1) * (c + 2) / 2 <= f) ++c;
    const int d = f - c * (c + 1) / 2;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int x0 = 64 * (wave & 1), y0 = 64 * (wave >> 1);
    Acc<4, 4> acc;
    const Operand Wc = {wt + (int64_t)c * kB * kB, kB, kB - 1};
    const int full = (int)(n / kB);                   // block columns of full width
    if (c < full) {
        nt_run<2, false>(acc, Wc, c == d ? Wc : s_block(S, n, d, c), x0, y0, kB);
        if (c + 1 < full) nt_run<2, false>(acc, s_block(S, n, c, c + 1), s_block(S, n, d, c + 1), x0, y0, kB * (full - c - 1));
    }
    if (full < nb)
        nt_run<2, true>(acc, c == full ? Wc : s_block(S, n, c, full), d == full ? Wc : s_block(S, n, d, full), x0, y0,
                        (int)(n - (int64_t)full * kB));
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t row0 = (int64_t)c * kB + x0 + (lane & 15), col0 = (int64_t)d * kB + y0 + (lane >> 4);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t j = col0 + 16 * b + 4 * r;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int64_t i = row0 + 16 * a;
                if (i < n && j <= i) {
                    const double wgt = i == j ? 1.0 : 2.0;
                    const double wa = wgt * av[i] * av[j], ws = wgt * acc.v[b][a][r];
                    const double eb = dB[i + j * n], en = dN[i + j * n];
                    s[0] = fma(wa, eb, s[0]);
                    s[1] = fma(ws, eb, s[1]);
                    s[2] = fma(wa, en, s[2]);
                    s[3] = fma(ws, en, s[3]);
                }
            }
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, 64);
        if (lane == 0) red[wave][q] = s[q];
    }
    __syncthreads();
    if (threadIdx.x < 4)
        part[4 * (int64_t)f + threadIdx.x] =
            red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// res[k] = sum_p part[p * stride + k] for k < stride, one workgroup, fixed order.
__global__ __launch_bounds__(256) void k_chol_sum(const double* __restrict__ part, int64_t np, int stride,
                                                  double* __restrict__ res)
{
    __shared__ double red[4];
    for (int k = 0; k < stride; ++k) {
        double s = 0.0;
        for (int64_t p = threadIdx.x; p < np; p += 256) s += part[p * stride + k];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) res[k] = red[0] + red[1] + red[2] + red[3];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_chol_begin(const double* __restrict__ z, double* __restrict__ zrow, int64_t n,
                                                    int* __restrict__ info)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) zrow[i] = z[i];
    if (i == 0) *info = 0;
}

int chol_solve(double* S, const double* dB, const double* dN, const double* z, int64_t n, const CholWork& wk,
               hipStream_t stream)
{
    const int nb = (int)chol_blocks(n), inverse = dB ? 1 : 0;
    const double *w = wk.w, *wt = wk.wt, *u = wk.u, *zrow = wk.zrow, *Sc = S;
    const dim3 wg(256);
    int st = launch(k_chol_begin, dim3((unsigned)((n + 255) / 256)), wg, stream, z, wk.zrow, n, wk.info);
    auto diag = [&](int k) {
        if (st == BK_OK)
            st = launch(k_chol_diag, dim3(1), wg, stream, Sc, n, nb, k, wk.w, wk.wt, zrow, wk.u, wk.part, wk.info);
    };
    auto panel = [&](int k) {
        const int blocks = nb - 1 - k + (inverse ? k : 0);
        if (st == BK_OK && blocks > 0) st = launch(k_chol_panel, dim3(4 * blocks), wg, stream, S, n, nb, w, u, wk.zrow, k);
    };
    auto column = [&](int k0, int m) {
        if (st == BK_OK && k0 < m)
            st = launch(k_chol_column, dim3(4 * (nb - m + (inverse ? m : 0))), wg, stream, S, n, nb, wt, k0, m, m);
    };
    // kStep panels a trailing update (its blocks of S are read and written that much less
    // often), each block column of the step brought up to date just before its turn
    for (int k = 0; k < nb; k += kStep) {
        const int ke = k + kStep < nb ? k + kStep : nb;
        for (int j = k; j < ke; ++j) {
            column(k, j);
            diag(j);
            panel(j);
        }
        if (st == BK_OK && ke < nb)
            st = launch(k_chol_update, dim3(nb - ke + (inverse ? ke : 0), nb - ke), wg, stream, S, n, nb, wt, k, ke, ke,
                        inverse);
    }
    const double* part = wk.part;
    if (st == BK_OK) st = launch(k_chol_sum, dim3(1), wg, stream, part, (int64_t)nb, 1, wk.res + 0);
    if (st == BK_OK) st = launch(k_chol_sum, dim3(1), wg, stream, part + nb, (int64_t)nb, 1, wk.res + 1);
    if (!inverse || st != BK_OK) return st;
    st = launch(k_chol_yu, dim3(nb, nb), wg, stream, Sc, n, wt, u, wk.ypart);
    if (st == BK_OK)
        st = launch(k_chol_ysum, dim3((unsigned)((n + 255) / 256)), wg, stream, (const double*)wk.ypart, n, nb, wk.a);
    const int64_t tiles = (int64_t)nb * (nb + 1) / 2;
    if (st == BK_OK)
        st = launch(k_chol_traces, dim3((unsigned)tiles), wg, stream, Sc, n, nb, wt, (const double*)wk.a, dB, dN, wk.part);
    if (st == BK_OK) st = launch(k_chol_sum, dim3(1), wg, stream, part, tiles, 4, wk.res + 2);
    return st;
}

}  // namespace bk
