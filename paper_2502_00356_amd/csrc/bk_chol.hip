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
// 128-column unblocked kernel alone 64 x 171 us); this 14.4 and 7.0.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "bk_chol.hpp"
#include "bk_internal.hpp"

namespace bk {

typedef double chol4_t __attribute__((ext_vector_type(4)));
constexpr int kB = kCholB;
// Block columns a trailing update (the sums run in the same order for any): 8,100 sites with
// gradient 15.25 ms with four, 15.2 with six and with eight; value alone 7.7, 7.7, 8.2. Where
// the launches' latencies are the time, fewer: one (no column launches) up to 16 block rows
// (1,024 sites, value, us: 417 with one, 422, 433, 439 with four), two up to 32 (2,025 sites
// 858, 857, 888, 881; 4,096 sites 1,999, 1,939, 1,944, 1,987); no trailing update at all up
// to four (256 sites 124 against 127 with one).
static int update_step(int nb) { return nb <= 4 ? 4 : (nb <= 16 ? 1 : (nb <= 32 ? 2 : 4)); }
// Where a launch has few blocks its tiles are cut finer, so that a wave's chain of products
// is shorter and more SIMDs have one (likelihood with gradient / value, ms):
//  - panels and columns by 16 rows in place of 32 up to this many blocks: 1,024 sites (8
//    blocks) 0.61 / 0.48 -> 0.57 / 0.45, 4,096 (32) 3.15 / 2.16 -> 2.96 / 1.99, 5,625 (44)
//    5.93 -> 6.04 with gradient;
constexpr int kFewBlocks = 40;
//  - the update by quarters of a block below this many: 1,024 sites 0.54 -> 0.49 (value),
//    4,096 sites 2.39 -> 2.17 against 2.25 with 256 and 2.19 with 512;
constexpr int kFewTiles = 1024;
//  - the traces by quarters (chol_trace_tiles): 1,024 sites 158 us -> 60.

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
// kNeg: 1 negates Y.
template <int D, bool kTail, int NA, int NB, int kNeg = 0>
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
                    acc.v[b][a] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[d][b], x[d][a], acc.v[b][a], 0, 0, kNeg);
        }
    }
}

// Block (i, k) of S as an operand.
__device__ __forceinline__ Operand s_block(const double* S, int64_t n, int i, int k)
{
    return {S + (int64_t)i * kB + (int64_t)k * kB * n, n, (int)min((int64_t)(kB - 1), n - 1 - (int64_t)i * kB)};
}

// The accumulators' elements of S, from row row0 and column col0: read before the products
// (zero for an upper block's first update, whose identity S does not hold) ...
template <int NA, int NB>
__device__ __forceinline__ void read_part(Acc<NA, NB>& acc, const double* S, int64_t n, int64_t row0, int64_t col0, bool over)
{
    if (over) return;
    const int lane = threadIdx.x & 63;
    row0 += lane & 15;
    col0 += lane >> 4;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int a = 0; a < NA; ++a)
                acc.v[b][a][r] = S[min(row0 + 16 * a, n - 1) + min(col0 + 16 * b + 4 * r, n - 1) * n];
}

// ... and written after them.
template <int NA, int NB>
__device__ __forceinline__ void write_part(double* S, int64_t n, int64_t row0, int64_t col0, const Acc<NA, NB>& acc)
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
            for (int a = 0; a < NA; ++a)
                if (row0 + 16 * a < n && col < n) S[row0 + 16 * a + col * n] = acc.v[b][a][r];
        }
}

// Minus rows of block row i times block row m's, block columns k0 .. k1 - 1 of L (lower i) or Y
// (upper i < k1, whose diagonal block is W^T).
template <int D, int NA, int NB>
__device__ __forceinline__ void panel_products(Acc<NA, NB>& acc, const double* S, int64_t n, const double* wt, int i, int m,
                                               int k0, int k1, int x0, int y0)
{
    if (i < m && i >= k0) {
        nt_run<D, false, NA, NB, 1>(acc, Operand{wt + (int64_t)i * kB * kB, kB, kB - 1}, s_block(S, n, m, i), x0, y0, kB);
        k0 = i + 1;
    }
    if (k0 < k1) nt_run<D, false, NA, NB, 1>(acc, s_block(S, n, i, k0), s_block(S, n, m, k0), x0, y0, kB * (k1 - k0));
}

// Trailing update of the block columns m >= m0 by the block columns k0 .. k1 - 1 (blockIdx.y:
// m - m0; blockIdx.x: lower blocks i = m ..., then with the inverse the upper ones i < k1).
// A tile is 128 x 128 (NA = 4; with NA = 2 a quarter of it, four workgroups a block, where
// there are few), a wave a quarter of that: NA = 4: 16 products of 2,048 operations a k step
// against 8 loads, so the matrix cores bound it (FP64: 78.6 TFLOP/s nominal, the library's
// product 71): 8.6 ms over all steps of 8,100 sites (38 TFLOP/s) with S's part read after the
// products and one k step of operands in flight; read before them 7.4, three steps in
// flight (64 more registers) 6.9 (48 TFLOP/s); seven spill.
template <int NA>
__global__ __launch_bounds__(256, 2) void k_chol_update(double* S, int64_t n, int nb, const double* __restrict__ wt,
                                                        int k0, int k1, int m0, int inverse)
{
    const int m = m0 + (int)blockIdx.y, lower = nb - m;
    const int x = NA == 4 ? (int)blockIdx.x : (int)blockIdx.x >> 2, quarter = NA == 4 ? 0 : (int)blockIdx.x & 3;
    const int i = x < lower ? m + x : x - lower;
    if (x >= lower && (!inverse || i >= k1)) return;
    const int wave = threadIdx.x >> 6;
    const int x0 = 64 * (quarter & 1) + 16 * NA * (wave & 1), y0 = 64 * (quarter >> 1) + 16 * NA * (wave >> 1);
    Acc<NA, NA> acc;
    read_part(acc, S, n, (int64_t)i * kB + x0, (int64_t)m * kB + y0, i < m && i >= k0);
    panel_products<4>(acc, S, n, wt, i, m, k0, k1, x0, y0);
    write_part(S, n, (int64_t)i * kB + x0, (int64_t)m * kB + y0, acc);
}

// The same for one block column m, 16 NA rows a workgroup (a wave 16 NA x 32), for a column's
// few tiles (8,100 sites: 24 us a launch as the update was, 17 with S's part read first and
// seven k steps in flight).
template <int NA>
__global__ __launch_bounds__(256) void k_chol_column(double* S, int64_t n, int nb, const double* __restrict__ wt, int k0,
                                                     int k1, int m)
{
    constexpr int kPer = 8 / NA;
    const int lower = nb - m, x = (int)blockIdx.x / kPer;
    const int i = x < lower ? m + x : x - lower;
    const int x0 = 16 * NA * ((int)blockIdx.x % kPer), y0 = 32 * (int)(threadIdx.x >> 6);
    Acc<NA, 2> acc;
    read_part(acc, S, n, (int64_t)i * kB + x0, (int64_t)m * kB + y0, i < m && i >= k0);
    panel_products<8>(acc, S, n, wt, i, m, k0, k1, x0, y0);
    write_part(S, n, (int64_t)i * kB + x0, (int64_t)m * kB + y0, acc);
}

// Panel k: S_ik <- S_ik W_k^T for every block i > k (and i < k with the inverse), 16 NA rows a
// workgroup (which alone reads and writes them), and for i > k the right-hand side's rows:
// zrow_i -= L_ik u_k.
template <int NA>
__global__ __launch_bounds__(256) void k_chol_panel(double* S, int64_t n, int nb, const double* __restrict__ w,
                                                    const double* __restrict__ u, double* __restrict__ zrow, int k)
{
    constexpr int kPer = 8 / NA;
    __shared__ double red[4][16 * NA];
    const int below = nb - 1 - k, x = (int)blockIdx.x / kPer;
    const int i = x < below ? k + 1 + x : x - below;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int x0 = 16 * NA * ((int)blockIdx.x % kPer), y0 = 32 * wave;
    const Operand X = s_block(S, n, i, k), W = {w + (int64_t)k * kB * kB, kB, kB - 1};
    const int kw = (int)min((int64_t)kB, n - (int64_t)k * kB);     // the last block column may be narrow
    Acc<NA, 2> acc;
    if (kw == kB) nt_run<4, false>(acc, X, W, x0, y0, kB);
    else nt_run<4, true>(acc, X, W, x0, y0, kw);
    __syncthreads();                 // the other waves have read these rows
    double* C = S + (int64_t)i * kB + (int64_t)k * kB * n;
    const int rows = (int)min((int64_t)kB, n - (int64_t)i * kB);
    const double* uk = u + (int64_t)k * kB;
    double dot[NA] = {};
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = y0 + 16 * b + 4 * r + q;
            const double uc = uk[col];
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const int row = x0 + 16 * a + r16;
                if (row < rows && col < kw) C[row + (int64_t)col * n] = acc.v[b][a][r];
                dot[a] = fma(acc.v[b][a][r], uc, dot[a]);
            }
        }
    if (i < k) return;               // uniform over the workgroup
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        dot[a] += __shfl_xor(dot[a], 16, 64);
        dot[a] += __shfl_xor(dot[a], 32, 64);
        if (q == 0) red[wave][16 * a + r16] = dot[a];
    }
    __syncthreads();
    const int t = (int)threadIdx.x;
    if (t < 16 * NA && x0 + t < rows) zrow[(int64_t)i * kB + x0 + t] -= (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
}

__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// 1 / sqrt(d) from the hardware's estimate y (about 2^-22) and one third-order step, y (1 +
// e / 2 + 3 e^2 / 8), e = 1 - d y^2.
__device__ __forceinline__ double rsqrt_step(double d)
{
    const double y = __builtin_amdgcn_rsq(d), e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Orders the LDS accesses of a wave whose lanes exchange data (the hardware runs them in
// program order; the compiler must not reorder them).
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

// The sum of a lane's value over the four lanes of its lane % 16 (swaps of half waves and of
// rows of 16: vector instructions, where a shuffle goes through LDS).
__device__ __forceinline__ double sum_rows(double v)
{
    {
        const unsigned lo = __double2loint(v), hi = __double2hiint(v);
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        v = __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    }
    const unsigned lo = __double2loint(v), hi = __double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}

// A barrier that orders LDS alone: __syncthreads also waits for the wave's global stores.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Diagonal block k: the inverse W_k of its factor (and its transpose), u_k = W_k zrow_k, and
// the block's share of log det L and |u|^2. One workgroup; by 16 x 16 sub-blocks, wave I
// holds block row I in the matrix cores' accumulators, every tile transposed: the lower
// tiles of A, then, in their place from the diagonal on, those of Y = L^-T, which is what
// the same operations make of an identity below A (see the head of this file). Column s:
//  1. wave s factors its diagonal tile as L D L^T, a lane a row, then scales by D^-1/2. The
//     chain from pivot to pivot is d' = a' - a^2 / d in every lane (a, a' read from their
//     lanes beforehand; a^2 is formed first, so the matrix's scale has to be far inside the
//     root of the double range): a reciprocal and four operations. Lanes 16 - 31 carry identity rows,
//     which the same instructions turn into rows of G^T = L_ss^-T, and lane 32 the
//     right-hand side's segment, which becomes u_s.
//  2. the other waves multiply by G (X^T = G A^T: a product's registers are the next one's
//     right operand); rows above s have their final tile of Y, which goes to memory;
//  3. every wave updates its tiles right of s from its own X and the others', in LDS in
//     operand order. Wave s + 1 has one such product, and then factors while others update.
// Rows past n are the identity's. A serial chain, bound by latency: 136 us in the first
// version, 53 with the block in LDS and its inverse built after its factor, 29 now: 128
// pivots of 0.1 us, 8 exchanges of 1.4 us, and 5 us before and after.
__global__ __launch_bounds__(512) void k_chol_diag(const double* __restrict__ S, int64_t n, int nb, int k,
                                                   double* __restrict__ w, double* __restrict__ wt,
                                                   const double* __restrict__ zrow, double* __restrict__ u,
                                                   double* __restrict__ part, int* __restrict__ info)
{
    constexpr int NS = kB / 16;
    static_assert(NS == 8, "a wave a block row");
    __shared__ double sT[16 * 17], sG[16 * 17], su[16], sX[NS][4][64], red[2][NS];
    const int lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int I = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t g0 = (int64_t)k * kB;
    const int live = (int)min((int64_t)kB, n - g0);
    const int row = 16 * I + r16;
    chol4_t acc[NS];                     // [j]: tile (I, s + j), rows of it in lanes r16
#pragma unroll
    for (int J = 0; J < NS; ++J)         // every load in flight; tiles right of the diagonal repeat its columns
#pragma unroll
        for (int c = 0; c < 4; ++c)
            acc[J][c] = S[g0 + min(row, live - 1) + (g0 + min(16 * min(J, I) + q + 4 * c, live - 1)) * n];
#pragma unroll
    for (int J = 0; J < NS; ++J)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int col = 16 * J + q + 4 * c;
            if (J > I) acc[J][c] = 0.0;
            else if (row >= live || col >= live) acc[J][c] = row == col ? 1.0 : 0.0;
        }
    double z = row < live ? zrow[g0 + row] : 0.0, us = 0.0, logs = 0.0;
    double* const wk = w + (int64_t)k * kB * kB;
    double* const wtk = wt + (int64_t)k * kB * kB;
    auto store = [&](int J, const chol4_t& y) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int col = 16 * J + q + 4 * c;
            wtk[row + col * kB] = y[c];
            wk[col + row * kB] = y[c];
        }
    };
    for (int s = 0; s < NS; ++s) {
        if (I == s) {
#pragma unroll
            for (int c = 0; c < 4; ++c) sT[(q + 4 * c) * 17 + r16] = acc[0][c];
            if (q == 0) su[r16] = z;
            wave_lds_order();
            double v[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const double a = q == 0 ? sT[c * 17 + r16] : su[c];      // A's row r16, or z
                v[c] = q == 1 ? (r16 == c ? 1.0 : 0.0) : a;
            }
            double d = lane_value(v[0], 0), pivot = d;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                double r = __builtin_amdgcn_rcp(d);              // about 2^-22, and one third-order step
                // the column's values in the rows below, and the next pivot before it: read
                // together (a lane read just before its use costs wait states)
                double b[16], a = 0.0;
                if (c < 15) a = lane_value(v[c + 1], c + 1);
#pragma unroll
                for (int c2 = c + 1; c2 < 16; ++c2) b[c2] = lane_value(v[c], c2);
                __builtin_amdgcn_sched_barrier(0);
                const double e = fma(-d, r, 1.0);
                r = fma(r, fma(e, e, e), r);
                const double wc = v[c] * r;
                if (c < 15) {
                    d = fma(-b[c + 1] * b[c + 1], r, a);
                    pivot = r16 == c + 1 ? d : pivot;
                }
#pragma unroll
                for (int c2 = c + 1; c2 < 16; ++c2) v[c2] = fma(-wc, b[c2], v[c2]);
            }
            const double y = rsqrt_step(pivot);
            us = y;                                              // 1 / L_rr until the barrier
#pragma unroll
            for (int c = 0; c < 16; ++c) v[c] *= lane_value(y, c);
            if (q == 1)
#pragma unroll
                for (int c = 0; c < 16; ++c) sG[c * 17 + r16] = v[c];
            if (lane == 32)
#pragma unroll
                for (int c = 0; c < 16; ++c) su[c] = v[c];
            if (!(pivot > 0.0)) *info = 1;
        }
        lds_barrier();
        chol4_t x = {0.0, 0.0, 0.0, 0.0};
        const double un = su[r16];
        if (I == s) {
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = sG[(q + 4 * c) * 17 + r16];
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(sG[r16 * 17 + q + 4 * c], acc[0][c], x, 0, 0, 0);
        }
        if (I > s) {
            double t = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                sX[I][c][lane] = x[c];
                t = fma(su[q + 4 * c], x[c], t);
            }
            z -= sum_rows(t);
        }
        lds_barrier();
#pragma unroll
        for (int j = 1; j < NS; ++j) {
            const int m = s + j;
            chol4_t t = acc[j];
            if (m < NS && (I <= s || m <= I)) {
#pragma unroll
                for (int c = 0; c < 4; ++c) t = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[m][c][lane], -x[c], t, 0, 0, 0);
            }
            acc[j - 1] = t;
        }
        // Y's tile (I, s), zero below the diagonal; the next wave to factor leaves its zeros
        // for the end
        if (I != s + 1) store(s, I <= s ? x : chol4_t{0.0, 0.0, 0.0, 0.0});
        if (I == s) {
            logs = -log(us);
            us = un;
        }
    }
    if (I > 0) store(I - 1, chol4_t{0.0, 0.0, 0.0, 0.0});
    if (q == 0) u[g0 + row] = us;
    double sq = us * us;
    for (int d = 8; d > 0; d >>= 1) {
        sq += __shfl_xor(sq, d, 64);
        logs += __shfl_xor(logs, d, 64);
    }
    if (lane == 0) {
        red[0][I] = logs;
        red[1][I] = sq;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < NS; ++i) t += red[threadIdx.x][i];
        part[(int64_t)threadIdx.x * nb + k] = t;
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
// longest sums (small c) come first. 177 GFLOP in 3.1 ms at 8,100 sites (57 TFLOP/s).
template <int NA>
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
    int d = f - c * (c + 1) / 2;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int x0 = 16 * NA * (wave & 1), y0 = 16 * NA * (wave >> 1);
    if (NA == 2) {                                    // tiles of 64 rows: their blocks and halves
        x0 += 64 * (c & 1);
        y0 += 64 * (d & 1);
        c >>= 1;
        d >>= 1;
    }
    Acc<NA, NA> acc;
    const Operand Wc = {wt + (int64_t)c * kB * kB, kB, kB - 1};
    const int full = (int)(n / kB);                   // block columns of full width
    if (c < full) {
        nt_run<4, false>(acc, Wc, c == d ? Wc : s_block(S, n, d, c), x0, y0, kB);
        if (c + 1 < full) nt_run<4, false>(acc, s_block(S, n, c, c + 1), s_block(S, n, d, c + 1), x0, y0, kB * (full - c - 1));
    }
    if (full < nb)
        nt_run<4, true>(acc, c == full ? Wc : s_block(S, n, c, full), d == full ? Wc : s_block(S, n, d, full), x0, y0,
                        (int)(n - (int64_t)full * kB));
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t row0 = (int64_t)c * kB + x0 + (lane & 15), col0 = (int64_t)d * kB + y0 + (lane >> 4);
#pragma unroll
    for (int b = 0; b < NA; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t j = col0 + 16 * b + 4 * r;
#pragma unroll
            for (int a = 0; a < NA; ++a) {
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

// res[k] = sum_p part[p * ps + k * ks], a workgroup each k, fixed order.
__global__ __launch_bounds__(256) void k_chol_sum(const double* __restrict__ part, int64_t np, int64_t ps, int64_t ks,
                                                  double* __restrict__ res)
{
    __shared__ double red[4];
    const int k = (int)blockIdx.x;
    double s = 0.0;
    for (int64_t p = threadIdx.x; p < np; p += 256) s += part[p * ps + k * ks];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) res[k] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void k_chol_begin(const double* __restrict__ z, double zscale, double* __restrict__ zrow,
                                                    int64_t n, int* __restrict__ info)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) zrow[i] = zscale * z[i];
    if (i == 0) *info = 0;
}

int chol_solve(double* S, const double* dB, const double* dN, const double* z, double zscale, int64_t n,
               const CholWork& wk, hipStream_t stream)
{
    const int nb = (int)chol_blocks(n), inverse = dB ? 1 : 0;
    const double *w = wk.w, *wt = wk.wt, *u = wk.u, *zrow = wk.zrow, *Sc = S;
    const dim3 wg(256);
    int st = launch(k_chol_begin, dim3((unsigned)((n + 255) / 256)), wg, stream, z, zscale, wk.zrow, n, wk.info);
    auto diag = [&](int k) {
        if (st == BK_OK)
            st = launch(k_chol_diag, dim3(1), dim3(512), stream, Sc, n, nb, k, wk.w, wk.wt, zrow, wk.u, wk.part, wk.info);
    };
    auto panel = [&](int k) {
        const int blocks = nb - 1 - k + (inverse ? k : 0);
        if (st != BK_OK || blocks <= 0) return;
        st = blocks <= kFewBlocks ? launch(k_chol_panel<1>, dim3(8 * blocks), wg, stream, S, n, nb, w, u, wk.zrow, k)
                                  : launch(k_chol_panel<2>, dim3(4 * blocks), wg, stream, S, n, nb, w, u, wk.zrow, k);
    };
    auto column = [&](int k0, int m) {
        if (st != BK_OK || k0 >= m) return;
        const int blocks = nb - m + (inverse ? m : 0);
        st = blocks <= kFewBlocks ? launch(k_chol_column<1>, dim3(8 * blocks), wg, stream, S, n, nb, wt, k0, m, m)
                                  : launch(k_chol_column<2>, dim3(4 * blocks), wg, stream, S, n, nb, wt, k0, m, m);
    };
    // several panels a trailing update (its blocks of S are read and written that much less
    // often), each block column of the step brought up to date just before its turn
    const int step = update_step(nb);
    for (int k = 0; k < nb; k += step) {
        const int ke = k + step < nb ? k + step : nb;
        for (int j = k; j < ke; ++j) {
            column(k, j);
            diag(j);
            panel(j);
        }
        if (st == BK_OK && ke < nb) {
            const int rows = nb - ke + (inverse ? ke : 0), cols = nb - ke;
            st = rows * cols >= kFewTiles ? launch(k_chol_update<4>, dim3(rows, cols), wg, stream, S, n, nb, wt, k, ke, ke, inverse)
                                         : launch(k_chol_update<2>, dim3(4 * rows, cols), wg, stream, S, n, nb, wt, k, ke, ke,
                                                  inverse);
        }
    }
    const double* part = wk.part;
    if (st == BK_OK) st = launch(k_chol_sum, dim3(2), wg, stream, part, (int64_t)nb, (int64_t)1, (int64_t)nb, wk.res);
    if (!inverse || st != BK_OK) return st;
    st = launch(k_chol_yu, dim3(nb, nb), wg, stream, Sc, n, wt, u, wk.ypart);
    if (st == BK_OK)
        st = launch(k_chol_ysum, dim3((unsigned)((n + 255) / 256)), wg, stream, (const double*)wk.ypart, n, nb, wk.a);
    const int64_t tiles = chol_trace_tiles(n);
    const dim3 grid((unsigned)tiles);
    if (st == BK_OK)
        st = nb >= kTraceBlocks
            ? launch(k_chol_traces<4>, grid, wg, stream, Sc, n, nb, wt, (const double*)wk.a, dB, dN, wk.part)
            : launch(k_chol_traces<2>, grid, wg, stream, Sc, n, nb, wt, (const double*)wk.a, dB, dN, wk.part);
    if (st == BK_OK) st = launch(k_chol_sum, dim3(4), wg, stream, part, tiles, (int64_t)4, (int64_t)1, wk.res + 2);
    return st;
}

}  // namespace bk
