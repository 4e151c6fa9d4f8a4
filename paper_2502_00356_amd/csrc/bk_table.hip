// bk_table.hip - Matern tiles (and their beta and nu derivatives) by interpolation in
// r^2 (bk_table.hpp): the table builder of the plain and mixed forms and of the
// gradient, the evaluation kernel shared with the learned form, and the rule that
// chooses between it and the per-entry kernels.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/besselk.h"
#include "bk_table.hpp"

namespace bk {

// The function fn at z, by the plain FP64 quadrature.
template <bool kGrad>
__device__ inline double tab_sample(const TabParams& P, double z, int fn, const double* T)
{
    const double L = kDefaultLPlain, Lq = kDefaultLqPlain;
    const double nu = kGrad && fn == TAB_DBETA ? fabs(P.nu - 1.0) : P.nu;
    const Solved s = plain_plan(nu, z, L, Lq, rule_tab(), T);
    double hs = s.p.h * sum_f64(nu, z, s.p, s.E, s.Ei, s.Sr, T);
    hs = fma(hs, s.dlo, hs);
    if (kGrad && fn == TAB_DBETA) return tab_assemble(P.scale * P.inv_beta, z, P.nu + 1.0, s.delta, hs);
    const double c = tab_assemble(P.scale, z, P.nu, s.delta, hs);
    if (!kGrad || fn == TAB_C) return c;
    double dd, dhs;
    dnu_integral(nu, z, s.p.t0, L, Lq, rule_tab(), T, dd, dhs);
    return fma(c, log(z) - kLn2 - P.psi, tab_assemble(P.scale, z, P.nu, dd, dhs));
}

// ---------------------------------------------------------------------------
// Builder: one plain FP64 evaluation per Chebyshev point, one lane each.
// ---------------------------------------------------------------------------
template <bool kF32, bool kGrad>
__global__ __launch_bounds__(64) void k_tab_build(TabParams P, TabIndex X, char* t0, char* t1, char* t2)
{
    __shared__ double s_tab[kTabLen], sh[64];
    stage_tab(s_tab);
    const TabWave<kF32> t = tab_point<kF32>(X, P.inv_beta, blockIdx.x);
    const int fn = kGrad ? (int)blockIdx.y : TAB_C;
    char* table = fn == TAB_C ? t0 : (fn == TAB_DBETA ? t1 : t2);
    if (!table) return;
    const double f = tab_sample<kGrad>(P, t.z, fn, s_tab);
    tab_fit<kF32>(t, f, X, sh, table);
    if (blockIdx.x == 0 && threadIdx.x == 0) *tab_done<kF32>(table) = 0u;
}

// ---------------------------------------------------------------------------
// Evaluation
// ---------------------------------------------------------------------------
// An entry whose distance is outside the table: z below kZMin or past 128, NaN or
// infinite coordinates. Out of line, so that its registers stay out of the tile loop.
template <int FN, int MODE>
__device__ __noinline__ double tab_cold(double q, TabParams P)
{
    const double r = sqrt(q);
    if (r == 0.0) return FN == TAB_C ? P.sigma2 : 0.0;
    const double z = r * P.inv_beta, lz = log(z);
    double L, Lq;
    if constexpr (MODE == BK_PLAIN_F64) { L = kDefaultLPlain; Lq = kDefaultLqPlain; }
    else { L = kDefaultLMixed; Lq = kDefaultLqMixed; }
    const double* T = rule_tab().tab;
    if constexpr (FN == TAB_DBETA) {
        return matern_dbeta(P.nu, z, lz, P.sigma2, P.inv_beta, P.pref, L, Lq, T);
    } else {
        Solved s;
        const double c = matern_entry<MODE>(P.nu, z, lz, P.sigma2, P.pref, L, Lq, T, s);
        if constexpr (FN == TAB_C) return c;
        else return matern_dnu(P.nu, z, lz, P.sigma2, P.pref, P.psi, L, Lq, T, c, s.p.t0);
    }
}

// The evaluation's launch: 512-lane workgroups, two on each of the 256 CUs (the FP64
// table takes 67 KB of LDS), 128 VGPRs. Measured on 30,000 sites in 1,024-tiles (FP64,
// 7.2 GB written): 1.52 ms; one 1,024-lane workgroup a CU the same, 64 VGPRs and twice
// the waves 1.55.
constexpr int kTabThreads = 512, kTabWaves = kTabThreads / 64;
constexpr unsigned kTabGrid = 512;

struct TabArgs {
    TileGeom g;                    // rb_per_tile: row blocks of 64 lanes; cb_per_tile: column blocks of `cols`
    int cols;
    unsigned items;                // tiles x row blocks x column blocks
    int64_t first;                 // first output element over the table
    TabIndex X;
    TabParams P;
};

// The slot of squared distance q. The conversion takes anything below the first
// interval (and NaN) to slot 0; that and the last slot hold a NaN constant term, so an
// entry out of the table shows in its value.
template <bool kF32>
__device__ __forceinline__ int tab_slot(const TabIndex& X, double q)
{
    return (int)min(__float2uint_rz(tab_pos(X, (float)q)), (unsigned)(TabShape<kF32>::kN - 1));
}

template <bool kF32>
__device__ __forceinline__ double tab_value(const TabIndex& X, const tab2_t* sT, double q, int i)
{
    constexpr int kN = TabShape<kF32>::kN;
    const tab2_t s0 = sT[i];
    const double v = q - s0[0];
    if constexpr (kF32) {
        const tab4f_t c = ((const tab4f_t*)sT)[kN + i];
        const float u = (float)v * X.vs;
        return fma((double)(fmaf(fmaf(fmaf(c[3], u, c[2]), u, c[1]), u, c[0]) * u), s0[1], s0[1]);
    } else {
        static_assert(TabShape<false>::kDeg == 8, "table planes");
        const tab2_t s1 = sT[kN + i], s2 = sT[2 * kN + i], s3 = sT[3 * kN + i], s4 = sT[4 * kN + i];
        double p = fma(s4[1], v, s4[0]);
        p = fma(p, v, s3[1]);
        p = fma(p, v, s3[0]);
        p = fma(p, v, s2[1]);
        p = fma(p, v, s2[0]);
        p = fma(p, v, s1[1]);
        p = fma(p, v, s1[0]);
        return fma(p, v, s0[1]);
    }
}

// R consecutive output elements, aligned to one element only.
template <typename OutT, int R>
struct __attribute__((packed, aligned(sizeof(OutT)))) TabRun {
    OutT v[R];
};

// One item: 64 R rows (R consecutive ones a lane, stored together) and `cols` columns
// of a tile; the elements in [lo, hi) of the output.
template <typename OutT, bool kF32, int FN, int MODE, int R>
__device__ __forceinline__ void tab_item(const TabArgs& A, const tab2_t* sT, const double* __restrict__ lx,
                                         const double* __restrict__ ly, OutT* out, int64_t I, int64_t J, int rb, int cb,
                                         int64_t lo, int64_t hi)
{
    const TileGeom& g = A.g;
    const int64_t mI = min((int64_t)g.ts, g.n - I * g.ts), nJ = min((int64_t)g.ts, g.n - J * g.ts);
    const int64_t jl0 = (int64_t)cb * A.cols, il0 = (int64_t)rb * (64 * R);
    if (jl0 >= nJ || il0 >= mI) return;
    const int lane = threadIdx.x & 63, row = lane * R;
    const int rows = (int)min((int64_t)(64 * R), mI - il0);
    const int cend = (int)min((int64_t)A.cols, nJ - jl0);
    const int64_t off0 = tile_offset(g.n, g.ts, g.T, g.lower, I, J) + jl0 * mI + il0;
    const bool clip = off0 < lo || off0 + (int64_t)(cend - 1) * mI + rows > hi;
    if (row >= rows) return;
    const bool whole = !clip && rows % R == 0;
    const double* __restrict__ xr = lx + I * g.ts + il0;
    const double* __restrict__ yr = ly + I * g.ts + il0;
    double xi[R], yi[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int e = min(row + k, rows - 1);
        xi[k] = xr[e];
        yi[k] = yr[e];
    }
    // the row points are waited for here, once: a wait for them inside the column loop
    // would also wait for the previous column's store
#pragma unroll
    for (int k = 0; k < R; ++k) asm volatile("" ::"v"(xi[k]), "v"(yi[k]));
    const double* __restrict__ xc = lx + J * g.ts + jl0;
    const double* __restrict__ yc = ly + J * g.ts + jl0;
    OutT* col = out + off0;
    for (int c = 0; c < cend; ++c) {
        const double xj = xc[c], yj = yc[c];
        double q[R], v[R];
        int i[R];
        TabRun<OutT, R> val;
        // no branch between the R entries: their LDS reads are in flight together
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const double dx = xj - xi[k], dy = yj - yi[k];
            q[k] = fma(dx, dx, dy * dy);
            i[k] = tab_slot<kF32>(A.X, q[k]);
        }
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = tab_value<kF32>(A.X, sT, q[k], i[k]);
        OutT any = (OutT)0;
#pragma unroll
        for (int k = 0; k < R; ++k) any += val.v[k] = (OutT)v[k];
        if (__builtin_expect(isnan(any), 0)) {
            bool cold = false;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if (q[k] == 0.0) val.v[k] = FN == TAB_C ? (OutT)A.P.sigma2 : (OutT)0;
                cold |= isnan(val.v[k]);
            }
            if (cold) {
#pragma unroll
                for (int k = 0; k < R; ++k)
                    if (isnan(val.v[k])) val.v[k] = (OutT)tab_cold<FN, MODE>(q[k], A.P);
            }
        }
        if (__builtin_expect(whole, 1)) {
            *(TabRun<OutT, R>*)(col + row) = val;
        } else {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int64_t o = (col - out) + row + k;
                if (row + k < rows && o >= lo && o < hi) col[row + k] = val.v[k];
            }
        }
        col += mI;
    }
}

// Persistent: a workgroup copies the table to LDS once and its waves take items in turn.
// Bound by the output's write: with the arithmetic taken out the same stores take 1.37 ms
// of the 1.52 (FP64, 30,000 sites in 1,024-tiles, 4.7 TB/s) and 0.70 of the 0.83 (FP32,
// 4.3 TB/s); without the stores the arithmetic and LDS reads take 0.89 and 0.64. 20 (FP32)
// and 25 (FP64) VALU instructions an entry against the per-entry quadrature's 1,839:
// 40,000 sites, lower 960-tiles, nu = 2.3, plain FP64 40.0 -> 1.39 ms; 9,001 sites, mixed
// FP32, 2.60 -> 0.137 ms; C, dC/dbeta and dC/dnu of 12,000 sites 16.6 -> 0.49 ms (tables
// included).
template <typename OutT, bool kF32, int FN, int MODE, int R>
__global__ __launch_bounds__(kTabThreads, 4) void k_matern_tab(const double* __restrict__ lx, const double* __restrict__ ly,
                                                           TabArgs A, char* table, OutT* out)
{
    constexpr int kSlots = TabShape<kF32>::kPlanes * TabShape<kF32>::kN;
    constexpr unsigned kWaves = kTabWaves;
    __shared__ tab2_t sT[kSlots];
    __shared__ unsigned s_last;
    for (int k = threadIdx.x; k < kSlots; k += kTabThreads) sT[k] = ((const tab2_t*)table)[k];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const TileGeom& g = A.g;
    const unsigned rbn = (unsigned)g.rb_per_tile, per_tile = rbn * (unsigned)g.cb_per_tile;
    for (unsigned it = blockIdx.x * kWaves + wave; it < A.items; it += gridDim.x * kWaves) {
        const unsigned p = it / per_tile, local = it - p * per_tile;
        int64_t I, J;
        tile_of(p, g, I, J);
        tab_item<OutT, kF32, FN, MODE, R>(A, sT, lx, ly, out, I, J, (int)(local % rbn), (int)(local / rbn), 0, A.first);
    }
    // The workgroup that finishes last (every other has read the table long before)
    // writes the elements the table lay in.
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(tab_done<kF32>(table), 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    const unsigned tiles = A.items / per_tile;
    for (unsigned p = tiles; p-- > 0;) {
        int64_t I, J;
        tile_of(p, g, I, J);
        const int64_t mI = min((int64_t)g.ts, g.n - I * g.ts), nJ = min((int64_t)g.ts, g.n - J * g.ts);
        const int64_t off = tile_offset(g.n, g.ts, g.T, g.lower, I, J);
        if (off + mI * nJ <= A.first) break;
        const unsigned cb0 = A.first > off ? (unsigned)((A.first - off) / mI / A.cols) : 0u;
        for (unsigned k = wave; k < (g.cb_per_tile - cb0) * rbn; k += kWaves)
            tab_item<OutT, kF32, FN, MODE, R>(A, sT, lx, ly, out, I, J, (int)(k % rbn), (int)(cb0 + k / rbn), A.first,
                                              INT64_MAX);
    }
}

// ---------------------------------------------------------------------------
// Host
// ---------------------------------------------------------------------------
static size_t table_bytes(bool f32_table) { return f32_table ? tab_bytes<true>() : tab_bytes<false>(); }

char* table_in_output(void* out, int64_t elems, int elem_bytes, bool f32_table, int64_t* first)
{
    *first = elems - (int64_t)((table_bytes(f32_table) + 16 + elem_bytes - 1) / elem_bytes);
    const uintptr_t a = (uintptr_t)out + (uintptr_t)*first * elem_bytes;
    return (char*)((a + 15) & ~(uintptr_t)15);
}

bool table_route(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only, int64_t min_entries)
{
    if (prm->L_window != 0.0 || prm->L_quad != 0.0) return false;
    if (!(prm->nu >= 0.01 && prm->nu <= 16.0)) return false;
    if (!(prm->beta >= 1e-8 && prm->beta <= 1e8)) return false;
    if (!(prm->sigma2 >= 1e-100 && prm->sigma2 <= 1e100)) return false;
    const int64_t n = locs->n, ts = tile_size < n ? tile_size : n, T = (n + ts - 1) / ts;
    if (n >= (1LL << 31)) return false;
    const int64_t items = (lower_only ? T * (T + 1) / 2 : T * T) * ((ts + 63) / 64) * ((ts + 7) / 8);
    if (T >= 60000 || items >= (1LL << 31)) return false;
    return bk_matern_out_elems(n, tile_size, lower_only) >= min_entries;
}

template <typename OutT, bool kF32, int FN, int MODE, int R>
static int eval_rows(const bk_locs* locs, TabArgs& A, char* table, OutT* out, hipStream_t stream)
{
    const int64_t tiles = A.g.lower ? (int64_t)A.g.T * (A.g.T + 1) / 2 : (int64_t)A.g.T * A.g.T;
    A.g.rb_per_tile = (A.g.ts + 64 * R - 1) / (64 * R);
    // 16 columns an item; fewer where that leaves waves of the grid without one
    for (A.cols = 16;; A.cols >>= 1) {
        A.g.cb_per_tile = (A.g.ts + A.cols - 1) / A.cols;
        A.items = (unsigned)(tiles * A.g.rb_per_tile * A.g.cb_per_tile);
        if (A.cols == 2 || A.items >= kTabWaves * kTabGrid) break;
    }
    const unsigned need = (A.items + kTabWaves - 1) / kTabWaves;
    return launch(k_matern_tab<OutT, kF32, FN, MODE, R>, dim3(need < kTabGrid ? need : kTabGrid), dim3(kTabThreads),
                  stream, locs->x, locs->y, A, table, out);
}

// Rows a lane: four, stored together (16 or 32 bytes), so that a wave writes 1 or 2 KB of
// a column at once and few 128-byte lines are written in parts where tile rows are not
// whole lines (30,000 sites in 1,000-tiles, FP64: 1.58 ms with four, 1.85 with two, 2.07
// with one; FP32 0.83, 1.18, 1.27). Two or one where four would leave over a fifth more
// lanes idle at the tile's end.
template <typename OutT, bool kF32, int FN, int MODE>
static int eval_launch(const bk_locs* locs, TabArgs& A, char* table, void* out, hipStream_t stream)
{
    auto lanes = [&](int r) { return (A.g.ts + 64 * r - 1) / (64 * r) * (64 * r); };
    if (5 * lanes(4) <= 6 * lanes(1))
        return eval_rows<OutT, kF32, FN, MODE, 4>(locs, A, table, (OutT*)out, stream);
    if (5 * lanes(2) <= 6 * lanes(1))
        return eval_rows<OutT, kF32, FN, MODE, 2>(locs, A, table, (OutT*)out, stream);
    return eval_rows<OutT, kF32, FN, MODE, 1>(locs, A, table, (OutT*)out, stream);
}

TabIndex tab_index(double beta, bool f32_table)
{
    const double a = f32_table ? TabShape<true>::kA : TabShape<false>::kA;
    const double b = f32_table ? TabShape<true>::kB : TabShape<false>::kB;
    const double z = f32_table ? TabShape<true>::kZMin : TabShape<false>::kZMin;
    // bits(q) 2^-23 at the first boundary: exponent field plus the mantissa's fraction
    int e;
    const double q = z * z * beta * beta, m = frexp(q, &e);
    TabIndex X;
    X.fa = (float)(a * 0x1p-23);
    X.fb = (float)(b / beta);
    X.fc = (float)(1.0 - a * ((double)(e - 1 + 127) + (2.0 * m - 1.0)) - b * z);     // slot 1
    X.vs = (float)(1.0 / (beta * beta));
    return X;
}

int launch_table_eval(const bk_locs* locs, const TabParams& P, int32_t tile_size, int32_t lower_only, int fn,
                      int cold_mode, bool f32_table, int out_dtype, void* out, hipStream_t stream)
{
    TabArgs A;
    A.P = P;
    const int64_t n = locs->n;
    const int elem = out_dtype == BK_OUT_F32 ? 4 : 8;
    char* table = table_in_output(out, bk_matern_out_elems(n, tile_size, lower_only), elem, f32_table, &A.first);
    A.g.n = n;
    A.g.ts = (int32_t)(tile_size < n ? tile_size : n);
    A.g.T = (int32_t)((n + A.g.ts - 1) / A.g.ts);
    A.g.lower = lower_only ? 1 : 0;
    A.X = tab_index(P.beta, f32_table);
    const bool f32 = out_dtype == BK_OUT_F32;
    if (f32_table) return eval_launch<float, true, TAB_C, BK_MIXED_F32C>(locs, A, table, out, stream);
    switch (fn) {
    case TAB_C:
        return f32 ? eval_launch<float, false, TAB_C, BK_PLAIN_F64>(locs, A, table, out, stream)
                   : eval_launch<double, false, TAB_C, BK_PLAIN_F64>(locs, A, table, out, stream);
    case TAB_DBETA:
        return f32 ? eval_launch<float, false, TAB_DBETA, BK_PLAIN_F64>(locs, A, table, out, stream)
                   : eval_launch<double, false, TAB_DBETA, BK_PLAIN_F64>(locs, A, table, out, stream);
    default:
        return f32 ? eval_launch<float, false, TAB_DNU, BK_PLAIN_F64>(locs, A, table, out, stream)
                   : eval_launch<double, false, TAB_DNU, BK_PLAIN_F64>(locs, A, table, out, stream);
    }
}

TabParams tab_params(const bk_params* prm, double psi)
{
    return {prm->sigma2, prm->beta, 1.0 / prm->beta, prm->nu, (1.0 - prm->nu) * kLn2 - lgamma(prm->nu), psi,
            (double)((long double)prm->sigma2 * exp2l(1.0L - prm->nu) / tgammal(prm->nu))};
}

int matern_table_tiles(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only, void* out,
                       hipStream_t stream)
{
    const bool f32_table = prm->mode == BK_MIXED_F32C;
    const TabParams P = tab_params(prm, 0.0);
    const TabIndex X = tab_index(prm->beta, f32_table);
    int64_t first;
    char* table = table_in_output(out, bk_matern_out_elems(locs->n, tile_size, lower_only),
                                  prm->out_dtype == BK_OUT_F32 ? 4 : 8, f32_table, &first);
    int st = f32_table ? launch(k_tab_build<true, false>, dim3(TabWave<true>::kBlocks), dim3(64), stream, P, X, table,
                                nullptr, nullptr)
                       : launch(k_tab_build<false, false>, dim3(TabWave<false>::kBlocks), dim3(64), stream, P, X, table,
                                nullptr, nullptr);
    if (st != BK_OK) return st;
    if (mark_kernel_event(prm, 0, stream) != hipSuccess) return BK_EHIP;
    st = launch_table_eval(locs, P, tile_size, lower_only, TAB_C, prm->mode, f32_table, prm->out_dtype, out, stream);
    if (st != BK_OK) return st;
    return mark_kernel_event(prm, 1, stream) == hipSuccess ? BK_OK : BK_EHIP;
}

int matern_grad_table_tiles(const bk_locs* locs, const bk_params* prm, double psi, int32_t tile_size,
                            int32_t lower_only, void* const outs[3], hipStream_t stream)
{
    const TabParams P = tab_params(prm, psi);
    const int64_t elems = bk_matern_out_elems(locs->n, tile_size, lower_only);
    const int elem = prm->out_dtype == BK_OUT_F32 ? 4 : 8;
    char* tab[3];
    int64_t first;
    for (int k = 0; k < 3; ++k) tab[k] = outs[k] ? table_in_output(outs[k], elems, elem, false, &first) : nullptr;
    int st = launch(k_tab_build<false, true>, dim3(TabWave<false>::kBlocks, 3), dim3(64), stream, P, tab_index(prm->beta, false), tab[0], tab[1],
                    tab[2]);
    for (int k = 0; k < 3 && st == BK_OK; ++k)
        if (outs[k])
            st = launch_table_eval(locs, P, tile_size, lower_only, k, BK_PLAIN_F64, false, prm->out_dtype, outs[k],
                                   stream);
    return st;
}

}  // namespace bk
