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

// The function fn at z, by the plain FP64 quadrature of kTabLanes lanes.
constexpr int kTabLanes = 4;

template <bool kGrad>
__device__ inline double tab_sample(const TabParams& P, double z, int fn, int sub, const double* T)
{
    const double L = kDefaultLPlain, Lq = kDefaultLqPlain;
    const double nu = kGrad && fn == TAB_DBETA ? fabs(P.nu - 1.0) : P.nu;
    float t0, t1;
    unsigned int N, mc;
    if (kGrad && fn == TAB_DNU) deriv_window_count(nu, z, L, Lq, t0, t1, N, mc);
    else window_count(nu, z, L, Lq, t0, t1, N, mc);
    const Solved s = plan_setup(nu, z, t0, t1, N, mc);
    const double h = fma(s.p.h, s.dlo, s.p.h);
    if (kGrad && fn == TAB_DNU) {
        const DerivSums S = sum_split<kTabLanes, true>(nu, z, s.p, s.E, s.Ei, s.Sr, sub, T);
        return tab_assemble(P.scale, z, P.nu, s.delta, h * fma(S.k, log(z) - kLn2 - P.psi, S.d));
    }
    const double hs = h * sum_split<kTabLanes, false>(nu, z, s.p, s.E, s.Ei, s.Sr, sub, T).k;
    if (kGrad && fn == TAB_DBETA) return tab_assemble(P.scale * P.inv_beta, z, P.nu + 1.0, s.delta, hs);
    return tab_assemble(P.scale, z, P.nu, s.delta, hs);
}

// ---------------------------------------------------------------------------
// Builder: one plain FP64 evaluation per Chebyshev point, by kTabLanes lanes; one wave's
// worth of points (TabWave) a workgroup. A hundred workgroups on 256 CUs, so its time is
// one lane's serial chain: 13.2 us with a lane a point and a 31-step search for each
// interval's ends, 12.1 with tab_bound's Newton steps, 9.0 with two lanes a point, 7.2
// with four, 8.2 with eight.
// ---------------------------------------------------------------------------
template <bool kF32, bool kGrad>
__global__ __launch_bounds__(64 * kTabLanes) void k_tab_build(TabParams P, TabIndex X, char* t0, char* t1, char* t2)
{
    __shared__ double s_tab[kTabLen], sh[64];
    stage_tab(s_tab);
    const int point = threadIdx.x / kTabLanes, sub = threadIdx.x % kTabLanes;
    const TabWave<kF32> t = tab_point<kF32>(X, P.inv_beta, blockIdx.x, point);
    const int fn = kGrad ? (int)blockIdx.y : TAB_C;
    char* table = fn == TAB_C ? t0 : (fn == TAB_DBETA ? t1 : t2);
    if (!table) return;
    const double f = tab_sample<kGrad>(P, t.z, fn, sub, s_tab);
    tab_fit<kF32>(t, f, X, sh, table, point, sub == 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) tab_clear<kF32>(table);
}

// ---------------------------------------------------------------------------
// Evaluation
// ---------------------------------------------------------------------------
// An entry past the table (kTabFar <= z < P.zero) by Hankel's series of K_nu(z) and its
// order derivative, K = sqrt(pi / 2z) e^-z sum_k prod_j (4 nu^2 - (2j-1)^2) / (8 j z): 16
// terms leave 3e-18 there for nu up to 16, and none cancels. e^-z as two factors, so that
// neither is subnormal before the product is. 25e6 entries at a mean z of 260:
// FP64 0.58 ms (1.13 by the quadrature), C, dC/dbeta and dC/dnu 1.9 (4.6).
template <int FN>
__device__ __forceinline__ double tab_far(double z, const TabParams& P)
{
    const double iz = 1.0 / z, nu = FN == TAB_DBETA ? P.nu - 1.0 : P.nu, mu = 4.0 * nu * nu;
    double s = 1.0, d = 0.0;
#pragma unroll
    for (int k = 16; k >= 1; --k) {
        const double f = (mu - (double)((2 * k - 1) * (2 * k - 1))) * (iz * (0.125 / k));
        if constexpr (FN == TAB_DNU) d = fma(f, d, nu * iz * (1.0 / k) * s);
        s = fma(f, s, 1.0);
    }
    double w = P.scale * pow(z, P.nu) * (1.2533141373155002512 * sqrt(iz));     // sqrt(pi / 2)
    if constexpr (FN == TAB_DBETA) w *= z * P.inv_beta;
    if constexpr (FN == TAB_DNU) s = fma(s, log(z) - kLn2 - P.psi, d);
    const double e = exp(-0.5 * z);
    return w * e * s * e;
}

// Entries below the table (z < kZMin): ranges far above the domain put all of them there.
// 5,000 sites, lower tiles, z near 5e-5, by the per-entry kernels, the quadrature out of line
// and these forms, us: plain 1,676, 1,747, 407; mixed 766, 997, 392; C, dC/dbeta and dC/dnu
// 6,757, 7,085, 1,005. Above 1e-14 neither K_nu nor z^nu leaves the double range (nu <= 16).
constexpr double kTabNear = 1e-14, kTabNearEnd = 0x1p-10;

// dC/dnu there. With y = z^2 / 4, e = nu - 1 and H = Gamma(2 - nu) / Gamma(1 + nu),
//   C / sigma2 = 1 + y (e^w - 1) / e + y^2 e^w / (e (1 + nu)) + O(y^2),  w = e a, a = ln y + ln H / e
// (the two power series of K_nu; the pole at nu = 1 is in neither part). The second part
// matters below nu = 0.95 only, e^w below 1.9. q0 = ln H / e and q1 its derivative: the result
// is within 1e-15 sigma2 (the quadrature cancels terms of size sigma2 |ln z|).
struct TabNear {
    double inv_beta, sigma2, nu, q0, q1;
};

__device__ __noinline__ double tab_near_dnu(double q, TabNear N)
{
    const double y = 0.25 * (q * N.inv_beta) * N.inv_beta, e = N.nu - 1.0;
    if (N.nu >= 1.9) return N.sigma2 * (y / (e * e));
    const double a = log(y) + N.q0, w = e * a, w1 = fma(e, N.q1, a), ew = exp(w);
    // (e^w - 1) / w and its derivative
    double f, fd;
    if (fabs(w) < 0.02) {
        f = fma(fma(fma(fma(fma(w, 1.0 / 720.0, 1.0 / 120.0), w, 1.0 / 24.0), w, 1.0 / 6.0), w, 0.5), w, 1.0);
        fd = fma(fma(fma(fma(w, 1.0 / 144.0, 1.0 / 30.0), w, 0.125), w, 1.0 / 3.0), w, 0.5);
    } else {
        f = expm1(w) / w;
        fd = (ew - f) / w;
    }
    double d = y * fma(N.q1, f, a * fd * w1);
    if (N.nu < 0.95) d += y * y * ew / (e * (1.0 + N.nu)) * (w1 - 1.0 / e - 1.0 / (1.0 + N.nu));
    return N.sigma2 * d;
}

// C and dC/dbeta there, by Temme's series.
template <int FN>
__device__ __forceinline__ double tab_near(double z, const TabParams& P, const double* T)
{
    const double nu = FN == TAB_DBETA ? fabs(P.nu - 1.0) : P.nu;
    const double w = pow(z, P.nu) * temme_k(nu, z, temme_tab(), T);
    return P.scale * (FN == TAB_DBETA ? w * z * P.inv_beta : w);
}

// An entry whose distance is outside the table: z below kZMin or past 128, NaN or
// infinite coordinates. Out of line, so that its registers stay out of the tile loop.
template <int FN, int MODE>
__device__ __noinline__ double tab_cold(double q, TabParams P)
{
    const double r = sqrt(q);
    if (r == 0.0) return FN == TAB_C ? P.sigma2 : 0.0;
    const double z = r * P.inv_beta;
    if (z >= kTabFar && z < __builtin_inf()) return z < P.zero ? tab_far<FN>(z, P) : 0.0;
    const double lz = log(z);
    double L, Lq;
    if constexpr (MODE == BK_PLAIN_F64) { L = kDefaultLPlain; Lq = kDefaultLqPlain; }
    else { L = kDefaultLMixed; Lq = kDefaultLqMixed; }
    const double* T = rule_tab().tab;
    if constexpr (FN != TAB_DNU)
        if (z >= kTabNear && z < kTabNearEnd) return tab_near<FN>(z, P, T);
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

// A call's output falls into three parts: the elements below `first`; the table's bytes
// [first, count), written once every workgroup has read the table; and the rest, which
// holds the counts of workgroups and is written by the last to finish. The first is cut
// into items over whole tiles of `cols` columns; the others into items of kTailCols
// columns, tile by tile from the one that holds their first element.
constexpr int kTailCols = 2;
// Workgroups that share the second part, written by the last to finish alone before: 517
// sites (FP32, lower 128-tiles) 32.5 us a call then, 23.3 with 16 or 64, 26 with 8; 1,024
// sites (FP64) 22.4, 22.4 and 24.3, 22.0. 20.1 and 21.2 now (TailStart, TailWalk).
constexpr unsigned kTailGroups = 16;

struct TailStart {
    int32_t I, J, col;
};

struct TailWalk : TailStart {
    unsigned base;
};

struct TabArgs {
    TileGeom g;                    // rb_per_tile: row blocks of 64 R; cb_per_tile: column blocks of `cols`
    int cols;
    unsigned items;
    TailStart first_at, count_at;  // tile and column that hold elements first and count
    int64_t first, count;
    TabIndex X;
    TabParams P;
    TabNear N;                     // dC/dnu: of entries with near <= r^2 < near_end
    double near, near_end;
};

// The slot of squared distance q. The conversion takes anything below the first
// interval (and NaN) to slot 0; that and the last slot hold a NaN constant term, so an
// entry out of the table shows in its value (an FP32 table's last slot 0 where the function
// rounds to 0 from there on).
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

// One item: 64 R rows (R consecutive ones a lane, stored together) from row il0 and up to
// `cols` columns from jl0 of a tile; the elements in [lo, hi) of the output.
template <typename OutT, bool kF32, int FN, int MODE, int R>
__device__ __forceinline__ void tab_item(const TabArgs& A, const tab2_t* sT, const double* __restrict__ lx,
                                         const double* __restrict__ ly, OutT* out, int64_t I, int64_t J, int64_t il0,
                                         int64_t jl0, int cols, int64_t lo, int64_t hi)
{
    const TileGeom& g = A.g;
    const int64_t mI = min((int64_t)g.ts, g.n - I * g.ts), nJ = min((int64_t)g.ts, g.n - J * g.ts);
    if (jl0 >= nJ || il0 >= mI) return;
    const int lane = threadIdx.x & 63, row = lane * R;
    const int rows = (int)min((int64_t)(64 * R), mI - il0);
    const int cend = (int)min((int64_t)cols, nJ - jl0);
    const int64_t off0 = tile_offset(g.n, g.ts, g.T, g.lower, I, J) + jl0 * mI + il0;
    if (off0 >= hi || off0 + (int64_t)(cend - 1) * mI + rows <= lo) return;
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
                    if (isnan(val.v[k]))
                        val.v[k] = (OutT)(FN == TAB_DNU && q[k] >= A.near && q[k] < A.near_end
                                              ? tab_near_dnu(q[k], A.N)
                                              : tab_cold<FN, MODE>(q[k], A.P));
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
// FP32, 2.60 -> 0.104 ms; C, dC/dbeta and dC/dnu of 12,000 sites 16.6 -> 0.45 ms (tables
// included).
template <typename OutT, bool kF32, int FN, int MODE, int R>
__global__ __launch_bounds__(kTabThreads, 4) void k_matern_tab(const double* __restrict__ lx, const double* __restrict__ ly,
                                                           TabArgs A, char* table, OutT* out)
{
    constexpr int kSlots = TabShape<kF32>::kPlanes * TabShape<kF32>::kN;
    constexpr unsigned kWaves = kTabWaves;
    __shared__ tab2_t sT[kSlots];
    __shared__ unsigned s_flag;
    __shared__ TailWalk s_walk[kWaves];     // not in registers, which the first part's loop would hold too
    unsigned* const counts = tab_counts<kF32>(table);
    for (int k = threadIdx.x; k < kSlots; k += kTabThreads) sT[k] = ((const tab2_t*)table)[k];
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&counts[0], 1u);
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grid = gridDim.x;
    const TileGeom& g = A.g;
    const unsigned rbn = (unsigned)g.rb_per_tile;
    unsigned it = blockIdx.x * kWaves + wave, stride = grid * kWaves;
    const unsigned per_tile = rbn * (unsigned)g.cb_per_tile;
    int64_t lo = 0, hi = A.first, I = 0, J = 0;
    // part by part; one copy of the item's code
    for (int part = 0;; ++part) {
        for (;; it += stride) {
            int64_t jl0;
            unsigned rb;
            if (part == 0) {
                if (it >= A.items) break;
                const unsigned t = it / per_tile, local = it - t * per_tile, cb = local / rbn;
                tile_of(t, g, I, J);
                rb = local - cb * rbn;
                jl0 = (int64_t)cb * A.cols;
            } else {
                // the tile of item `it`, from column w.col of tile (w.I, w.J) on, whose first item
                // is w.base. The tiles of a column have equally many items (all but the part's
                // first), so the walk is over columns (tile by tile it took 0.4 us a tile: 470
                // sites in 4-tiles 266 us)
                TailWalk w = s_walk[wave];
                unsigned rel;
                while (w.J < g.T) {
                    const int nJ = (int)min((int64_t)g.ts, g.n - (int64_t)w.J * g.ts);
                    const unsigned ntile = (unsigned)((nJ - w.col + kTailCols - 1) / kTailCols) * rbn;
                    rel = it - w.base;
                    if (rel < ntile) break;
                    const unsigned k = w.col > 0 ? 1u : min(rel / ntile, (unsigned)(g.T - w.I));
                    w.base += k * ntile;
                    w.col = 0;
                    w.I += (int)k;
                    if (w.I == g.T) {
                        ++w.J;
                        w.I = g.lower ? w.J : 0;
                    }
                }
                if (w.J == g.T) break;
                s_walk[wave] = w;
                I = w.I;
                J = w.J;
                const unsigned cb = rel / rbn;
                rb = rel - cb * rbn;
                jl0 = w.col + (int64_t)cb * kTailCols;
            }
            tab_item<OutT, kF32, FN, MODE, R>(A, sT, lx, ly, out, I, J, (int64_t)rb * (64 * R), jl0,
                                              part == 0 ? A.cols : kTailCols, lo, hi);
        }
        if (part == 2) return;
        unsigned skipped = 0u;
        if (part == 0) {
            // the table's bytes, shared by the workgroups launched last if all have read
            // the table by now (looked up a few times, never waited for: a workgroup may
            // not have started); one that finds any missing leaves its share to the last
            const unsigned share = grid - 1u - blockIdx.x;
            if (share < kTailGroups) {
                if (threadIdx.x == 0) {
                    unsigned c = 0u;
                    for (int k = 0; k < 4 && c != grid; ++k) c = atomicAdd(&counts[0], 0u);
                    s_flag = c == grid ? 1u : 0u;
                }
                __syncthreads();
                skipped = s_flag ? 0u : 1u << 16;
                if (!skipped) {
                    it = share * kWaves + wave;
                    stride = min(grid, kTailGroups) * kWaves;
                    s_walk[wave] = {A.first_at, 0u};
                    lo = A.first;
                    hi = A.count;
                    continue;
                }
            }
            ++part;
        }
        // the workgroup that finishes last: the counts' elements, and shares left to it
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned c = atomicAdd(&counts[1], 1u + skipped) + 1u + skipped;
            s_flag = (c & 0xffffu) == grid ? c : 0u;
        }
        __syncthreads();
        if (!s_flag) return;
        const bool left = (s_flag >> 16) != 0u;
        it = wave;
        stride = kWaves;
        s_walk[wave] = {left ? A.first_at : A.count_at, 0u};
        lo = left ? A.first : A.count;
        hi = INT64_MAX;
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
    const int64_t items = (lower_only ? T * (T + 1) / 2 : T * T) * ((ts + 63) / 64) * ((ts + 1) / 2);
    if (T >= 60000 || items >= (1LL << 31)) return false;
    return bk_matern_out_elems(n, tile_size, lower_only) >= min_entries;
}

// The packed tile that holds element e, and e's column in it.
static TailStart tail_start(const TileGeom& g, int64_t e)
{
    const int64_t T = g.T, ts = g.ts;
    int64_t lo = 0, hi = T - 1;                       // last column of tiles that starts at or before e
    while (lo < hi) {
        const int64_t m = (lo + hi + 1) / 2;
        if (tile_offset(g.n, ts, T, g.lower, g.lower ? m : 0, m) <= e) lo = m;
        else hi = m - 1;
    }
    const int64_t J = lo, I0 = g.lower ? J : 0, nJ = J == T - 1 ? g.n - J * ts : ts;
    const int64_t k = (e - tile_offset(g.n, ts, T, g.lower, I0, J)) / (nJ * ts), I = I0 + k < T ? I0 + k : T - 1;
    const int64_t mI = I == T - 1 ? g.n - I * ts : ts;
    return {(int32_t)I, (int32_t)J, (int32_t)((e - tile_offset(g.n, ts, T, g.lower, I, J)) / mI)};
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
    A.count = ((char*)tab_counts<kF32>(table) - (char*)out) / (int64_t)sizeof(OutT);
    A.first_at = tail_start(A.g, A.first);
    A.count_at = tail_start(A.g, A.count);
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

TabIndex tab_index(double beta, const TabParams& P, bool f32_table)
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
    // most entries of a short range are past the table: at no cost where they are 0 (25e6
    // at a mean z of 260: mixed 45 us, each by the quadrature 1,280)
    X.end = f32_table && P.zero <= kTabFar ? 0.0f : __builtin_nanf("");
    return X;
}

static TabNear tab_near_params(const TabParams& P)
{
    TabNear N = {P.inv_beta, P.sigma2, P.nu, 0.0, 0.0};
    const long double e = (long double)P.nu - 1.0L;
    if (P.nu >= 1.9) return N;
    if (fabsl(e) < 1e-4L) {            // ln H = (2 gamma - 1) e + e^2 / 2 + (2 zeta(3) - 1) / 3 e^3 + ...
        const long double h3 = 0.46803793543952952L;
        N.q0 = (double)(0.15443132980306573L + e * (0.5L + h3 * e));
        N.q1 = (double)(0.5L + 2.0L * h3 * e);
    } else {
        const long double h = logl(tgammal(1.0L - e) / tgammal(2.0L + e));
        N.q0 = (double)(h / e);
        N.q1 = (double)((-(digamma_host((double)(1.0L - e)) + digamma_host((double)(2.0L + e))) * e - h) / (e * e));
    }
    return N;
}

int launch_table_eval(const bk_locs* locs, const TabParams& P, const TabIndex& X, int32_t tile_size, int32_t lower_only, int fn,
                      bool f32_table, int out_dtype, void* out, hipStream_t stream)
{
    TabArgs A = {};
    A.P = P;
    const int64_t n = locs->n;
    const int elem = out_dtype == BK_OUT_F32 ? 4 : 8;
    char* table = table_in_output(out, bk_matern_out_elems(n, tile_size, lower_only), elem, f32_table, &A.first);
    A.g.n = n;
    A.g.ts = (int32_t)(tile_size < n ? tile_size : n);
    A.g.T = (int32_t)((n + A.g.ts - 1) / A.g.ts);
    A.g.lower = lower_only ? 1 : 0;
    A.X = X;
    if (fn == TAB_DNU) {
        A.N = tab_near_params(P);
        A.near = kTabNear / P.inv_beta * (kTabNear / P.inv_beta);
        A.near_end = kTabNearEnd / P.inv_beta * (kTabNearEnd / P.inv_beta);
    }
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

TabParams tab_params(const bk_params* prm, bool grad, double psi)
{
    TabParams P = {prm->sigma2, 1.0 / prm->beta, prm->nu, (1.0 - prm->nu) * kLn2 - lgamma(prm->nu), psi,
                   (double)((long double)prm->sigma2 * exp2l(1.0L - prm->nu) / tgammal(prm->nu)), kTabFar};
    // cosh t >= 1 + t^2 / 2 under the integrals: K_a(z) <= sqrt(pi / 2z) e^(a^2 / 2z - z), and
    // |dK_a/da| at most a / z of that. In z^nu K_nu both fall with z from kTabFar on (nu <= 16).
    const double a = grad && P.nu < 1.0 ? 1.0 : P.nu;
    const double tiny = (prm->out_dtype == BK_OUT_F32 ? -150.0 : -1075.0) * kLn2 - 0.5;
    for (; P.zero < 4000.0; P.zero += 1.0) {
        const double z = P.zero, lz = log(z);
        double b = log(P.scale) + (P.nu - 0.5) * lz - z + 0.5 * a * a / z + 0.2258;
        if (grad) b += fmax(lz + log(P.inv_beta), log(lz + kLn2 + fabs(psi) + a));
        if (b < tiny) break;
    }
    return P;
}

int matern_table_tiles(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only, void* out,
                       hipStream_t stream)
{
    const bool f32_table = prm->mode == BK_MIXED_F32C;
    const TabParams P = tab_params(prm, false, 0.0);
    const TabIndex X = tab_index(prm->beta, P, f32_table);
    int64_t first;
    char* table = table_in_output(out, bk_matern_out_elems(locs->n, tile_size, lower_only),
                                  prm->out_dtype == BK_OUT_F32 ? 4 : 8, f32_table, &first);
    int st = f32_table ? launch(k_tab_build<true, false>, dim3(TabWave<true>::kBlocks), dim3(64 * kTabLanes), stream, P, X, table,
                                nullptr, nullptr)
                       : launch(k_tab_build<false, false>, dim3(TabWave<false>::kBlocks), dim3(64 * kTabLanes), stream, P, X, table,
                                nullptr, nullptr);
    if (st != BK_OK) return st;
    if (mark_kernel_event(prm, 0, stream) != hipSuccess) return BK_EHIP;
    st = launch_table_eval(locs, P, X, tile_size, lower_only, TAB_C, f32_table, prm->out_dtype, out, stream);
    if (st != BK_OK) return st;
    return mark_kernel_event(prm, 1, stream) == hipSuccess ? BK_OK : BK_EHIP;
}

int matern_grad_table_tiles(const bk_locs* locs, const bk_params* prm, double psi, int32_t tile_size,
                            int32_t lower_only, void* const outs[3], hipStream_t stream)
{
    const TabParams P = tab_params(prm, true, psi);
    const TabIndex X = tab_index(prm->beta, P, false);
    const int64_t elems = bk_matern_out_elems(locs->n, tile_size, lower_only);
    const int elem = prm->out_dtype == BK_OUT_F32 ? 4 : 8;
    char* tab[3];
    int64_t first;
    for (int k = 0; k < 3; ++k) tab[k] = outs[k] ? table_in_output(outs[k], elems, elem, false, &first) : nullptr;
    int st = launch(k_tab_build<false, true>, dim3(TabWave<false>::kBlocks, 3), dim3(64 * kTabLanes), stream, P,
                    X, tab[0], tab[1], tab[2]);
    for (int k = 0; k < 3 && st == BK_OK; ++k)
        if (outs[k])
            st = launch_table_eval(locs, P, X, tile_size, lower_only, k, false, prm->out_dtype, outs[k], stream);
    return st;
}

}  // namespace bk
