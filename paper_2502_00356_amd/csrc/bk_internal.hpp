// bk_internal.hpp - declarations shared between the translation units of libbesselk.
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

#include <tuple>
#include <utility>

#include "../../include/besselk.h"
#include "bk_math.hpp"

namespace bk {

// Default thresholds. Plain: L = 36 ~ -ln(2^-52) (Sec. IV-B takes the window at
// machine epsilon), node target e^-35. Mixed and learned: L = 15, node target
// e^-14.5; the quadrature error is then ~2.5e-7 at most over nu in [0.01, 10],
// x in [1e-4, 1e3], leaving the rest of a 2e-6 relative budget to the FP32
// rounding of the node terms.
constexpr double kDefaultLPlain = 36.0;
constexpr double kDefaultLqPlain = 35.0;
constexpr double kDefaultLMixed = 15.0;
constexpr double kDefaultLqMixed = 14.5;

// The paper's refined algorithm: b = 40 bins on [0, 9] for x >= 0.1, Temme's
// series below (Sec. IV-C, Alg. 2).
constexpr int kPaperBins = 40;
constexpr double kPaperT = 9.0;
constexpr double kPaperTemmeX = 0.1;

void resolve_thresholds(int mode, double L_in, double Lq_in, double* L, double* Lq);

// Records the caller's kernel_events[k] on stream when both events are set
// (hipSuccess otherwise).
inline hipError_t mark_kernel_event(const bk_params* p, int k, hipStream_t stream)
{
    if (!p->kernel_events[0] || !p->kernel_events[1]) return hipSuccess;
    return hipEventRecord((hipEvent_t)p->kernel_events[k], stream);
}

template <typename... P, size_t... I>
inline int launch_args(void (*k)(P...), dim3 grid, dim3 block, hipStream_t stream, std::tuple<P...>& args,
                       std::index_sequence<I...>)
{
    void* ptrs[] = {static_cast<void*>(&std::get<I>(args))...};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), grid, block, ptrs, 0, stream) == hipSuccess ? BK_OK
                                                                                                       : BK_EHIP;
}

// Enqueues kernel k on stream, its arguments converted to the kernel's parameter
// types. The status is the launch's own (BK_OK or BK_EHIP): no error state left by
// other code is read or cleared.
template <typename... P, typename... A>
inline int launch(void (*k)(P...), dim3 grid, dim3 block, hipStream_t stream, A&&... a)
{
    static_assert(sizeof...(P) == sizeof...(A), "kernel argument count");
    std::tuple<P...> args(std::forward<A>(a)...);
    return launch_args(k, grid, block, stream, args, std::index_sequence_for<P...>{});
}

// Largest per-lane value over a wave (every lane active).
__device__ inline unsigned int wave_max_u32(unsigned int v)
{
    for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned int)__shfl_xor((int)v, o, 64));
    return v;
}

// Tiling of a Matern call: T x T tiles (or the lower ones) of ts rows and columns,
// each cut into rb_per_tile row blocks of 64 and cb_per_tile column blocks (four waves of
// `cols` columns where the per-entry kernels of bk_kernels.hip take it).
struct TileGeom {
    int64_t n;
    int32_t ts, T, lower;
    int32_t rb_per_tile, cb_per_tile, cols;
};

// Element offset of tile (I, J) in the packed output.
__host__ __device__ inline int64_t tile_offset(int64_t n, int64_t ts, int64_t T, int lower, int64_t I, int64_t J)
{
    int64_t nJ = (J == T - 1) ? n - J * ts : ts;
    if (lower) return ts * (J * n - ts * (J * (J - 1) / 2)) + nJ * (I - J) * ts;
    return J * ts * n + nJ * I * ts;
}

// Tile (I, J) of packed tile p (tiles column by column). Lower: column J starts at
// s(J) = J T - J (J - 1) / 2; the FP32 root of s(J) = p lands within a step or two of
// J (values below 2^34 at ~6e-8 relative; the cancellation in b^2 - 8 p adds a few
// steps only for T in the tens of thousands), and the loops settle it exactly. The
// work is uniform across the wave: scalar integer loops after a handful of FP32
// vector instructions.
__device__ inline void tile_of(int64_t p, const TileGeom& g, int64_t& I, int64_t& J)
{
    int64_t T = g.T;
    if (!g.lower) { J = p / T; I = p - J * T; return; }
    const float b = 2.0f * (float)T + 1.0f;
    int64_t j = (int64_t)((b - __builtin_amdgcn_sqrtf(fmaxf(fmaf(b, b, -8.0f * (float)p), 0.0f))) * 0.5f);
    if (j < 0) j = 0;
    if (j > T - 1) j = T - 1;
    while (j > 0 && j * T - j * (j - 1) / 2 > p) --j;
    while (j + 1 <= T - 1 && (j + 1) * T - (j + 1) * j / 2 <= p) ++j;
    J = j;
    I = J + (p - (J * T - J * (J - 1) / 2));
}

// z for the plain sums of the per-entry kernels: past 1e306 their exponents leave exp_node's
// range, and at a finite z past 1e300 the prefactor is 0 whatever the sum.
__device__ __forceinline__ double sum_z(double z) { return z > 1e300 && z < __builtin_inf() ? 1e300 : z; }

// One entry of the plain (MODE BK_PLAIN_F64) or mixed form at z = r / beta > 0:
// sigma2 c z^nu K_nu(z), pref = ln c = ln(2^(1-nu) / Gamma(nu)). s: the entry's solve
// (for the caller's counts and for dC/dnu). T: exp_tab's tables.
template <int MODE>
__device__ __forceinline__ double matern_entry(double nu, double z, double lz, double sigma2, double pref, double L,
                                               double Lq, const double* T, Solved& s)
{
    double hs;
    if constexpr (MODE == BK_PLAIN_F64) {
        const double zs = sum_z(z);
        s = plain_plan(nu, zs, L, Lq, rule_tab(), T);
        hs = s.p.h * sum_f64<true>(nu, zs, s.p, s.E, s.Ei, s.Sr, T);
        hs = fma(hs, s.dlo, hs);
    } else {
        s = plain_solve(nu, z, L, Lq, rule_tab(), T);
        hs = s.p.h * sum_mixed(nu, z, s.p, s.A, T);
    }
    return sigma2 * exp(pref + nu * lz + (s.delta - z)) * hs;
}

// dC/dbeta = sigma2 c z^(nu+1) K_{nu-1}(z) / beta at z > 0 (lz = ln z).
__device__ __forceinline__ double matern_dbeta(double nu, double z, double lz, double sigma2, double inv_beta,
                                               double pref, double L, double Lq, const double* T)
{
    const double nu1 = fabs(nu - 1.0), zs = sum_z(z);
    const Solved s1 = plain_plan(nu1, zs, L, Lq, rule_tab(), T);
    const double hs1 = s1.p.h * sum_f64<true>(nu1, zs, s1.p, s1.E, s1.Ei, s1.Sr, T);
    return sigma2 * inv_beta * exp(pref + (nu + 1.0) * lz + (s1.delta - z)) * fma(hs1, s1.dlo, hs1);
}

// dC/dnu = C (ln z - ln 2 - psi(nu)) + sigma2 c z^nu dK_nu/dnu(z) at z > 0, from C = vc
// and the start t0 of its window.
__device__ __forceinline__ double matern_dnu(double nu, double z, double lz, double sigma2, double pref, double psi,
                                             double L, double Lq, const double* T, double vc, double t0)
{
    double delta, hs;
    dnu_integral(nu, z, t0, L, Lq, rule_tab(), T, delta, hs);
    return vc * (lz - kLn2 - psi) + sigma2 * exp(pref + nu * lz + (delta - z)) * hs;
}

// psi(v), v > 0, on the host.
double digamma_host(double v);
int bk_besselk_learned(const double* nu, const double* x, double* out, int64_t n, const bk_params* prm,
                       double L, double Lq, hipStream_t stream);
// Workspace bytes of the learned Matern form for one call (window table, interval
// plans, wave bitmap); 0 if the sizes are invalid.
size_t matern_learned_workspace_bytes(int64_t n, int32_t tile_size, int32_t lower_only);
int bk_matern_learned(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only,
                      void* out, double L, double Lq, void* workspace, size_t workspace_bytes, hipStream_t stream);
// bk_matern_tiles with the learned form's workspace given explicitly (the caller's,
// or the no-allocation entry point's static scratch).
int matern_tiles_dispatch(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only,
                          void* out, void* workspace, size_t workspace_bytes, hipStream_t stream);

}  // namespace bk
