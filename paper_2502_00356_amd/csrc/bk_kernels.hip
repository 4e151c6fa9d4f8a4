// bk_kernels.hip - HIP kernels and C ABI for standalone K_nu(x), the window
// export, tiled Matern covariance generation (arXiv 2502.00356, Sec. IV-B,
// Sec. III-A, Alg. 3), the paper's refined algorithm (Sec. IV-A, IV-C, Alg. 2),
// and the derivatives of K_nu and of the Matern covariance, for gfx950.
//
// Mapping: one lane per output entry. Standalone K_nu and its derivatives: workgroups of 64 to
// 1,024 entries, sorted through LDS (coalesced FP64 loads, stores to each entry's own index);
// the other kernels: 256-lane workgroups.
// Matern: each wave covers 64 consecutive rows of a tile column (one 512-byte
// FP64 or 256-byte FP32 store per column); the row location lives in VGPRs and
// the column location is wave-uniform, so it is read through scalar loads
// instead of being staged in LDS.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "../../include/besselk.h"
#include "bk_math.hpp"
#include "bk_internal.hpp"
#include "bk_table.hpp"

namespace bk {

void resolve_thresholds(int mode, double L_in, double Lq_in, double* L, double* Lq)
{
    bool plain = (mode == BK_PLAIN_F64);
    *L = L_in > 0.0 ? L_in : (plain ? kDefaultLPlain : kDefaultLMixed);
    *Lq = Lq_in > 0.0 ? Lq_in : (plain ? kDefaultLqPlain : kDefaultLqMixed);
}

// Sum of a per-lane value over a workgroup of nw wave64s (nw <= 16), added once to
// a global counter.
__device__ void block_count_w(unsigned long long* dst, unsigned long long v, int nw)
{
    __shared__ unsigned long long red[16];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wid] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < nw; ++w) t += red[w];
        atomicAdd(dst, t);
    }
}

// Special values shared by every form; returns true if handled.
__device__ __forceinline__ bool special_value(double v, double z, int result, double& r)
{
    if (isnan(v) || isnan(z) || z < 0.0) { r = __builtin_nan(""); return true; }
    if (z == 0.0 || isinf(v)) { r = __builtin_inf(); return true; }
    if (isinf(z)) { r = (result == BK_RESULT_LOG) ? -__builtin_inf() : 0.0; return true; }
    return false;
}

// Final assembly from exp(-x) exp(Delta) h S (see bk_math.hpp).
__device__ __forceinline__ double assemble(double z, double delta, double hs, int result, const double* T)
{
    if (result == BK_RESULT_SCALED && fabs(delta) < 700.0) return exp_wide(delta, T) * hs;
    if (result == BK_RESULT_SCALED) return exp(delta) * hs;
    if (result == BK_RESULT_LOG) return (delta - z) + log(hs);
    const double d = delta - z;
    if (fabs(d) < 700.0) {
        // e^d is a normal number; its argument's rounding is carried before hs, whose product may overflow
        const double v = exp_wide(d, T);
        return fma(v, two_sum_err(delta, -z, d), v) * hs;
    }
    if (z < 708.0) return exp(-z) * exp(delta) * hs;
    // subnormal range: e^(-z) formed 2^64 larger, product scaled back (one rounding)
    return ldexp(exp(64.0 * kLn2 - z) * exp(delta) * hs, -64);
}

// The plain and mixed forms take Temme's series with the forward recurrence (Sec. IV-A; the
// paper's branch for x < 0.1 in Alg. 2) where x < 0.1 and K_nu(x) stays far inside
// the double range: log K_nu(x) <= log Gamma(nu) + nu log(2/x) for x < 0.1, bounded
// here by nu (log(2/x) + log(nu + 1)) + log(1/nu + 1) < 600. On 2^24 pairs with
// x in [1e-4, 0.1) it is 3.7 times faster than the windowed FP64 quadrature and as
// accurate (max relative error 3.0e-15 against 6.4e-15); it also takes 10% off the
// FP32-term form on the 2^24 grid, at FP64 accuracy for those entries.
__device__ __forceinline__ bool temme_applies(double v, double z)
{
    if (!(z < kPaperTemmeX) || !(v > 0.0)) return false;
    if (z >= 1e-10 && v <= 20.0 && v >= 1e-20) return true;      // the bound below is at most 536 there
    const float vf = (float)v;
    const float lb = vf * (__logf(2.0f / (float)z) + __logf(vf + 1.0f)) + __logf(1.0f / vf + 1.0f);
    return lb < 600.0f;
}

// K_nu(z) by Temme's series, as the requested result (K, e^z K or log K).
__device__ __forceinline__ double temme_result(double v, double z, int result, const double* T)
{
    const double k = temme_k(v, z, temme_tab(), T);
    if (result == BK_RESULT_SCALED) return k * exp(z);
    if (result == BK_RESULT_LOG) return log(k);
    return k;
}

// Counting sort of a block's lanes by a small key (0..63): returns the lane's slot
// in key order. Equal keys keep no particular order; results do not depend on it,
// since every entry is computed by one lane from its own inputs.
template <int NB>
__device__ unsigned int block_sort_slot(int key, unsigned int* hist)
{
    const int tid = threadIdx.x;
    if (tid < 64) hist[tid] = 0u;
    __syncthreads();
    const unsigned int rank = atomicAdd(&hist[key], 1u);
    __syncthreads();
    if (tid < 64) {
        const unsigned int h = hist[tid];
        hist[tid] = wave_incl_scan(h) - h;
    }
    __syncthreads();
    const unsigned int slot = hist[key] + rank;
    __syncthreads();   // hist may be reused by the caller after this
    return slot;
}

// Mixed K_nu. A block of kSolveBlock entries is processed in three
// phases, with the lanes re-sorted between them through LDS so that each wave
// holds entries that take the same branches and loop counts:
//  1. entry order: special values; key = peak regime (0: nu^2 <= x, t* = 0;
//     1: interior peak, window from t = 0; 2: interior peak with a left root
//     likely, estimated by nu asinh(nu/x) > L; 4: x < 0.1, Temme's series);
//  2. regime order: Temme's series (and its store), or the FP64 peak / window
//     solve and node count;
//  3. node-count order: the node walk, the prefactor and the store to the
//     entry's own index.
constexpr int kSolveBlock = 512;

__global__ __launch_bounds__(kSolveBlock) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_besselk_mixed(const double* __restrict__ nu,
                                                         const double* __restrict__ x,
                                                         double* __restrict__ out, int64_t n, int result,
                                                         double L, double Lq, 
                                                         unsigned long long* __restrict__ stats)
{
    __shared__ unsigned int hist[64];
    __shared__ double s_tab[kTabLen];
    // staged per entry between phases: v, z, t_ref, h, Delta, t0, x cosh(t_ref) / 2
    __shared__ double s_d[7][kSolveBlock];
    __shared__ int s_i[3][kSolveBlock];
    const int tid = threadIdx.x;
    if (tid < kTabLen) s_tab[tid] = rule_tab().tab[tid];   // read after the sorts' barriers
    const int64_t i = (int64_t)blockIdx.x * kSolveBlock + tid;
    double v = 0.0, z = 1.0;
    bool work = false;
    if (i < n) {
        v = fabs(nu[i]);
        z = x[i];
        double r;
        if (special_value(v, z, result, r)) out[i] = r;
        else work = true;
    }
    int key = 0;
    if (work && v * v > z) key = ((float)v * asinhf((float)(v / z)) > (float)L) ? 2 : 1;
    if (work && temme_applies(v, z)) key = 4;
    // phase 1 -> 2: sort by regime (Temme's series in waves of their own)
    unsigned int slot = block_sort_slot<kSolveBlock>(work ? key : 3, hist);
    s_d[0][slot] = v;
    s_d[1][slot] = z;
    s_i[0][slot] = work ? (int)(i - (int64_t)blockIdx.x * kSolveBlock) : -1;
    s_i[1][slot] = key;
    __syncthreads();
    int li = s_i[0][tid];
    const double v2 = s_d[0][tid], z2 = s_d[1][tid];
    const bool temme = li >= 0 && s_i[1][tid] == 4;
    __syncthreads();
    Solved sv;
    sv.p.N = -1;
    if (temme) {
        out[(int64_t)blockIdx.x * kSolveBlock + li] = temme_result(v2, z2, result, s_tab);
        li = -1;
    } else if (li >= 0) {
        sv = plain_solve(v2, z2, L, Lq, rule_tab(), s_tab);
    }
    // phase 2 -> 3: sort by node count
    const int nkey = li < 0 ? 0 : (sv.p.N < 63 ? sv.p.N : 63);
    slot = block_sort_slot<kSolveBlock>(nkey, hist);
    s_d[0][slot] = v2;
    s_d[1][slot] = z2;
    s_d[2][slot] = sv.p.tref;
    s_d[3][slot] = sv.p.h;
    s_d[4][slot] = sv.delta;
    s_d[5][slot] = sv.p.t0;
    s_d[6][slot] = sv.A;
    s_i[0][slot] = li;
    s_i[1][slot] = sv.p.N;
    s_i[2][slot] = sv.p.mc;
    __syncthreads();
    const int l3 = s_i[0][tid];
    unsigned long long nodes = 0, ents = 0;
    if (l3 >= 0) {
        const double v3 = s_d[0][tid], z3 = s_d[1][tid];
        Plan p;
        p.tref = s_d[2][tid];
        p.h = s_d[3][tid];
        p.N = s_i[1][tid];
        p.mc = s_i[2][tid];
        p.t0 = s_d[5][tid];
        const double hs = p.h * sum_mixed(v3, z3, p, s_d[6][tid], s_tab);
        out[(int64_t)blockIdx.x * kSolveBlock + l3] = assemble(z3, s_d[4][tid], hs, result, s_tab);
        nodes = (unsigned long long)(p.N + 1);
        ents = 1;
    }
    if (stats) {
        block_count_w(stats + BK_STAT_NODES, nodes, kSolveBlock / 64);
        block_count_w(stats + BK_STAT_ENTRIES, ents, kSolveBlock / 64);
        const unsigned int wmax = wave_max_u32((unsigned int)nodes);
        block_count_w(stats + BK_STAT_LANE_SLOTS, (threadIdx.x & 63) == 0 ? 64ull * wmax : 0ull, kSolveBlock / 64);
    }
}

// The entries of a workgroup, sorted by key in LDS: kThreads lanes place kPer each, and the
// workgroup's waves then draw them 64 at a time. Equal keys keep no particular order;
// results do not depend on it, since every entry is computed by one lane from its own inputs.
constexpr unsigned kEntryTemme = 1023u, kEntryExact = 1022u;      // in place of a node count

template <int kThreads, int kPer>
struct DrawBlock {
    static constexpr int kEntries = kThreads * kPer;
    static_assert(kEntries <= 1024, "entry index bits");
    unsigned int hist[64], next;
    double v[kEntries], z[kEntries];
    float t0[kEntries], t1[kEntries];
    unsigned int e[kEntries];        // entry | mc << 10 | N << 20 (N <= 512; 0: none)

    __device__ __forceinline__ void begin()
    {
        if (threadIdx.x < 64) hist[threadIdx.x] = 0u;
        if (threadIdx.x == 0) next = 0u;
        __syncthreads();
    }

    // Largest node counts first, then the series; entries with nothing to do last.
    static __device__ __forceinline__ int key_of(unsigned int N, double nu)
    {
        return N == kEntryTemme ? (nu < 4.5 ? 62 : 61) : (N == 0u ? 63 : 60 - (int)min(N, 60u));
    }

    __device__ __forceinline__ void place(const double (&pv)[kPer], const double (&pz)[kPer], const float (&p0)[kPer],
                                          const float (&p1)[kPer], const unsigned int (&pe)[kPer],
                                          const int (&key)[kPer], const unsigned int (&rank)[kPer])
    {
        __syncthreads();
        if (threadIdx.x < 64) {
            const unsigned int h = hist[threadIdx.x];
            hist[threadIdx.x] = wave_incl_scan(h) - h;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const unsigned int slot = hist[key[k]] + rank[k];
            v[slot] = pv[k];
            z[slot] = pz[k];
            t0[slot] = p0[k];
            t1[slot] = p1[k];
            e[slot] = pe[k];
        }
        __syncthreads();
    }

    // An entry's rank among those of its key (taken as soon as its key is known).
    __device__ __forceinline__ unsigned int rank(int key) { return atomicAdd(&hist[key], 1u); }

    // The wave's next 64 entries: their first slot, or -1.
    __device__ __forceinline__ int draw()
    {
        unsigned int c = 0u;
        if ((threadIdx.x & 63) == 0) c = atomicAdd(&next, 1u);
        c = __builtin_amdgcn_readfirstlane(c);
        return c < (unsigned)(kEntries / 64) ? (int)(c * 64u) : -1;
    }
};

// Per-lane sums of a kernel that draws entries, for the statistics.
struct DrawCounts {
    unsigned int nodes = 0u, ents = 0u, slots = 0u;

    __device__ __forceinline__ void add(unsigned int walked)      // every lane of the wave
    {
        nodes += walked;
        ents += walked ? 1u : 0u;
        const unsigned int w = wave_max_u32(walked);
        slots += (threadIdx.x & 63) == 0 ? 64u * w : 0u;
    }
    __device__ __forceinline__ void store(unsigned long long* stats, int waves) const
    {
        block_count_w(stats + BK_STAT_NODES, nodes, waves);
        block_count_w(stats + BK_STAT_ENTRIES, ents, waves);
        block_count_w(stats + BK_STAT_LANE_SLOTS, slots, waves);
    }
};

// Plain K_nu. A workgroup takes kThreads x kPer entries in two phases:
//  1. entry order: special values; the FP32 window and node count (cheap enough to run
//     before any sort), or Temme's series (x < 0.1), or plain_plan (plan_fast_ok false: the
//     window for a walk by products, or the exact solve) as keys of their own; counting sort
//     into LDS, largest node counts first;
//  2. its waves draw the sorted entries 64 at a time: set-up at the reference node, the
//     paired walk, the prefactor and the store to the entry's own index; or the whole of
//     the other two.
// VALU-bound. 2^24 pairs of the (nu, x) grid: 1,264 us with the exact solve between two
// sorts (2,266 VALU instructions a wave of 64), 755 with the FP32 window there, 640 with
// one sort of 512 entries, one a lane (1,207 instructions), 463 with 1,024 drawn by four
// waves: fewer waves hold both branches, and none waits for a block's slowest; 450 with the
// nodes' exponents by second differences (CoshPair), 431 with one Newton step an end and the
// step rule's cosine by its series. (512
// entries in 128 lanes 528, in 256 489; constants hoisted out of the draw loop spill: 548.)
template <int kThreads, int kPer>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_besselk_plain(
    const double* __restrict__ nu, const double* __restrict__ x, double* __restrict__ out, int64_t n, int result,
    double L, double Lq, unsigned long long* __restrict__ stats)
{
    __shared__ double s_tab[kTabLen];
    __shared__ DrawBlock<kThreads, kPer> B;
    const int tid = threadIdx.x;
    for (int j = tid; j < kTabLen; j += kThreads) s_tab[j] = rule_tab().tab[j];   // read after the barriers
    B.begin();
    const int64_t i0 = (int64_t)blockIdx.x * B.kEntries;
    double v[kPer], z[kPer];
    float t0[kPer], t1[kPer];
    unsigned int e[kPer], rank[kPer];
    int key[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = i0 + k * kThreads + tid;
        unsigned int N = 0u, mc = 0u;
        v[k] = 0.0;
        z[k] = 1.0;
        t0[k] = t1[k] = 0.0f;
        if (i < n) {
            v[k] = fabs(nu[i]);
            z[k] = x[i];
            double r;
            if (special_value(v[k], z[k], result, r)) out[i] = r;
            else if (temme_applies(v[k], z[k])) N = kEntryTemme;
            else if (!plan_fast_ok(v[k], z[k], L, Lq)) N = kEntryExact;
            else window_count(v[k], z[k], L, Lq, t0[k], t1[k], N, mc);
        }
        e[k] = (unsigned int)(k * kThreads + tid) | (mc << 10) | (N << 20);
        key[k] = B.key_of(N, v[k]);
        rank[k] = B.rank(key[k]);
    }
    B.place(v, z, t0, t1, e, key, rank);
    DrawCounts cnt;
    for (int c = B.draw(); c >= 0; c = B.draw()) {
        const int j = c + (tid & 63);
        const unsigned int ej = B.e[j], N = ej >> 20;
        unsigned int walked = 0u;
        if (N != 0u) {
            const double vj = B.v[j], zj = B.z[j];
            double r;
            if (N == kEntryTemme) {
                r = temme_result(vj, zj, result, s_tab);
            } else {
                Solved s;
                double hs;
                if (N == kEntryExact) {           // any x: the left side by products
                    s = plain_plan(vj, zj, L, Lq, rule_tab(), s_tab);
                    hs = s.p.h * sum_f64<true, true>(vj, zj, s.p, s.E, s.Ei, s.Sr, s_tab);
                } else {                          // x >= 0.1, or nu far above 1 (temme_applies)
                    s = plan_setup(vj, zj, B.t0[j], B.t1[j], N, (ej >> 10) & 1023u);
                    hs = s.p.h * sum_f64<false>(vj, zj, s.p, s.E, s.Ei, s.Sr, s_tab);
                }
                hs = fma(hs, s.dlo, hs);          // the low part of Delta
                r = assemble(zj, s.delta, hs, result, s_tab);
                walked = (unsigned int)(s.p.N + 1);
            }
            out[i0 + (ej & 1023u)] = r;
        }
        if (stats) cnt.add(walked);
    }
    if (stats) cnt.store(stats, kThreads / 64);
}

// The paper's refined algorithm (Alg. 2), one lane per entry, FP64: Temme's
// series with the forward recurrence for x < 0.1, the fixed-window sum otherwise.
__global__ __launch_bounds__(256) void k_besselk_paper(const double* __restrict__ nu, const double* __restrict__ x,
                                                       double* __restrict__ out, int64_t n, int result, int bins,
                                                       double T, 
                                                       
                                                       unsigned long long* __restrict__ stats)
{
    __shared__ double s_tab[kTabLen];
    stage_tab(s_tab);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned long long nodes = 0, ents = 0;
    if (i < n) {
        const double v = fabs(nu[i]), z = x[i];
        double r;
        if (!special_value(v, z, result, r)) {
            if (z < kPaperTemmeX) {
                // K directly; written as exp(-z) exp(0) (e^z K) for the shared assembly
                r = assemble(z, 0.0, temme_k(v, z, temme_tab(), s_tab) * exp(z), result, s_tab);
            } else {
                const FixedOut f = paper_fixed(v, z, bins, T, s_tab);
                // K = exp(lscale) h S, written through Delta = lscale + z so that the
                // shared assembly (exp(-z) exp(Delta) h S) applies
                r = assemble(z, f.lscale + z, f.hs, result, s_tab);
                nodes = (unsigned long long)(bins + 1);
                ents = 1;
            }
        }
        out[i] = r;
    }
    if (stats) {
        block_count_w(stats + BK_STAT_NODES, nodes, 4);
        block_count_w(stats + BK_STAT_ENTRIES, ents, 4);
    }
}

__global__ __launch_bounds__(256) void k_window(const double* __restrict__ nu,
                                                const double* __restrict__ x,
                                                double* __restrict__ tlo, double* __restrict__ thi,
                                                int32_t* __restrict__ nodes, int64_t n, double L,
                                                double Lq)
{
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double v = fabs(nu[i]), z = x[i];
    if (!(z > 0.0) || isinf(z) || isnan(v) || isinf(v)) {
        tlo[i] = __builtin_nan(""); thi[i] = __builtin_nan(""); nodes[i] = 0;
        return;
    }
    Solved s = plain_solve(v, z, L, Lq, rule_tab(), rule_tab().tab);
    tlo[i] = s.p.t0;
    thi[i] = s.t1;
    nodes[i] = s.p.N;
}

// e^x-scaled value s to the requested result (K or e^x K).
__device__ __forceinline__ double unscale(double z, double s, int result)
{
    if (result == BK_RESULT_SCALED) return s;
    if (z < 708.0) return exp(-z) * s;
    return ldexp(exp(64.0 * kLn2 - z) * s, -64);
}

// exp_tab's tables in LDS, for a kernel (which fills them) and its out-of-line function alike.
__device__ __forceinline__ double* lds_tab()
{
    __shared__ double t[kTabLen];
    return t;
}

// K, dK/dx and dK/dnu where the fast window does not apply: the K integral at orders nu and
// |nu - 1| (for dK/dx) and the dK/dnu integral, each with its own exact solve. Out of line and
// rare.
struct DerivOut {
    double k, dx, dn;
    unsigned int nodes;
};

__device__ __noinline__ DerivOut deriv_exact(double v, double z, double L, double Lq, int result, bool want_dx, bool want_dn)
{
    const RuleTable& R = rule_tab();
    const double* T = lds_tab();
    DerivOut o;
    const Solved s0 = plain_plan(v, z, L, Lq, R, T);
    double hs0 = s0.p.h * sum_f64<true, true>(v, z, s0.p, s0.E, s0.Ei, s0.Sr, T);
    hs0 = fma(hs0, s0.dlo, hs0);
    o.k = assemble(z, s0.delta, hs0, result, T);
    o.nodes = (unsigned int)(s0.p.N + 1);
    o.dx = o.dn = 0.0;
    if (want_dx) {
        const double v1 = fabs(v - 1.0);
        const Solved s1 = plain_plan(v1, z, L, Lq, R, T);
        double hs1 = s1.p.h * sum_f64<true, true>(v1, z, s1.p, s1.E, s1.Ei, s1.Sr, T);
        hs1 = fma(hs1, s1.dlo, hs1);
        // by assemble where K is in range: e^Delta need not be (nu = 1,000 at x = 500)
        if (result == BK_RESULT_K && fabs(s0.delta - z) < 700.0)
            o.dx = -fma(v / z, o.k, assemble(z, s1.delta, hs1, result, T));
        else
            o.dx = -unscale(z, exp(s1.delta) * hs1 + (v / z) * (exp(s0.delta) * hs0), result);
        o.nodes += (unsigned int)(s1.p.N + 1);
    }
    if (want_dn && v > 0.0) {
        const Solved sd = dnu_solve(v, z, s0.p.t0, L, Lq, R, T);
        o.dn = assemble(z, sd.delta, sd.p.h * sum_dnu_f64(v, sd.p, sd.A, sd.B, T), result, T);
        o.nodes += (unsigned int)(sd.p.N + 1);
    }
    return o;
}

// K_nu(x), dK/dx and dK/dnu, FP64, by one window and one walk for the three integrals
// (sum_deriv), the entries sorted and drawn as in k_besselk_plain. NULL outputs are not
// stored. dK/dnu carries the sign of nu. 2^22 pairs of the (nu, x) grid: 1,729 us with a
// solve and a walk for each integral, unsorted (1,205 with the FP32 windows
// there), 300 with one walk, 296 with its right side by second differences.
template <int kThreads, int kPer>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_besselk_deriv(
    const double* __restrict__ nu, const double* __restrict__ x, double* __restrict__ k, double* __restrict__ dkdx,
    double* __restrict__ dkdnu, int64_t n, int result, double L, double Lq, unsigned long long* __restrict__ stats)
{
    double* const s_tab = lds_tab();
    __shared__ DrawBlock<kThreads, kPer> B;
    const int tid = threadIdx.x;
    for (int j = tid; j < kTabLen; j += kThreads) s_tab[j] = rule_tab().tab[j];   // read after the barriers
    B.begin();
    const int64_t i0 = (int64_t)blockIdx.x * B.kEntries;
    auto store = [&](int64_t i, double rk, double rx, double rn) {
        if (k) k[i] = rk;
        if (dkdx) dkdx[i] = rx;
        if (dkdnu) dkdnu[i] = rn;
    };
    double v[kPer], z[kPer];
    float t0[kPer], t1[kPer];
    unsigned int e[kPer], rank[kPer];
    int key[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int64_t i = i0 + q * kThreads + tid;
        unsigned int N = 0u, mc = 0u;
        v[q] = 0.0;
        z[q] = 1.0;
        t0[q] = t1[q] = 0.0f;
        if (i < n) {
            const double nr = nu[i], av = fabs(nr);
            v[q] = nr;
            z[q] = x[i];
            if (isnan(nr) || isnan(z[q]) || z[q] < 0.0)
                store(i, __builtin_nan(""), __builtin_nan(""), __builtin_nan(""));
            else if (z[q] == 0.0 || isinf(av))
                store(i, __builtin_inf(), -__builtin_inf(), av == 0.0 ? 0.0 : copysign(__builtin_inf(), nr));
            else if (isinf(z[q]))
                store(i, 0.0, -0.0, copysign(0.0, nr));
            else if (!deriv_fast_ok(av, z[q], L, Lq) || !deriv_window_count(av, z[q], L, Lq, t0[q], t1[q], N, mc))
                N = kEntryExact;
        }
        e[q] = (unsigned int)(q * kThreads + tid) | (mc << 10) | (N << 20);
        key[q] = B.key_of(N, v[q]);
        rank[q] = B.rank(key[q]);
    }
    B.place(v, z, t0, t1, e, key, rank);
    DrawCounts cnt;
    for (int c = B.draw(); c >= 0; c = B.draw()) {
        const int j = c + (tid & 63);
        const unsigned int ej = B.e[j], N = ej >> 20;
        unsigned int walked = 0u;
        if (N != 0u) {
            const double nr = B.v[j], vj = fabs(nr), zj = B.z[j];
            double rk, rx, rn;
            if (N == kEntryExact) {
                const DerivOut o = deriv_exact(vj, zj, L, Lq, result, dkdx != nullptr, dkdnu != nullptr);
                rk = o.k;
                rx = o.dx;
                rn = o.dn;
                walked = o.nodes;
            } else {
                const Solved s = plan_setup(vj, zj, B.t0[j], B.t1[j], N, (ej >> 10) & 1023u);
                const DerivSums S = sum_deriv(vj, zj, s.p, s.E, s.Ei, s.Sr, s_tab);
                const double h = fma(s.p.h, s.dlo, s.p.h);      // with the low part of Delta
                rk = assemble(zj, s.delta, h * S.k, result, s_tab);
                // cosh t = cosh t_ref + (x (cosh t - cosh t_ref)) / x
                rx = -assemble(zj, s.delta, h * fma(0.5 * (s.E + s.Ei), S.k, S.x * recip(zj)), result, s_tab);
                rn = assemble(zj, s.delta, h * S.d, result, s_tab);
                walked = (unsigned int)(s.p.N + 1);
            }
            store(i0 + (ej & 1023u), rk, rx, copysign(vj > 0.0 ? rn : 0.0, nr));
        }
        if (stats) cnt.add(walked);
    }
    if (stats) cnt.store(stats, kThreads / 64);
}

// ---------------------------------------------------------------------------
// Matern tiles
// ---------------------------------------------------------------------------
constexpr int kRowsPerWave = 64;
// Columns a wave takes in turn: one in calls that then still leave the chip unfilled (every
// column a wave is one more entry in its serial chain), kMaxCols in larger ones, whose
// blocks stage the tables less often. Plain FP64, nu = 17: 600 sites 57 us with eight,
// 28 with one; 2,000 166 and 156; 2,800 319 and 318; 6,000 1,251 and 1,283. A counting call
// keeps eight: every workgroup adds to the same three counters (2,000 sites, plain, with
// statistics 268 us with eight, 600 with one).
constexpr int kMaxCols = 8;
static int cols_per_wave(int64_t entries) { return entries < 8000000 ? 1 : kMaxCols; }

// kStats: the statistics variant, which also counts the entries evaluated by
// quadrature and their nodes (lanes past a ragged tile's last row stay in the
// wave, idle, so that the wave can sum its counts).
template <int MODE, typename OutT, bool kStats>
__global__ __launch_bounds__(256, 4) void k_matern(const double* __restrict__ lx,
                                                const double* __restrict__ ly, TileGeom g,
                                                int64_t tile_base, double sigma2, double inv_beta,
                                                double nu, double pref, double L, double Lq,
                                                int bins, double T, OutT* __restrict__ out,
                                                unsigned long long* __restrict__ stats)
{
    __shared__ double s_tab[kTabLen];
    stage_tab(s_tab);                   // before any wave leaves
    // block -> (tile, row block, column block) in 32-bit arithmetic (a 64-bit
    // division is a long instruction sequence)
    const unsigned wg_per_tile = (unsigned)g.rb_per_tile * (unsigned)g.cb_per_tile;
    const unsigned tq = blockIdx.x / wg_per_tile, local = blockIdx.x - tq * wg_per_tile;
    const int64_t p = tile_base + (int64_t)tq;
    const int rb = (int)(local % (unsigned)g.rb_per_tile), cb = (int)(local / (unsigned)g.rb_per_tile);
    int64_t I, J;
    tile_of(p, g, I, J);
    const int64_t mI = min((int64_t)g.ts, g.n - I * g.ts);
    const int64_t nJ = min((int64_t)g.ts, g.n - J * g.ts);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t il = (int64_t)rb * kRowsPerWave + lane;
    const int64_t jl0 = ((int64_t)cb * 4 + wave) * g.cols;
    const bool row_ok = il < mI;
    // the statistics variant keeps every wave to the end for its block-wide sums
    if (!kStats && (jl0 >= nJ || !row_ok)) return;
    const int64_t base = tile_offset(g.n, g.ts, g.T, g.lower, I, J);
    const int64_t ilr = row_ok ? il : 0;
    const double xi = lx[I * g.ts + ilr], yi = ly[I * g.ts + ilr];
    const int cend = (kStats && (!row_ok || jl0 >= nJ)) ? 0 : (int)min((int64_t)g.cols, nJ - jl0);
    unsigned int c_ent = 0, c_nodes = 0;
    unsigned int col_nodes[kMaxCols] = {};      // statistics: nodes per column walked
    for (int c = 0; c < cend; ++c) {
        const int64_t jl = jl0 + c;
        const double xj = lx[J * g.ts + jl], yj = ly[J * g.ts + jl];
        const double dx = xj - xi, dy = yj - yi;
        const double r = sqrt(dx * dx + dy * dy);
        double val;
        if (r == 0.0) {
            val = sigma2;
        } else {
            const double z = r * inv_beta;
            if (MODE == BK_PAPER_REFINED) {
                if (z < kPaperTemmeX) {
                    val = sigma2 * exp(pref + nu * log(z)) * temme_k(nu, z, temme_tab(), s_tab);
                } else {
                    const FixedOut f = paper_fixed(nu, z, bins, T, s_tab);
                    val = sigma2 * exp(pref + nu * log(z) + f.lscale) * f.hs;
                    c_nodes += (unsigned int)(bins + 1);
                    c_ent += 1;
                    if (kStats) col_nodes[c] = (unsigned int)(bins + 1);
                }
            } else {
                Solved s;
                val = matern_entry<MODE>(nu, z, log(z), sigma2, pref, L, Lq, s_tab, s);
                c_nodes += (unsigned int)(s.p.N + 1);
                c_ent += 1;
                if (kStats) col_nodes[c] = (unsigned int)(s.p.N + 1);
            }
        }
        out[base + il + jl * mI] = (OutT)val;
    }
    if (kStats) {      // one atomic per counter per workgroup
        unsigned int slots = 0;
#pragma unroll
        for (int c = 0; c < kMaxCols; ++c) slots += 64u * wave_max_u32(col_nodes[c]);
        block_count_w(stats + BK_STAT_ENTRIES, c_ent, 4);
        block_count_w(stats + BK_STAT_NODES, c_nodes, 4);
        block_count_w(stats + BK_STAT_LANE_SLOTS, (threadIdx.x & 63) == 0 ? slots : 0u, 4);
    }
}

// Matern covariance and its partial derivatives in beta and nu (Sec. III-A
// formula, differentiated), FP64, same tiling and lane mapping as k_matern. With
// z = r / beta and c(nu) = 2^(1-nu) / Gamma(nu):
//   M       = sigma2 c z^nu K_nu(z)
//   dM/dbeta = sigma2 c z^(nu+1) K_{nu-1}(z) / beta     (d/dz z^nu K_nu = -z^nu K_{nu-1})
//   dM/dnu   = M (ln z - ln 2 - psi(nu)) + sigma2 c z^nu dK_nu/dnu(z)
// pref = ln c and psi = psi(nu) come from the host. A NULL output is skipped.
template <typename OutT>
__global__ __launch_bounds__(256) void k_matern_grad(const double* __restrict__ lx, const double* __restrict__ ly,
                                                     TileGeom g, int64_t tile_base, double sigma2, double inv_beta,
                                                     double nu, double pref, double psi, double L, double Lq,
                                                      OutT* __restrict__ oc,
                                                     OutT* __restrict__ ob, OutT* __restrict__ on)
{
    __shared__ double s_tab[kTabLen];
    stage_tab(s_tab);                   // before any wave leaves
    // block -> (tile, row block, column block) in 32-bit arithmetic (a 64-bit
    // division is a long instruction sequence)
    const unsigned wg_per_tile = (unsigned)g.rb_per_tile * (unsigned)g.cb_per_tile;
    const unsigned tq = blockIdx.x / wg_per_tile, local = blockIdx.x - tq * wg_per_tile;
    const int64_t p = tile_base + (int64_t)tq;
    const int rb = (int)(local % (unsigned)g.rb_per_tile), cb = (int)(local / (unsigned)g.rb_per_tile);
    int64_t I, J;
    tile_of(p, g, I, J);
    const int64_t mI = min((int64_t)g.ts, g.n - I * g.ts);
    const int64_t nJ = min((int64_t)g.ts, g.n - J * g.ts);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t il = (int64_t)rb * kRowsPerWave + lane;
    const int64_t jl0 = ((int64_t)cb * 4 + wave) * g.cols;
    if (il >= mI || jl0 >= nJ) return;
    const int64_t base = tile_offset(g.n, g.ts, g.T, g.lower, I, J);
    const double xi = lx[I * g.ts + il], yi = ly[I * g.ts + il];
    const int cend = (int)min((int64_t)g.cols, nJ - jl0);
    for (int c = 0; c < cend; ++c) {
        const int64_t jl = jl0 + c;
        const double xj = lx[J * g.ts + jl], yj = ly[J * g.ts + jl];
        const double dx = xj - xi, dy = yj - yi;
        const double r = sqrt(dx * dx + dy * dy);
        double vc = sigma2, vb = 0.0, vn = 0.0;
        if (r != 0.0) {
            const double z = r * inv_beta, lz = log(z);
            // the same function as k_matern, so that C is bit-identical with or without the derivatives
            Solved s0;
            vc = matern_entry<BK_PLAIN_F64>(nu, z, lz, sigma2, pref, L, Lq, s_tab, s0);
            if (ob) vb = matern_dbeta(nu, z, lz, sigma2, inv_beta, pref, L, Lq, s_tab);
            if (on) vn = matern_dnu(nu, z, lz, sigma2, pref, psi, L, Lq, s_tab, vc, s0.p.t0);
        }
        const int64_t o = base + il + jl * mI;
        if (oc) oc[o] = (OutT)vc;
        if (ob) ob[o] = (OutT)vb;
        if (on) on[o] = (OutT)vn;
    }
}

}  // namespace bk

using namespace bk;

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" const char* bk_status_str(int status)
{
    switch (status) {
    case BK_OK: return "BK_OK";
    case BK_EINVAL: return "BK_EINVAL: invalid argument";
    case BK_EHIP: return "BK_EHIP: HIP runtime error";
    case BK_ENOMEM: return "BK_ENOMEM: workspace too small or allocation failed";
    case BK_ENOMODEL: return "BK_ENOMODEL: learned form requested without a trained model";
    case BK_EIO: return "BK_EIO: model file error";
    case BK_ENOTPD: return "BK_ENOTPD: covariance matrix not positive definite";
    default: return "unknown bk_status";
    }
}

extern "C" int bk_version(void) { return 10000; }

extern "C" int bk_besselk(const double* nu, const double* x, double* out, int64_t n, hipStream_t stream)
{
    bk_params p;
    memset(&p, 0, sizeof(p));
    p.mode = BK_PLAIN_F64;
    return bk_besselk_ex(nu, x, out, n, &p, stream);
}

constexpr int64_t kPlainSmall = 1 << 17, kPlainMid = 800000, kDerivSmall = 16384, kDerivMid = 900000;

// One kernel between the caller's optional event pair.
template <typename K, typename... A>
static int launch_timed(const bk_params* prm, K k, dim3 grid, dim3 block, hipStream_t stream, A&&... a)
{
    if (mark_kernel_event(prm, 0, stream) != hipSuccess) return BK_EHIP;
    const int st = launch(k, grid, block, stream, std::forward<A>(a)...);
    if (st != BK_OK) return st;
    return mark_kernel_event(prm, 1, stream) == hipSuccess ? BK_OK : BK_EHIP;
}

extern "C" int bk_besselk_ex(const double* nu, const double* x, double* out, int64_t n,
                             const bk_params* prm, hipStream_t stream)
{
    if (!prm || n < 0) return BK_EINVAL;
    if (n == 0) return BK_OK;
    if (!nu || !x || !out) return BK_EINVAL;
    if (prm->result < BK_RESULT_K || prm->result > BK_RESULT_LOG) return BK_EINVAL;
    if (prm->L_window < 0.0 || prm->L_quad < 0.0) return BK_EINVAL;
    double L, Lq;
    resolve_thresholds(prm->mode, prm->L_window, prm->L_quad, &L, &Lq);
    const int64_t blocks = (n + kSolveBlock - 1) / kSolveBlock;
    if (blocks > 0x7fffffffLL) return BK_EINVAL;
    switch (prm->mode) {
    case BK_PLAIN_F64:
        // Small calls take one wave a workgroup: no CU waits for another's sort (4,096 pairs
        // 11.4 us against 21.5; 65,536 15 against 22; 200,000 28 against 19 to 23).
        // Between, 512 entries a workgroup (200,000 pairs of the grid 14.7 us, 20.2 with 1,024;
        // 800,000 34.7 and 37.6; 1,048,576 39.5 and 39.2; entries with long windows or solves of
        // their own gain more: 200,000 with x in 1e5 .. 1e8 by the solve 208 and 332). Thresholds
        // that send every entry to the solve: 256, four waves at once (200,000 such pairs 179).
        if (n < kPlainSmall)
            return launch_timed(prm, k_besselk_plain<64, 1>, dim3((unsigned)((n + 63) / 64)), dim3(64), stream, nu, x,
                                out, n, prm->result, L, Lq, prm->stats);
        if (!plan_wide_ok(1.0, 1.0, L, Lq))
            return launch_timed(prm, k_besselk_plain<256, 1>, dim3((unsigned)((n + 255) / 256)), dim3(256), stream, nu,
                                x, out, n, prm->result, L, Lq, prm->stats);
        if (n < kPlainMid)
            return launch_timed(prm, k_besselk_plain<256, 2>, dim3((unsigned)((n + 511) / 512)), dim3(256), stream, nu,
                                x, out, n, prm->result, L, Lq, prm->stats);
        return launch_timed(prm, k_besselk_plain<256, 4>, dim3((unsigned)((n + 1023) / 1024)), dim3(256), stream, nu,
                            x, out, n, prm->result, L, Lq, prm->stats);
    case BK_MIXED_F32C:
        return launch_timed(prm, k_besselk_mixed, dim3((unsigned)blocks), dim3(kSolveBlock), stream, nu, x,
                            out, n, prm->result, L, Lq, prm->stats);
    case BK_LEARNED:
        return bk_besselk_learned(nu, x, out, n, prm, L, Lq, stream);
    case BK_PAPER_REFINED: {
        if (prm->bins < 0 || prm->bins > 100000 || prm->t_upper < 0.0) return BK_EINVAL;
        const int64_t b256 = (n + 255) / 256;
        return launch_timed(prm, k_besselk_paper, dim3((unsigned)b256), dim3(256), stream, nu, x, out, n,
                            prm->result, prm->bins > 0 ? prm->bins : kPaperBins,
                            prm->t_upper > 0.0 ? prm->t_upper : kPaperT, prm->stats);
    }
    default:
        return BK_EINVAL;
    }
}

extern "C" int bk_window(const double* nu, const double* x, double* t_lo, double* t_hi, int32_t* nodes,
                         int64_t n, double L_window, double L_quad, hipStream_t stream)
{
    if (n < 0 || L_window < 0.0 || L_quad < 0.0) return BK_EINVAL;
    if (n == 0) return BK_OK;
    if (!nu || !x || !t_lo || !t_hi || !nodes) return BK_EINVAL;
    double L, Lq;
    resolve_thresholds(BK_MIXED_F32C, L_window, L_quad, &L, &Lq);
    const int64_t blocks = (n + 255) / 256;
    if (blocks > 0x7fffffffLL) return BK_EINVAL;
    return launch(k_window, dim3((unsigned)blocks), dim3(256), stream, nu, x, t_lo, t_hi, nodes, n, L, Lq);
}

extern "C" int64_t bk_matern_out_elems(int64_t n, int32_t tile_size, int32_t lower_only)
{
    if (n < 0 || tile_size <= 0) return -1;
    if (n == 0) return 0;
    int64_t ts = tile_size, T = (n + ts - 1) / ts;
    if (!lower_only) return n * n;
    return tile_offset(n, ts, T, 1, T - 1, T - 1) + (n - (T - 1) * ts) * (n - (T - 1) * ts);
}

extern "C" int64_t bk_matern_tile_offset(int64_t n, int32_t tile_size, int32_t lower_only, int32_t I, int32_t J)
{
    if (n <= 0 || tile_size <= 0) return -1;
    int64_t ts = tile_size, T = (n + ts - 1) / ts;
    if (I < 0 || J < 0 || I >= T || J >= T) return -1;
    if (lower_only && J > I) return -1;
    return tile_offset(n, ts, T, lower_only ? 1 : 0, I, J);
}

// Matern tiles of the plain, mixed and paper forms: launches of at most 2^23
// workgroups (below 2^31 work-items each); the caller's event pair, if any,
// brackets them all.
template <int MODE, typename OutT>
static int launch_matern(const bk_locs* locs, const bk_params* prm, const TileGeom& g, int64_t ntiles,
                         double L, double Lq, void* out, hipStream_t stream)
{
    const double nu = prm->nu;
    const double pref = (1.0 - nu) * kLn2 - lgamma(nu);
    const int64_t wg_per_tile = (int64_t)g.rb_per_tile * g.cb_per_tile;
    const int64_t max_wg = 1LL << 23;
    const int64_t tiles_per_launch = max_wg / wg_per_tile > 0 ? max_wg / wg_per_tile : 1;
    const int bins = prm->bins > 0 ? prm->bins : kPaperBins;
    const double T = prm->t_upper > 0.0 ? prm->t_upper : kPaperT;
    if (mark_kernel_event(prm, 0, stream) != hipSuccess) return BK_EHIP;
    for (int64_t t0 = 0; t0 < ntiles; t0 += tiles_per_launch) {
        const int64_t nt = ntiles - t0 < tiles_per_launch ? ntiles - t0 : tiles_per_launch;
        const dim3 grid((unsigned)(nt * wg_per_tile));
        const int st = prm->stats
            ? launch(k_matern<MODE, OutT, true>, grid, dim3(256), stream, locs->x, locs->y, g, t0, prm->sigma2,
                     1.0 / prm->beta, nu, pref, L, Lq, bins, T, (OutT*)out, prm->stats)
            : launch(k_matern<MODE, OutT, false>, grid, dim3(256), stream, locs->x, locs->y, g, t0, prm->sigma2,
                     1.0 / prm->beta, nu, pref, L, Lq, bins, T, (OutT*)out, prm->stats);
        if (st != BK_OK) return st;
    }
    return mark_kernel_event(prm, 1, stream) == hipSuccess ? BK_OK : BK_EHIP;
}

namespace bk {

int matern_tiles_dispatch(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only,
                          void* out, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (!locs || !prm || tile_size <= 0 || locs->n < 0) return BK_EINVAL;
    if (!(prm->beta > 0.0) || !(prm->nu > 0.0) || !(prm->sigma2 >= 0.0) || isinf(prm->nu) || isinf(prm->beta))
        return BK_EINVAL;
    if (prm->out_dtype != BK_OUT_F64 && prm->out_dtype != BK_OUT_F32) return BK_EINVAL;
    if (prm->L_window < 0.0 || prm->L_quad < 0.0) return BK_EINVAL;
    if (locs->n == 0) return BK_OK;
    if (!locs->x || !locs->y || !out) return BK_EINVAL;
    TileGeom g;
    g.n = locs->n;
    g.ts = (int32_t)(tile_size < locs->n ? tile_size : locs->n);
    g.T = (int32_t)((locs->n + g.ts - 1) / g.ts);
    g.lower = lower_only ? 1 : 0;
    g.rb_per_tile = (g.ts + kRowsPerWave - 1) / kRowsPerWave;
    g.cols = prm->stats ? kMaxCols : cols_per_wave(bk_matern_out_elems(locs->n, tile_size, lower_only));
    g.cb_per_tile = (g.ts + 4 * g.cols - 1) / (4 * g.cols);
    const int64_t T = g.T;
    const int64_t ntiles = g.lower ? T * (T + 1) / 2 : T * T;
    double L, Lq;
    resolve_thresholds(prm->mode, prm->L_window, prm->L_quad, &L, &Lq);
    const bool f32 = prm->out_dtype == BK_OUT_F32;
    // Large builds by tables. A call with statistics first runs the per-entry form, which
    // counts, and its output is then written as any other call of the size writes it.
    if ((prm->mode == BK_PLAIN_F64 || (prm->mode == BK_MIXED_F32C && f32)) &&
        table_route(locs, prm, tile_size, lower_only, prm->mode == BK_MIXED_F32C ? kTabMinF32 : kTabMinF64)) {
        if (prm->stats) {
            bk_params count = *prm;
            count.kernel_events[0] = count.kernel_events[1] = nullptr;
            const int st = prm->mode == BK_MIXED_F32C
                ? launch_matern<BK_MIXED_F32C, float>(locs, &count, g, ntiles, L, Lq, out, stream)
                : (f32 ? launch_matern<BK_PLAIN_F64, float>(locs, &count, g, ntiles, L, Lq, out, stream)
                       : launch_matern<BK_PLAIN_F64, double>(locs, &count, g, ntiles, L, Lq, out, stream));
            if (st != BK_OK) return st;
        }
        return matern_table_tiles(locs, prm, tile_size, lower_only, out, stream);
    }
    switch (prm->mode) {
    case BK_PLAIN_F64:
        return f32 ? launch_matern<BK_PLAIN_F64, float>(locs, prm, g, ntiles, L, Lq, out, stream)
                   : launch_matern<BK_PLAIN_F64, double>(locs, prm, g, ntiles, L, Lq, out, stream);
    case BK_MIXED_F32C:
        return f32 ? launch_matern<BK_MIXED_F32C, float>(locs, prm, g, ntiles, L, Lq, out, stream)
                   : launch_matern<BK_MIXED_F32C, double>(locs, prm, g, ntiles, L, Lq, out, stream);
    case BK_LEARNED:
        return bk_matern_learned(locs, prm, tile_size, lower_only, out, L, Lq, workspace, workspace_bytes, stream);
    case BK_PAPER_REFINED:
        if (prm->bins < 0 || prm->bins > 100000 || prm->t_upper < 0.0) return BK_EINVAL;
        return f32 ? launch_matern<BK_PAPER_REFINED, float>(locs, prm, g, ntiles, L, Lq, out, stream)
                   : launch_matern<BK_PAPER_REFINED, double>(locs, prm, g, ntiles, L, Lq, out, stream);
    default:
        return BK_EINVAL;
    }
}

}  // namespace bk

extern "C" int bk_matern_tiles(const bk_locs* locs, const bk_params* prm, int32_t tile_size,
                               int32_t lower_only, void* out, hipStream_t stream)
{
    if (!prm) return BK_EINVAL;
    return matern_tiles_dispatch(locs, prm, tile_size, lower_only, out, prm->workspace, prm->workspace_bytes,
                                 stream);
}

// Digamma psi(v), v > 0, on the host in long double: shift up with
// psi(v) = psi(v + 1) - 1/v until v >= 12, then the asymptotic expansion
// ln v - 1/(2v) - 1/(12 v^2) + 1/(120 v^4) - 1/(252 v^6) + 1/(240 v^8) - 1/(132 v^10)
// + 691/(32760 v^12) (Abramowitz & Stegun 6.3.18); the first omitted term,
// 1/(12 v^14), is below 3e-17 of psi(12).
double bk::digamma_host(double v)
{
    long double t = v, acc = 0.0L;
    for (; t < 12.0L; t += 1.0L) acc -= 1.0L / t;
    const long double w = 1.0L / (t * t);
    const long double tail =
        w * (1.0L / 12 - w * (1.0L / 120 - w * (1.0L / 252 - w * (1.0L / 240 - w * (1.0L / 132 - w * (691.0L / 32760))))));
    return (double)(acc + logl(t) - 0.5L / t - tail);
}

static int check_deriv_params(const bk_params* prm, bk_params* use)
{
    if (prm) *use = *prm;
    else memset(use, 0, sizeof(*use));
    if (use->mode != BK_PLAIN_F64) return BK_EINVAL;
    if (use->result != BK_RESULT_K && use->result != BK_RESULT_SCALED) return BK_EINVAL;
    if (use->L_window < 0.0 || use->L_quad < 0.0) return BK_EINVAL;
    return BK_OK;
}

extern "C" int bk_besselk_deriv(const double* nu, const double* x, double* k, double* dk_dx, double* dk_dnu,
                                int64_t n, const bk_params* prm, hipStream_t stream)
{
    bk_params p;
    if (n < 0) return BK_EINVAL;
    int st = check_deriv_params(prm, &p);
    if (st != BK_OK) return st;
    if (n == 0) return BK_OK;
    if (!nu || !x || (!k && !dk_dx && !dk_dnu)) return BK_EINVAL;
    double L, Lq;
    resolve_thresholds(BK_PLAIN_F64, p.L_window, p.L_quad, &L, &Lq);
    if ((n + 255) / 256 > 0x7fffffffLL) return BK_EINVAL;
    // as bk_besselk_ex's plain form; in between four waves on 256 entries, which hold up none of
    // the exact solves (us by one wave, by four on 256 and on 1,024: 20,000 pairs of the grid 21,
    // 20, 42; 200,000 42, 37, 45; 800,000 107, 94, 97; 1,048,576 136, 117, 103; 400,000 by the
    // solves 237, 238, 315)
    if (n < kDerivSmall)
        return launch(k_besselk_deriv<64, 1>, dim3((unsigned)((n + 63) / 64)), dim3(64), stream, nu, x, k, dk_dx, dk_dnu,
                      n, p.result, L, Lq, p.stats);
    if (n < kDerivMid || L < 8.0 || !plan_wide_ok(1.0, 1.0, L, Lq))
        return launch(k_besselk_deriv<256, 1>, dim3((unsigned)((n + 255) / 256)), dim3(256), stream, nu, x, k, dk_dx,
                      dk_dnu, n, p.result, L, Lq, p.stats);
    return launch(k_besselk_deriv<256, 4>, dim3((unsigned)((n + 1023) / 1024)), dim3(256), stream, nu, x, k, dk_dx,
                  dk_dnu, n, p.result, L, Lq, p.stats);
}

template <typename OutT>
static int launch_matern_grad(const bk_locs* locs, const bk_params* prm, const TileGeom& g, int64_t ntiles,
                              double L, double Lq, void* c, void* db, void* dn, hipStream_t stream)
{
    const double nu = prm->nu;
    const double pref = (1.0 - nu) * kLn2 - lgamma(nu);
    const double psi = digamma_host(nu);
    const int64_t wg_per_tile = (int64_t)g.rb_per_tile * g.cb_per_tile;
    const int64_t max_wg = 1LL << 23;
    const int64_t tiles_per_launch = max_wg / wg_per_tile > 0 ? max_wg / wg_per_tile : 1;
    for (int64_t t0 = 0; t0 < ntiles; t0 += tiles_per_launch) {
        const int64_t nt = ntiles - t0 < tiles_per_launch ? ntiles - t0 : tiles_per_launch;
        const int st = launch(k_matern_grad<OutT>, dim3((unsigned)(nt * wg_per_tile)), dim3(256), stream, locs->x,
                              locs->y, g, t0, prm->sigma2, 1.0 / prm->beta, nu, pref, psi, L, Lq, (OutT*)c,
                              (OutT*)db, (OutT*)dn);
        if (st != BK_OK) return st;
    }
    return BK_OK;
}

extern "C" int bk_matern_grad_tiles(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only,
                                    void* c, void* dc_dbeta, void* dc_dnu, hipStream_t stream)
{
    if (!locs || !prm || tile_size <= 0 || locs->n < 0) return BK_EINVAL;
    if (prm->mode != BK_PLAIN_F64) return BK_EINVAL;
    if (!(prm->beta > 0.0) || !(prm->nu > 0.0) || !(prm->sigma2 >= 0.0) || isinf(prm->nu) || isinf(prm->beta))
        return BK_EINVAL;
    if (prm->out_dtype != BK_OUT_F64 && prm->out_dtype != BK_OUT_F32) return BK_EINVAL;
    if (prm->L_window < 0.0 || prm->L_quad < 0.0) return BK_EINVAL;
    if (locs->n == 0) return BK_OK;
    if (!locs->x || !locs->y || (!c && !dc_dbeta && !dc_dnu)) return BK_EINVAL;
    if (table_route(locs, prm, tile_size, lower_only, kTabMinF64)) {
        void* const outs[3] = {c, dc_dbeta, dc_dnu};
        return matern_grad_table_tiles(locs, prm, digamma_host(prm->nu), tile_size, lower_only, outs, stream);
    }
    TileGeom g;
    g.n = locs->n;
    g.ts = (int32_t)(tile_size < locs->n ? tile_size : locs->n);
    g.T = (int32_t)((locs->n + g.ts - 1) / g.ts);
    g.lower = lower_only ? 1 : 0;
    g.rb_per_tile = (g.ts + kRowsPerWave - 1) / kRowsPerWave;
    g.cols = cols_per_wave(bk_matern_out_elems(locs->n, tile_size, lower_only));
    g.cb_per_tile = (g.ts + 4 * g.cols - 1) / (4 * g.cols);
    const int64_t T = g.T;
    const int64_t ntiles = g.lower ? T * (T + 1) / 2 : T * T;
    double L, Lq;
    resolve_thresholds(BK_PLAIN_F64, prm->L_window, prm->L_quad, &L, &Lq);
    if (prm->out_dtype == BK_OUT_F32)
        return launch_matern_grad<float>(locs, prm, g, ntiles, L, Lq, c, dc_dbeta, dc_dnu, stream);
    return launch_matern_grad<double>(locs, prm, g, ntiles, L, Lq, c, dc_dbeta, dc_dnu, stream);
}
