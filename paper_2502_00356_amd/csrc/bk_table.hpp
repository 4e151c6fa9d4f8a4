// bk_table.hpp - Matern tiles by interpolation in r^2: table shapes, the interval
// fit shared by the table builders (bk_table.hip, bk_mlp.hip), and the launches.
//
// At one (sigma^2, beta, nu) every entry of a Matern matrix is one function of the
// squared distance q = r^2. A large build therefore evaluates the quadrature at the
// Chebyshev points of a few hundred intervals of q, and every entry by its interval's
// polynomial: no square root, no exponential and no window solve per entry.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bk_internal.hpp"

namespace bk {

// Intervals: p(q) = fa bits(q) + fb sqrt(q) + fc advances by one per interval, q in
// FP32, bits(q) its bit pattern (2^-23 of it is log2 q, linear within an octave): kA
// intervals per octave of z^2 and kB per unit of z = r / beta, from z = kZMin. The
// octaves keep an interval narrow against its distance from the branch point at z = 0,
// the linear part against the e^-z decay; kN intervals (the first and last unused)
// reach z = 128. FP64 table:
// degree 8, truncation below 6e-16 relative for C and dC/dbeta over nu in [0.05, 15]
// (largest near z = 64; below 2e-16 for z < 2). FP32 table: degree 4, below 2.3e-9.
template <bool kF32>
struct TabShape;
template <>
struct TabShape<false> {
    static constexpr int kDeg = 8, kPlanes = 5, kN = 832;
    static constexpr double kA = 10.0, kB = 3.2, kZMin = 0x1p-14;
};
template <>
struct TabShape<true> {
    static constexpr int kDeg = 4, kPlanes = 2, kN = 1075;
    static constexpr double kA = 8.0, kB = 6.0, kZMin = 0x1p-12;
};

// The interval rule of a call, the scale of the FP32 table's argument (1 / beta^2) and the
// last slot's constant term: NaN, or 0 where an FP32 table's function rounds to 0 there.
struct TabIndex {
    float fa, fb, fc, vs, end;
};

__device__ __forceinline__ float tab_pos(const TabIndex& X, float q)
{
    return fmaf((float)__float_as_uint(q), X.fa, fmaf(__builtin_amdgcn_sqrtf(q), X.fb, X.fc));
}

typedef double tab2_t __attribute__((ext_vector_type(2)));
typedef float tab4f_t __attribute__((ext_vector_type(4)));

// A table is kPlanes planes of kN 16-byte slots, then 16 bytes of counts. Slot i of the planes
// in turn: {centre, c0}, {c1, c2}, ... {c7, c8}, the polynomial in q - centre (r^2 units);
// FP32 table: {centre, c0}, {c1 .. c4 in FP32, relative to c0}, the polynomial's argument
// scaled by 1 / beta^2. Planes rather than records: the 16 slots of one LDS bank row are then
// 16 neighbouring intervals.
template <bool kF32>
constexpr size_t tab_bytes()
{
    return (size_t)TabShape<kF32>::kPlanes * TabShape<kF32>::kN * 16 + 16;
}

// Which function a table holds.
enum TabFn { TAB_C = 0, TAB_DBETA = 1, TAB_DNU = 2 };

// The function of a call: host values. pref = ln c, scale = sigma2 c, c = 2^(1-nu) /
// Gamma(nu); psi = digamma(nu), for dC/dnu. zero: a z (at least kTabFar) from which the
// call's functions round to 0 in the output's type. Seven doubles: with eight they pass
// to the evaluation's out-of-line function through the stack (5 us a launch).
struct TabParams {
    double sigma2, inv_beta, nu, pref, psi, scale, zero;
};
TabParams tab_params(const bk_params* prm, bool grad, double psi);

// Below the last slot's first z (128, less the steps of log2's linear pieces).
constexpr double kTabFar = 127.0;

// The q where tab_pos(q) = t, to a few of tab_pos's own roundings (1e-4 of an interval:
// an entry that the rule puts on the other side of a boundary reads its neighbour's
// polynomial that far past the end). Newton on the bit pattern b, in which tab_pos is
// convex up to the steps of log2's linear pieces, from the smaller of the two terms' own
// solutions (the other at most doubles the value there); five steps leave up to 0.25 of an
// interval, six and seven 2.4e-4.
__device__ __forceinline__ float tab_bound(const TabIndex& X, float t)
{
    // the log term alone, and the linear one over the first boundary's log term
    const float rfa = __builtin_amdgcn_rcpf(X.fa), b1 = (t - X.fc) * rfa;
    const float r = fmaxf(t, 0.0f) * __builtin_amdgcn_rcpf(X.fb), b2 = (float)__float_as_uint(fmaxf(r * r, 0x1p-120f));
    unsigned b = (unsigned)fminf(fmaxf(fminf(b1, b2), 0x1p24f), 0x7f0p20f);
    for (int k = 0; k < 7; ++k) {
        const float q = __uint_as_float(b);
        const float e = __uint_as_float(b & 0x7f800000u) * 0x1p-23f;                // dq/db
        const float d = fmaf(0.5f * X.fb * e, __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(q)), X.fa);
        b = (unsigned)min(max((int)b + (int)((t - tab_pos(X, q)) * __builtin_amdgcn_rcpf(d)), 1 << 24), 0x7f000000);
    }
    return __uint_as_float(b);
}

// cos(n pi (j + 1/2) / M) and the monomial coefficients of T_n.
template <int M>
struct ChebTab {
    double cosn[M][M], mono[M][M];
};
#include "bk_cheb.inc"      // kCheb5, kCheb9

template <bool kF32>
__device__ __forceinline__ const ChebTab<TabShape<kF32>::kDeg + 1>& cheb_tab()
{
    if constexpr (kF32) return kCheb5;
    else return kCheb9;
}

// A builder's workgroup takes one wave's worth of Chebyshev points: kPer intervals (kTabLanes
// lanes a point in bk_table.hip, one in bk_mlp.hip).
template <bool kF32>
struct TabWave {
    static constexpr int kM = TabShape<kF32>::kDeg + 1, kPer = 64 / kM;
    static constexpr int kBlocks = (TabShape<kF32>::kN + kPer - 1) / kPer;
    int g, j, i;          // interval within the wave, Chebyshev point, interval
    double c, w, z;       // centre and half-width in r^2, the lane's point z = r / beta
};

// Point `lane` of a workgroup. Idle ones (past kPer intervals) repeat the last interval's first.
template <bool kF32>
__device__ __forceinline__ TabWave<kF32> tab_point(const TabIndex& X, double inv_beta, int block, int lane)
{
    TabWave<kF32> t;
    t.g = min(lane / TabWave<kF32>::kM, TabWave<kF32>::kPer - 1);
    t.j = lane < TabWave<kF32>::kPer * TabWave<kF32>::kM ? lane - t.g * TabWave<kF32>::kM : 0;
    const int i0 = block * TabWave<kF32>::kPer;
    t.i = i0 + t.g;
    const float qb = tab_bound(X, (float)(i0 + (threadIdx.x & 63)));      // the wave's lane's boundary
    const double ql = (double)__shfl(qb, t.g, 64), qh = (double)__shfl(qb, t.g + 1, 64);
    t.c = 0.5 * (ql + qh);
    t.w = 0.5 * (qh - ql);
    t.z = sqrt(fma(t.w, cheb_tab<kF32>().cosn[1][t.j], t.c)) * inv_beta;
    return t;
}

// Fits the wave's intervals to the lanes' samples f and writes their slots. The
// Chebyshev coefficients come from the differences to the middle sample and are then
// expanded in powers, so that neither sum rounds at the size of f. sh: 64 doubles.
template <bool kF32>
__device__ inline void tab_fit(const TabWave<kF32>& t, double f, const TabIndex& X, double* sh, char* table, int lane,
                               bool first)
{
    constexpr int M = TabWave<kF32>::kM, kN = TabShape<kF32>::kN;
    const ChebTab<M>& C = cheb_tab<kF32>();
    const bool live = first && lane < TabWave<kF32>::kPer * M && t.i < kN;
    if (first) sh[lane] = f;
    __syncthreads();
    const double* s = sh + t.g * M;
    const double mid = s[M / 2];
    double cn = 0.0;
    for (int j = 0; j < M; ++j) cn = fma(s[j] - mid, C.cosn[t.j][j], cn);
    cn *= (t.j == 0 ? 1.0 : 2.0) / M;
    __syncthreads();
    if (first) sh[lane] = cn;
    __syncthreads();
    double a = 0.0;
    for (int n = M - 1; n >= 0; --n) a = fma(C.mono[n][t.j], s[n], a);
    if (t.j == 0) a += mid;
    // powers of q - centre (FP32 table: of the scaled difference)
    const double iw = 1.0 / (kF32 ? t.w * (double)X.vs : t.w);
    for (int k = 0; k < t.j; ++k) a *= iw;
    if (kF32) {
        __syncthreads();
        if (first) sh[lane] = a;
        __syncthreads();
        if (t.j > 0) a /= s[0];
    }
    if (!live) return;
    double* slots = (double*)table;
    if (t.j == 0) slots[2 * t.i] = t.c;
    if (kF32 && t.j > 0) {
        ((float*)table)[4 * (kN + t.i) + t.j - 1] = t.i == kN - 1 ? 0.0f : (float)a;
    } else {
        const int e = t.j + 1;
        // the first and last slots stand for everything out of the table
        if (t.j == 0 && t.i == 0) a = __builtin_nan("");
        if (t.j == 0 && t.i == kN - 1) a = (double)X.end;
        slots[2 * ((e >> 1) * kN + t.i) + (e & 1)] = a;
    }
}

// scale z^e e^(delta - z) hs, the quadrature's assembly of a sample: the power taken as
// such and the roundings of delta - z and of the products carried (the samples set the
// error of every entry; the per-entry kernels add these factors' logarithms instead).
__device__ __forceinline__ double tab_assemble(double scale, double z, double e, double delta, double hs)
{
    const double d = delta - z, lo = two_sum_err(delta, -z, d);
    const double w = pow(z, e), x = exp(d);
    const double p = scale * w, pe = fma(scale, w, -p), q = x * hs, qe = fma(x, hs, -q);
    const double v = p * q, ve = fma(p, q, -v);
    return v + fma(pe, q, fma(p, qe, fma(v, lo, ve)));
}

// The evaluation kernel's counts, cleared by the builder: workgroups that have read the
// table, and that have finished (in the high half: those that left their share of the
// table's bytes to the last).
template <bool kF32>
__host__ __device__ __forceinline__ unsigned int* tab_counts(char* table)
{
    return (unsigned int*)(table + (size_t)TabShape<kF32>::kPlanes * TabShape<kF32>::kN * 16);
}

template <bool kF32>
__device__ __forceinline__ void tab_clear(char* table)
{
    tab_counts<kF32>(table)[0] = 0u;
    tab_counts<kF32>(table)[1] = 0u;
}

// Entries from which a call takes a table (FP64: plain form and gradient; FP32: mixed).
// Per-entry form against table, us: plain 130,000 entries 16.9 / 20.2, 262,000 21.3 / 19.8;
// gradient 44 / 48 and 57 / 48; mixed 65,500 16.4 / 16.9, 130,000 20.8 / 17.6. The learned
// form's own launches take longer at any size (10,000 entries 47 / 22): from a little above
// the least output that holds its table on (8,610 entries). In tiles below 24 rows the items
// of the table's bytes are many and short, which small outputs mostly consist of (40,000
// entries in 4-tiles 29 / 50, 114,000 in 16-tiles 40 / 41, in 24-tiles 45 / 32; 220,900 in
// 1-tiles 200 / 226, 500,500 724 / 518): from 500,000 there.
constexpr int64_t kTabMinF64 = 200000, kTabMinF32 = 70000, kTabMinLearned = 10000, kTabMinLearnedNarrow = 500000;
constexpr int kTabNarrow = 24;

// Whether a call takes the tables, and where in an output of elems elements of
// elem_bytes its table is built: its last bytes, which the evaluation writes last.
bool table_route(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only, int64_t min_entries);
char* table_in_output(void* out, int64_t elems, int elem_bytes, bool f32_table, int64_t* first);
TabIndex tab_index(double beta, const TabParams& P, bool f32_table);

// Evaluation over all tiles from the table in `out` (built on the same stream); fn: a TabFn.
// Entries outside the table take a series, NaN and infinite distances and those next to 0 the
// plain form (from an FP32 table the mixed one).
int launch_table_eval(const bk_locs* locs, const TabParams& P, const TabIndex& X, int32_t tile_size, int32_t lower_only, int fn,
                      bool f32_table, int out_dtype, void* out, hipStream_t stream);
// Plain and mixed forms: builds the table and evaluates. bk_status.
int matern_table_tiles(const bk_locs* locs, const bk_params* prm, int32_t tile_size, int32_t lower_only, void* out,
                       hipStream_t stream);
int matern_grad_table_tiles(const bk_locs* locs, const bk_params* prm, double psi, int32_t tile_size,
                            int32_t lower_only, void* const outs[3], hipStream_t stream);

}  // namespace bk
