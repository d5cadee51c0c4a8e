// exec.hip -- execution of a planned transform (Alg. 2): local blocks by the
// Wimp expansion (Sec. 3.1), asymptotic blocks by type-3 NUFFTs of Hankel's
// expansion (Sec. 3.2) or, the smaller ones, Chebyshev expansions in both
// variables, direct blocks entry by entry or through such expansions.
//
// Column side (reductions over points):  gather c -> local moments ->
//   ES spreading of 2M weight channels onto each asymptotic block's grid.
// Grid stage:  reduce spread partials; for large grids deconvolve by the
//   inner kernel's transform, zero-pad and FFT.
// Row side (one thread per frequency): walk the block tree from the root and
//   add, level by level, the row's local, asymptotic and (at the end) direct
//   contributions; write g once, in the caller's order.
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

#include "nuht_device.h"
#include "nuht_launch.h"

namespace nuht {

// Orders the LDS accesses of the wave's lanes around it (the region is
// written and read by different lanes of the same wave).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Every execution kernel is a body taking the transform (P) and the index of
// its workgroup within that transform's work.  A single transform's kernel
// passes P by value and blockIdx.x; a batched kernel covers every transform
// of a batch in one launch: its workgroup finds its transform in a table of
// segments (WorkSeg, ascending g0) and runs the body on that transform's
// PlanDev, kept in device memory, as its workgroup blockIdx.x - g0.
// ---------------------------------------------------------------------------
// A batch's PlanDev array is written once, before the graph that reads it is
// recorded, and never while a batched kernel runs: it is read through the
// constant address space, like a kernel argument, so that the compiler may
// load its fields through the scalar unit.
typedef const __attribute__((address_space(4))) PlanDev ConstPlanDev;
__device__ __forceinline__ const PlanDev& plan_of(const PlanDev* plans, int t)
{
    return *(const PlanDev*)((ConstPlanDev*)plans + t);
}

// The segment of this workgroup (the last one with g0 <= blockIdx.x).
template <class Seg>
__device__ __forceinline__ int find_seg_index(const Seg* __restrict__ segs, int nseg)
{
    const int g = blockIdx.x;
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].g0 <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The transform of this workgroup and the workgroup's index within it.
__device__ __forceinline__ WorkSeg find_seg(const WorkSeg* __restrict__ segs, int nseg)
{
    const int s = find_seg_index(segs, nseg);
    return WorkSeg{segs[s].t, (int32_t)blockIdx.x - segs[s].g0};
}

// cs[k] = c[perm[k]] (times the sorted point r_k when scale is set).
__device__ __forceinline__ void gather_body(const PlanDev& P, int bid, const double* c, bool scale)
{
    const int32_t k = bid * blockDim.x + threadIdx.x;
    if (k >= P.n) return;
    const double v = c[P.perm_r[k]];
    P.cs[k] = scale ? v * P.rs[k] : v;
}

// c is read from c_slot when that is set.
__global__ void k_gather(PlanDev P, const double* c, const double* const* c_slot, int scale)
{
    gather_body(P, blockIdx.x, c_slot ? *c_slot : c, scale != 0);
}

__global__ void k_gather_many(const PlanDev* __restrict__ plans, const WorkSeg* __restrict__ segs, int nseg,
                              const double* const* c_table)
{
    const WorkSeg w = find_seg(segs, nseg);
    gather_body(plan_of(plans, w.t), w.g0, c_table[w.t], false);
}

// A transform with no points: the output is zero.
__global__ void k_zero_output(double* g, double* const* g_slot, int64_t m)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    double* gp = g_slot ? *g_slot : g;
    gp[i] = 0.0;
}

__global__ void k_zero_output_many(const PlanDev* __restrict__ plans, const WorkSeg* __restrict__ segs, int nseg,
                                   double* const* g_table)
{
    const WorkSeg w = find_seg(segs, nseg);
    const int64_t i = (int64_t)w.g0 * blockDim.x + threadIdx.x;
    if (i < plan_of(plans, w.t).m) g_table[w.t][i] = 0.0;
}

__global__ void k_fill_value(double* __restrict__ x, int64_t n, double v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

struct PtrArgs {
    void* p[224];
};

__global__ void k_set_pointers(void** table, PtrArgs a, int count)
{
    int i = threadIdx.x;
    if (i < count) table[i] = a.p[i];
}

// out = w (a - b) / 2: the derivative J_nu' = (J_{nu-1} - J_{nu+1}) / 2 applied
// to the two shifted-order transforms.
__global__ void k_half_difference(const double* __restrict__ w, const double* __restrict__ a,
                                  const double* __restrict__ b, double* __restrict__ out, int32_t n)
{
    int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[k] = 0.5 * w[k] * (a[k] - b[k]);
}

// ---------------------------------------------------------------------------
// Local moments t_l = sum_k c_k T_{2l(+1)}(r_k / R) of one chunk of a local
// block's columns (Sec. 3.1: T^T applied first).  The Chebyshev polynomials
// come from the recurrence in u = 2y^2 - 1:  T_{2(l+1)+e}(y) = 2u T_{2l+e}(y) - T_{2(l-1)+e}(y).
// Moments are produced in passes of up to 64 (a multiple of 8: all L + 1 in
// one pass up to L = 63, so no pass repeats the recurrence through an earlier
// pass's moments there).  One 64-lane wave per item: each lane accumulates its
// points' moments in registers (points strided over the lanes), and the wave
// reduces them with cross-lane sums, in chunks of 64, 32, 16 and 8 moments.
// ---------------------------------------------------------------------------
// One reduce-scatter level: v[0 .. 2H) -> v[0 .. H), lanes with bit H set
// keeping the upper half; partner lane ^ H holds the other copy.
template <int H, int NQ>
__device__ __forceinline__ void reduce_scatter_half(double (&v)[NQ], int lane)
{
    const bool upper = (lane & H) != 0;
    #pragma unroll
    for (int i = 0; i < H; ++i) {
        double keep = upper ? v[i + H] : v[i];
        double send = upper ? v[i] : v[i + H];
        v[i] = keep + __shfl_xor(send, H);
    }
}

// Sum over the wave of the C moments acc[off .. off + C) (C a power of two,
// 8 to 64): a reduce-scatter at offsets C/2 .. 1 leaves lane q with moment
// off + (q mod C) summed over the lanes congruent to q; exchanges at offsets
// C .. 32 complete the sums.
template <int C, int NQ>
__device__ __forceinline__ double reduce_chunk(const double (&acc)[NQ], int off, int lane)
{
    double v[C];
    #pragma unroll
    for (int i = 0; i < C; ++i) v[i] = acc[off + i];
    if constexpr (C >= 64) reduce_scatter_half<32>(v, lane);
    if constexpr (C >= 32) reduce_scatter_half<16>(v, lane);
    if constexpr (C >= 16) reduce_scatter_half<8>(v, lane);
    reduce_scatter_half<4>(v, lane);
    reduce_scatter_half<2>(v, lane);
    reduce_scatter_half<1>(v, lane);
    double mine = v[0];
    #pragma unroll
    for (int o = C; o < 64; o <<= 1) mine += __shfl_xor(mine, o);
    return mine;
}

// A moment as the row evaluations use it: u_0 = t_0, u_l = 2 (-1)^l t_l
// (integer orders), t_l itself (half-integer orders: the factors are in the
// table).
__device__ __forceinline__ double moment_as_used(const PlanDev& P, int l, double t)
{
    return (l == 0 || P.half) ? t : ((l & 1) ? -2.0 * t : 2.0 * t);
}

// Stores the chunk of C moments starting at s0 + off (those up to L); `whole`:
// they are a block's only item, stored as used.
template <int C, int NQ>
__device__ __forceinline__ void store_chunk(const PlanDev& P, const double (&acc)[NQ], int off, int s0, int lane,
                                            bool whole, double* __restrict__ dst)
{
    const double mine = reduce_chunk<C>(acc, off, lane);
    const int l = s0 + off + lane;
    if (lane < C && l <= P.L) dst[l] = whole ? moment_as_used(P, l, mine) : mine;
}

// Moments s0 .. s0 + NQ - 1 of the item (those up to L are stored); NQ a
// multiple of 8 up to 64.
template <int NQ>
__device__ __forceinline__ void lmom_pass(const PlanDev& P, const Item& I, const LBlock& B, const double* __restrict__ cs,
                                          double* __restrict__ lpart, int s0, int lane, int bid)
{
    static_assert(NQ % 8 == 0 && NQ >= 8 && NQ <= 64, "pass width");
    const int L = P.L;
    const int odd = P.nu & 1;
    double acc[NQ];
    #pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    // y = r / R through the block's reciprocal (within an ulp of the
    // quotient; y only enters the Chebyshev recurrence)
    const double inv_R = 1.0 / B.R;
    // two points per lane per step (the second with weight 0 past the end):
    // both loads issue together and the recurrences are independent chains
    for (int k = I.ka + lane; k < I.kb; k += 128) {
        const bool two = k + 64 < I.kb;
        const int k2 = two ? k + 64 : k;
        const double ya = P.rs[k] * inv_R, yb = P.rs[k2] * inv_R;
        double ca = cs[k], cb = two ? cs[k2] : 0.0;
        if (P.half) {          // half-integer orders: weights c sqrt(r / R)
            ca *= sqrt(ya);
            cb *= sqrt(yb);
        }
        const double ua2 = 2.0 * __builtin_fma(2.0 * ya, ya, -1.0);
        const double ub2 = 2.0 * __builtin_fma(2.0 * yb, yb, -1.0);
        double a0, a1, b0, b1;
        if (odd) { a0 = ya; a1 = ya * (ua2 - 1.0); b0 = yb; b1 = yb * (ub2 - 1.0); }
        else { a0 = 1.0; a1 = 0.5 * ua2; b0 = 1.0; b1 = 0.5 * ub2; }
        for (int l = 0; l < s0; ++l) {
            const double a2 = __builtin_fma(ua2, a1, -a0), b2 = __builtin_fma(ub2, b1, -b0);
            a0 = a1; a1 = a2; b0 = b1; b1 = b2;
        }
        #pragma unroll
        for (int q = 0; q < NQ; ++q) {
            acc[q] = __builtin_fma(cb, b0, __builtin_fma(ca, a0, acc[q]));
            const double a2 = __builtin_fma(ua2, a1, -a0), b2 = __builtin_fma(ub2, b1, -b0);
            a0 = a1; a1 = a2; b0 = b1; b1 = b2;
        }
    }
    // the pass's moments in chunks of 64, 32, 16 and 8 (NQ's binary digits)
    const bool whole = B.nitems == 1;
    double* __restrict__ dst = whole ? P.lmom + (int64_t)I.blk * (L + 1) : lpart + (int64_t)bid * (L + 1);
    constexpr int c64 = NQ & 64, c32 = NQ & 32, c16 = NQ & 16, c8 = NQ & 8;
    if constexpr (c64) store_chunk<64>(P, acc, 0, s0, lane, whole, dst);
    if constexpr (c32) store_chunk<32>(P, acc, c64, s0, lane, whole, dst);
    if constexpr (c16) store_chunk<16>(P, acc, c64 + c32, s0, lane, whole, dst);
    if constexpr (c8) store_chunk<8>(P, acc, c64 + c32 + c16, s0, lane, whole, dst);
}

// MAXQ: the widest pass (32 or 64).  A kernel's registers follow its widest
// pass, so orders with L < 32 run the 32-wide instance at twice the waves.
template <int MAXQ>
__device__ __forceinline__ void lmom_body(const PlanDev& P, int bid)
{
    const Item I = P.litems[bid];
    const LBlock B = P.lb[I.blk];
    const int L = P.L;
    const int lane = threadIdx.x;
    const double* __restrict__ cs = P.cs;
    double* __restrict__ lpart = P.lpart;
    // passes of up to MAXQ moments, each the multiple of 8 that covers what is left
    for (int s0 = 0; s0 <= L;) {
        const int rem = L + 1 - s0;
        const int nq = rem >= MAXQ ? MAXQ : (rem + 7) / 8 * 8;
        if (nq == 8) lmom_pass<8>(P, I, B, cs, lpart, s0, lane, bid);
        else if (nq == 16) lmom_pass<16>(P, I, B, cs, lpart, s0, lane, bid);
        else if (nq == 24) lmom_pass<24>(P, I, B, cs, lpart, s0, lane, bid);
        else if (nq == 32) lmom_pass<32>(P, I, B, cs, lpart, s0, lane, bid);
        else if constexpr (MAXQ > 32) {
            if (nq == 40) lmom_pass<40>(P, I, B, cs, lpart, s0, lane, bid);
            else if (nq == 48) lmom_pass<48>(P, I, B, cs, lpart, s0, lane, bid);
            else if (nq == 56) lmom_pass<56>(P, I, B, cs, lpart, s0, lane, bid);
            else lmom_pass<64>(P, I, B, cs, lpart, s0, lane, bid);
        }
        s0 += nq;
    }
}

// The instance for an order's local rank L.
constexpr int lmom_width(int L) { return L + 1 <= 32 ? 32 : 64; }

template <int MAXQ>
__global__ __launch_bounds__(64) void k_lmom(PlanDev P) { lmom_body<MAXQ>(P, blockIdx.x); }

template <int MAXQ>
__global__ __launch_bounds__(64) void k_lmom_many(const PlanDev* __restrict__ plans,
                                                  const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    lmom_body<MAXQ>(plan_of(plans, w.t), w.g0);
}

// Sum of a local block's item partials (blocks of several items), in a fixed
// order.  A block can hold a thousand items (the top-level local block spans
// most columns) and a sum's loads are a chain of latencies, so a wave takes
// eight moments and eight lanes share each: lane group s adds items s, s + 8,
// .., four loads in flight, and the groups' sums are combined pairwise.  The
// moments of a partition (blocks times L + 1) can outnumber what 32 bits count
// in lanes, so a workgroup takes every kLmomReduceMax-th group of 32 beyond.
constexpr int64_t kLmomReduceMax = 1 << 20;

__host__ __device__ inline int64_t lmom_reduce_blocks(int64_t n_l, int64_t L)
{
    const int64_t b = (n_l * (L + 1) + 31) / 32;
    return b < kLmomReduceMax ? b : kLmomReduceMax;
}

__device__ __forceinline__ void lmom_reduce_body(const PlanDev& P, int bid)
{
    const int lane = threadIdx.x & 63, sub = lane >> 3;
    const int32_t Lp = P.L + 1;
    const int64_t total = (int64_t)P.n_l * Lp, step = 32 * lmom_reduce_blocks(P.n_l, P.L);
    // (all eight lanes of a moment leave the loop together)
    for (int64_t t = (int64_t)bid * 32 + (threadIdx.x >> 6) * 8 + (lane & 7); t < total; t += step) {
        // (a 32-bit division wherever the counts allow it)
        const int32_t b = total <= INT32_MAX ? (int32_t)t / Lp : (int32_t)(t / Lp);
        const int32_t l = (int32_t)(t - (int64_t)b * Lp);
        const int32_t nitems = P.lb[b].nitems;
        if (nitems == 1) continue;                   // stored by its item
        const double* __restrict__ col = P.lpart + (int64_t)P.lb[b].item0 * Lp + l;
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        int32_t it = sub;
        for (; it + 24 < nitems; it += 32) {
            #pragma unroll
            for (int q = 0; q < 4; ++q) a[q] += col[(int64_t)(it + 8 * q) * Lp];
        }
        #pragma unroll
        for (int q = 0; q < 3; ++q)
            if (it + 8 * q < nitems) a[q] += col[(int64_t)(it + 8 * q) * Lp];
        double s = (a[0] + a[1]) + (a[2] + a[3]);
        #pragma unroll
        for (int o = 8; o < 64; o <<= 1) s += __shfl_xor(s, o);
        if (sub == 0) P.lmom[t] = moment_as_used(P, l, s);
    }
}

__global__ void k_lmom_reduce(PlanDev P) { lmom_reduce_body(P, blockIdx.x); }

__global__ void k_lmom_reduce_many(const PlanDev* __restrict__ plans, const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    lmom_reduce_body(plan_of(plans, w.t), w.g0);
}

// ---------------------------------------------------------------------------
// Rank blocks: asymptotic blocks whose (half r range) x (half omega range) is
// small enough (a few times kRankPanels) that their kernel, without its fast
// phases, is a smooth function of both variables.  With r = C + b,
// omega = D + a,
//   J_nu(omega r) = sqrt(2/pi) (omega r)^(-1/2) Re( e^{i (omega C + phi)} e^{i D b} F(r, omega) ),
//   F = H(omega r) e^{i a b},   H(x) = sum_p beta_p x^(-p)  (Hankel's M terms),
// and F is its Chebyshev interpolant in both variables, K terms in each
// (rank_terms bounds the error).  In place of 2M type-3 transforms per block:
//   moments      t_m = sum_k c_k sqrt(r0 / r_k) e^{i D b_k} T_m(y_k), one set per
//                panel of points (y in [-1, 1] across the panel);
//   weights      the sums at the panel's K nodes, a cosine transform of t;
//   translation  u_t = sum over panels and nodes s of F(r_s, omega_t) weight_s at
//                the K nodes of each panel of frequencies, then the
//                coefficients v_m of the function through them;
//   rows         (omega r0)^(-1/2) Re( e^{i (omega C + phi)} sum_m v_m T_m(eta) ).
// A point or row costs its phase and 3 K operations, where spreading costs w
// taps x 4M sums and a row N1 >= w + 2 cells x (4M + 2).
// ---------------------------------------------------------------------------
// Moments of one item, four waves, a point per lane and step, 2 KC sums in
// registers.  At the end of a panel each wave adds its lanes' sums: half-wave
// and row exchanges leave a quarter of the sums in each row of 16 lanes, and
// the rows are added through LDS.  Where the waves share a panel, the four
// waves' sums are added in order.  Bound by FP64 issue: the phase is about 70
// instructions and a term 3.  The next step's point is loaded a step ahead.
constexpr int kRankWaves = 4;

// What the moments of a rank block need of it.
struct RankCols {
    double C, D, r0, cw;
    int32_t pc, cpan0;
};

// a <- a + a of the other half-wave in lanes 0 .. 31, b likewise in 32 .. 63.
__device__ __forceinline__ double add_halves(double a, double b)
{
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// The same for rows of 16 lanes: a in rows 0 and 2 (with the row above), b in
// rows 1 and 3 (with the row below).
__device__ __forceinline__ double add_rows(double a, double b)
{
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// Sum over the wave of acc[v], in lane v < N (N a multiple of 8, at most 64);
// s: the wave's N / 4 x 64 doubles of LDS.
template <int N>
__device__ __forceinline__ double wave_sums(double (&acc)[N], double* s, int lane)
{
    constexpr int Q = N / 4;
    #pragma unroll
    for (int i = 0; i < 2 * Q; ++i) acc[i] = add_halves(acc[i], acc[i + 2 * Q]);   // values i | i + 2Q
    #pragma unroll
    for (int i = 0; i < Q; ++i) s[i * 64 + lane] = add_rows(acc[i], acc[i + Q]);   // row h: value i + h Q
    wave_sync();
    const int v = lane < N ? lane : 0, h = v / Q, j = v - h * Q;
    const double* row = s + j * 64 + h * 16;
    double sum = 0.0;
    #pragma unroll
    for (int l = 0; l < 16; ++l) sum += row[(l + lane) & 15];
    wave_sync();
    return sum;
}

// Sums over the wave of columns first + 64 stride j + lane < kb of panel q,
// in lane v < 2 KC.
template <int KC>
__device__ __forceinline__ double rank_moments_wave(const PlanDev& P, const RankCols B, int q, int first, int stride,
                                                    int kb, double* s)
{
    const double* __restrict__ cs = P.cs;
    const double* __restrict__ rs = P.rs;
    const int lane = threadIdx.x & 63;
    const double inv_r0 = rcp_refined(B.r0);
    const double inv_w = B.cw > 0.0 ? rcp_refined(B.cw) : 0.0;
    const double mid = rank_mid(q, B.pc, B.cw);
    double acc[2 * KC];
    #pragma unroll
    for (int m = 0; m < 2 * KC; ++m) acc[m] = 0.0;
    int k = first + lane;
    double r_nx = B.r0, c_nx = 0.0;
    if (k < kb) { r_nx = rs[k]; c_nx = cs[k]; }
    for (int k0 = first; k0 < kb; k0 += 64 * stride) {
        const double r = r_nx, c = c_nx;
        k += 64 * stride;
        r_nx = B.r0; c_nx = 0.0;
        if (k < kb) { r_nx = rs[k]; c_nx = cs[k]; }
        const dd tp = two_sum(r, -B.C);
        const dd ph = two_prod(B.D, tp.hi);
        double cth, sth;
        cis_dd(ph.hi, __builtin_fma(B.D, tp.lo, ph.lo), cth, sth);
        const double w0 = c * rsqrt_refined(r * inv_r0);
        const double xr = w0 * cth, xi = w0 * sth;
        const double y = ((tp.hi - mid) + tp.lo) * inv_w, y2 = y + y;
        double t0 = 1.0, t1 = y;
        #pragma unroll
        for (int m = 0; m < KC; ++m) {
            acc[2 * m] = __builtin_fma(xr, t0, acc[2 * m]);
            acc[2 * m + 1] = __builtin_fma(xi, t0, acc[2 * m + 1]);
            const double t2 = __builtin_fma(y2, t1, -t0);
            t0 = t1;
            t1 = t2;
        }
    }
    return wave_sums<2 * KC>(acc, s, lane);
}

// The K-term instance for an item's block.
template <class F>
__device__ __forceinline__ void rank_dispatch(int K, F&& f)
{
    if (K <= 12) f(std::integral_constant<int, 12>());
    else if (K <= 16) f(std::integral_constant<int, 16>());
    else if (K <= 20) f(std::integral_constant<int, 20>());
    else f(std::integral_constant<int, 24>());
}

// Workgroups 0 .. n_ritems - 1: a large item each; then four small items
// each, one per wave.
//
// A large item (four waves) within one or two panels: the waves share each
// panel's points.  Over more panels: a panel per wave in turn.  A small item's
// wave takes its panels one after the other, kRankWavePanels at most: a panel
// is more than a microsecond however few its points, and 300 log-spaced points
// of order 1.5 in one block of 40 panels kept one wave busy for 50 us of a
// pass of 121 (about 40 us less with four waves).
__device__ __forceinline__ void rank_moments_body(const PlanDev& P, int bid)
{
    __shared__ double s_m[kRankWaves][2 * kRankK];
    __shared__ double s_wave[kRankWaves * (kRankK / 2 * 64)];
    const bool large = bid < P.n_ritems;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = large ? bid : (bid - P.n_ritems) * kRankWaves + wave;
    if (!large && i >= P.n_rsmall) return;
    const RankItem I = P.rlist[large ? i : P.rlist_cap - 1 - i];
    const ABlock& A = P.ab[I.blk];
    const int K = A.K;
    const RankCols B{A.C, A.D, A.r0, A.cw, A.pc, A.cpan0};
    double* s = s_wave + wave * (kRankK / 2 * 64);
    const bool shared = large && I.nq <= 2;
    const int first = large && !shared ? wave : 0, step = large && !shared ? kRankWaves : 1;
    rank_dispatch(K, [&](auto kc) {
        constexpr int KC = decltype(kc)::value;
        for (int h = first; h < I.nq; h += step) {
            const int q = I.q0 + h;
            int ka = I.ka, kb = I.kb;
            if (B.pc > 1) {
                const Panel T = P.cpans[B.cpan0 + q];
                ka = T.ka > ka ? T.ka : ka;
                kb = T.kb < kb ? T.kb : kb;
            }
            double* out = (double*)(P.rmom + (int64_t)(I.slot + q) * kRankK);
            const double v = rank_moments_wave<KC>(P, B, q, shared ? ka + 64 * wave : ka, shared ? kRankWaves : 1, kb, s);
            if (!shared) {
                if (lane < 2 * KC) out[lane] = v;
                continue;
            }
            if (lane < 2 * KC) s_m[wave][lane] = v;
            __syncthreads();
            if (threadIdx.x < 2 * KC) {
                double t = s_m[0][lane];
                #pragma unroll
                for (int w = 1; w < kRankWaves; ++w) t += s_m[w][lane];
                out[lane] = t;
            }
            __syncthreads();
        }
    });
}

static inline int rank_moments_blocks(const Summary& S) { return S.n_ritems + (S.n_rsmall + kRankWaves - 1) / kRankWaves; }

__global__ __launch_bounds__(64 * kRankWaves) void k_rank_moments(PlanDev P) { rank_moments_body(P, blockIdx.x); }

__global__ __launch_bounds__(64 * kRankWaves) void k_rank_moments_many(const PlanDev* __restrict__ plans,
                                                                       const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    rank_moments_body(plan_of(plans, w.t), w.g0);
}

// Sum over items i0 .. i1 - 1 (step `step`) of moment `lane` of panel `pan`,
// in item order within eight running sums.
__device__ __forceinline__ double rank_moment_sum(const PlanDev& P, int pan, int i0, int i1, int step, int lane)
{
    const double* __restrict__ src = (const double*)(P.rmom + (int64_t)pan * kRankK) + lane;
    constexpr int kStride = 2 * kRankK;
    double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int i = i0;
    for (; i + 7 * step < i1; i += 8 * step) {
        #pragma unroll
        for (int u = 0; u < 8; ++u) a[u] += src[(int64_t)(i + u * step) * kStride];
    }
    #pragma unroll
    for (int u = 0; u < 7; ++u)
        if (i + u * step < i1) a[u] += src[(int64_t)(i + u * step) * kStride];
    return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}

// v of lane `src` (the same in every lane), through the scalar unit.
__device__ __forceinline__ double read_lane(double v, int src)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, src), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | lo);
}

// Lane s < K: weight_s = (1/K) (t_0 + 2 sum_{m>=1} t_m cos(pi m (2 s + 1) / (2 K))),
// t the moment of lane 2m (real) and 2m + 1 (imaginary).
__device__ __forceinline__ double2 rank_nodal_weight(const double* __restrict__ tab, int K, double t, int lane)
{
    const int s = lane < K ? lane : K - 1;
    double wr = 0.0, wi = 0.0;
    for (int m0 = 0; m0 < K; m0 += 4) {      // m = 0 with factor 1 (taken off below)
        double c[4];
        #pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = tab[(m0 + u) * K + s];
        #pragma unroll
        for (int u = 0; u < 4; ++u) {
            wr = __builtin_fma(read_lane(t, 2 * (m0 + u)), c[u], wr);
            wi = __builtin_fma(read_lane(t, 2 * (m0 + u) + 1), c[u], wi);
        }
    }
    const double inv = 1.0 / K;
    return make_double2((wr + wr - read_lane(t, 0)) * inv, (wi + wi - read_lane(t, 1)) * inv);
}

// Lane m < K: v_m = (2 - [m = 0]) / K sum_t u_t cos(pi m (2 t + 1) / (2 K)),
// u_t in lane t.
__device__ __forceinline__ void rank_store_coefs(const PlanDev& P, const double* __restrict__ tab, int K, int pan,
                                                 double ur, double ui, int lane)
{
    const int m = lane < K ? lane : K - 1;
    const double* __restrict__ col = tab + K * K + m;
    double vr = 0.0, vi = 0.0;
    for (int h0 = 0; h0 < K; h0 += 4) {
        double c[4];
        #pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = col[(h0 + u) * K];
        #pragma unroll
        for (int u = 0; u < 4; ++u) {
            vr = __builtin_fma(read_lane(ur, h0 + u), c[u], vr);
            vi = __builtin_fma(read_lane(ui, h0 + u), c[u], vi);
        }
    }
    const double f = (m == 0 ? 1.0 : 2.0) / K;
    if (lane < K) P.rcoef[(int64_t)pan * kRankK + lane] = make_double2(vr * f, vi * f);
}

// Hankel's terms H(x), from MP >= M pairs of channel factors held in (scalar)
// registers (the factors beyond 2M are zero); MP = 0: from memory.
template <int MP>
struct Hankel {
    const PlanDev& P;
    double f[MP > 0 ? 2 * MP : 1];
    __device__ __forceinline__ Hankel(const PlanDev& plan) : P(plan)
    {
        #pragma unroll
        for (int i = 0; i < 2 * MP; ++i) f[i] = plan.chan[i];
    }
    __device__ __forceinline__ void at(double x, double& hr, double& hi) const
    {
        const double inv = rcp_refined(x), inv2 = inv * inv;
        if constexpr (MP > 0) {
            hr = f[2 * MP - 2];
            hi = f[2 * MP - 1];
            #pragma unroll
            for (int l = MP - 2; l >= 0; --l) {
                hr = __builtin_fma(hr, inv2, f[2 * l]);
                hi = __builtin_fma(hi, inv2, f[2 * l + 1]);
            }
        } else {
            hr = 0.0;
            hi = 0.0;
            for (int l = P.M - 1; l >= 0; --l) {
                hr = __builtin_fma(hr, inv2, P.chan[2 * l]);
                hi = __builtin_fma(hi, inv2, P.chan[2 * l + 1]);
            }
        }
        hi *= inv;
    }
};

// The instance for a plan's M: 4 and 8 pairs in registers, beyond from memory.
template <class F>
__device__ __forceinline__ void hankel_dispatch(int M, F&& f)
{
    if (M <= 4) f(std::integral_constant<int, 4>());
    else if (M <= 8) f(std::integral_constant<int, 8>());
    else f(std::integral_constant<int, 0>());
}

// e^{i a b}, to the rounding of a and b's low parts
__device__ __forceinline__ void rank_phase(dd a, dd b, double& c, double& s)
{
    const dd ph = two_prod(a.hi, b.hi);
    cis_dd(ph.hi, __builtin_fma(a.hi, b.lo, __builtin_fma(a.lo, b.hi, ph.lo)), c, s);
}

// Nodal weights of one panel of points of a block of several panels or many
// items: the four waves each sum every fourth item, the four sums are added
// in order, and the first wave forms the weights.
__device__ __forceinline__ void rank_weights_panel(const PlanDev& P, const Panel& T, double (*s_t)[64])
{
    const ABlock B = P.ab[T.blk];
    const int pan = B.cpan0 + T.q;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, K = B.K;
    double t = 0.0;
    if (T.kb > T.ka && lane < 2 * K) {
        const int i0 = B.item0 + (T.ka - B.k0) / P.spread_chunk, i1 = B.item0 + (T.kb - 1 - B.k0) / P.spread_chunk + 1;
        t = rank_moment_sum(P, pan, i0 + wave, i1, 4, lane);
    }
    s_t[wave][lane] = t;
    __syncthreads();
    if (wave > 0) return;
    t = ((s_t[0][lane] + s_t[1][lane]) + s_t[2][lane]) + s_t[3][lane];
    const double2 w = rank_nodal_weight(P.rank_tab + rank_tab_off(K), K, t, lane);
    if (lane < K) P.rwts[(int64_t)pan * kRankK + lane] = w;
}

// One panel of frequencies of a block of one panel of points and few items,
// a wave: moments summed, weights, translation, coefficients.  Groups of 8,
// 16 or 32 lanes hold the frequency nodes and share the point nodes.
__device__ __forceinline__ void rank_translate_single(const PlanDev& P, const Panel& T)
{
    const ABlock B = P.ab[T.blk];
    const int pan = B.rpan0 + T.q;
    const int lane = threadIdx.x & 63, K = B.K;
    const double* __restrict__ tab = P.rank_tab + rank_tab_off(K);   // row m = 1: the nodes
    const double tm = lane < 2 * K ? rank_moment_sum(P, B.cpan0, B.item0, B.item0 + B.nitems, 1, lane) : 0.0;
    const double2 w = rank_nodal_weight(tab, K, tm, lane);
    const int logt = K <= 8 ? 3 : K <= 16 ? 4 : 5, groups = 64 >> logt;
    const int t = lane & ((1 << logt) - 1), g = lane >> logt;
    const dd a = two_sum(rank_mid(T.q, B.pr, B.rw), B.rw * tab[K + (t < K ? t : K - 1)]);
    const double om = B.D + a.hi;
    double ur = 0.0, ui = 0.0;
    hankel_dispatch(P.M, [&](auto mp) {
        const Hankel<decltype(mp)::value> H(P);
        for (int s0 = 0; s0 < K; s0 += groups) {
            const int s = s0 + g < K ? s0 + g : K - 1;
            double wr = __shfl(w.x, s), wi = __shfl(w.y, s);
            if (s0 + g >= K) { wr = 0.0; wi = 0.0; }
            const double d = B.cw * tab[K + s];
            double hr, hi, c, sn;
            H.at(om * (B.C + d), hr, hi);
            rank_phase(a, dd{d, 0.0}, c, sn);
            const double fr = __builtin_fma(hr, c, -hi * sn), fi = __builtin_fma(hr, sn, hi * c);
            ur = __builtin_fma(fr, wr, __builtin_fma(-fi, wi, ur));
            ui = __builtin_fma(fr, wi, __builtin_fma(fi, wr, ui));
        }
    });
    for (int o = 32; o >= (1 << logt); o >>= 1) { ur += __shfl_xor(ur, o); ui += __shfl_xor(ui, o); }
    rank_store_coefs(P, tab, K, pan, ur, ui, lane);
}

// Workgroups 0 .. n_wmulti - 1: the weights of a panel of points each; then
// four panels of frequencies of one-wave blocks each, one per wave.
__device__ __forceinline__ void rank_weights_body(const PlanDev& P, int bid)
{
    __shared__ double s_t[4][64];
    if (bid < P.n_wmulti) {
        rank_weights_panel(P, P.wlist[bid], s_t);
        return;
    }
    const int i = (bid - P.n_wmulti) * 4 + (threadIdx.x >> 6);
    if (i < P.n_tsingle) rank_translate_single(P, P.tlist[i]);
}

static inline int rank_weights_blocks(const Summary& S) { return S.n_wmulti + (S.n_tsingle + 3) / 4; }

__global__ __launch_bounds__(256) void k_rank_weights(PlanDev P) { rank_weights_body(P, blockIdx.x); }

__global__ __launch_bounds__(256) void k_rank_weights_many(const PlanDev* __restrict__ plans,
                                                           const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    rank_weights_body(plan_of(plans, w.t), w.g0);
}

// One panel of frequencies of the other rank blocks, a workgroup of 512
// threads: 16 groups of 32 lanes, a lane per frequency node.  A group takes
// point nodes s of every panel; from panel to panel the phase turns by the
// same angle (restarted every 8 panels, so that the rotations' rounding stays
// at that of one phase).
constexpr int kRankTransThreads = 512;

__device__ __forceinline__ void rank_translate_body(const PlanDev& P, int bid)
{
    // the block's nodal weights first, the groups' sums afterwards
    __shared__ double2 s_w[kRankPanels * kRankK];
    static_assert(kRankPanels * kRankK >= kRankTransThreads, "room for the groups' sums");
    const Panel T = P.tlist[P.tlist_cap - 1 - bid];
    const ABlock B = P.ab[T.blk];
    const int pan = B.rpan0 + T.q;
    constexpr int kGroups = kRankTransThreads / 32;
    const int K = B.K, t = threadIdx.x & 31, g = threadIdx.x >> 5;
    const double* __restrict__ tab = P.rank_tab + rank_tab_off(K);
    const double2* __restrict__ wts = P.rwts + (int64_t)B.cpan0 * kRankK;
    for (int e = threadIdx.x; e < B.pc * kRankK; e += kRankTransThreads) s_w[e] = wts[e];
    const dd a = two_sum(rank_mid(T.q, B.pr, B.rw), B.rw * tab[K + (t < K ? t : K - 1)]);
    const double om = B.D + a.hi;
    double er, ei;
    rank_phase(a, dd{2.0 * B.cw, 0.0}, er, ei);
    __syncthreads();
    double ur = 0.0, ui = 0.0;
    // (node, run of 8 panels) pairs, dealt to the groups in turn
    const int runs = (B.pc + 7) >> 3;
    hankel_dispatch(P.M, [&](auto mp) {
        const Hankel<decltype(mp)::value> H(P);
        for (int j = g; j < K * runs; j += kGroups) {
            const int run = j / K, s = j - run * K;
            const int q1 = 8 * run + 8 < B.pc ? 8 * run + 8 : B.pc;
            const double d = B.cw * tab[K + s];
            double c, sn;
            rank_phase(a, two_sum(rank_mid(8 * run, B.pc, B.cw), d), c, sn);
            for (int q = 8 * run; q < q1; ++q) {
                double hr, hi;
                H.at(om * (B.C + (rank_mid(q, B.pc, B.cw) + d)), hr, hi);
                const double2 w = s_w[q * kRankK + s];
                const double fr = __builtin_fma(hr, c, -hi * sn), fi = __builtin_fma(hr, sn, hi * c);
                ur = __builtin_fma(fr, w.x, __builtin_fma(-fi, w.y, ur));
                ui = __builtin_fma(fr, w.y, __builtin_fma(fi, w.x, ui));
                const double cn = __builtin_fma(c, er, -sn * ei);
                sn = __builtin_fma(c, ei, sn * er);
                c = cn;
            }
        }
    });
    __syncthreads();
    double2* s_sum = s_w;
    s_sum[threadIdx.x] = make_double2(ur, ui);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    ur = 0.0; ui = 0.0;
    for (int h = 0; h < kGroups; ++h) {
        const double2 v = s_sum[32 * h + t];
        ur += v.x;
        ui += v.y;
    }
    rank_store_coefs(P, tab, K, pan, ur, ui, threadIdx.x);
}

__global__ __launch_bounds__(kRankTransThreads) void k_rank_translate(PlanDev P) { rank_translate_body(P, blockIdx.x); }

__global__ __launch_bounds__(kRankTransThreads) void k_rank_translate_many(const PlanDev* __restrict__ plans,
                                                                           const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    rank_translate_body(plan_of(plans, w.t), w.g0);
}

// A rank block's contribution at frequency om.  UNI: the block is the same in
// every lane; where the panel is too, its coefficients come through the
// scalar unit.
__device__ __forceinline__ double rank_series(const double2* __restrict__ v, int K, double eta, double cr, double ci)
{
    double t0 = 1.0, t1 = eta, ar = 0.0, ai = 0.0;
    const double e2 = eta + eta;
    for (int m = 0; m < K; m += 4) {
        #pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double2 c = v[m + u];
            ar = __builtin_fma(c.x, t0, ar);
            ai = __builtin_fma(c.y, t0, ai);
            const double t2 = __builtin_fma(e2, t1, -t0);
            t0 = t1;
            t1 = t2;
        }
    }
    return __builtin_fma(cr, ar, -ci * ai);
}

template <bool UNI>
__device__ __forceinline__ double rank_eval(const PlanDev& P, const ABlock& B, double om)
{
    const double rs = rsqrt_refined(om * B.r0);
    const dd pc = two_prod(om, B.C);
    const dd ph = two_sum(pc.hi, P.phi_hi);
    double cr, ci;
    cis_dd(ph.hi, ph.lo + pc.lo + P.phi_lo, cr, ci);
    const double inv = B.rw > 0.0 ? rcp_refined(B.rw) : 0.0;
    const dd a = two_sum(om, -B.D);
    int q = (int)(0.5 * __builtin_fma(a.hi, inv, (double)B.pr));
    q = q < 0 ? 0 : q > B.pr - 1 ? B.pr - 1 : q;
    const double eta = ((a.hi - rank_mid(q, B.pr, B.rw)) + a.lo) * inv;
    double v;
    if constexpr (UNI) {
        const int qu = __builtin_amdgcn_readfirstlane(q);
        if (__all(q == qu)) v = rank_series(P.rcoef + (int64_t)(B.rpan0 + qu) * kRankK, B.rK, eta, cr, ci);
        else v = rank_series(P.rcoef + (int64_t)(B.rpan0 + q) * kRankK, B.rK, eta, cr, ci);
    } else {
        v = rank_series(P.rcoef + (int64_t)(B.rpan0 + q) * kRankK, B.rK, eta, cr, ci);
    }
    return kSqrt2OverPi * rs * v;
}

// ---------------------------------------------------------------------------
// ES spreading of one chunk of an asymptotic block's points (type-3 NUFFT,
// step one).  Point k of the block carries the 2M channel weights
//   x_k^(p) = c_k (r0/r_k)^(p+1/2) e^{i D (r_k - C)},   p = 0 .. 2M-1
// (the weights c_k r_k^(-p-1/2) of Sec. 3.2, normalised by the block's
// smallest point r0, times the type-3 pre-phase), placed at grid coordinate
// u_k = (r_k - C)/h.  Cell l receives sum_k x_k^(p) ES((l - u_k) 2/w).
//
// The points of an item are taken in sub-chunks of kSpreadSub.
// Phase 1: one thread per point forms the offset r - C and the phase
// D (r - C) as double-doubles (so the kernel position and the phase are exact
// to FP64 relative to themselves), the weight and the ratio r0 / r, the first
// cell l0 it reaches, and its w kernel values from the polynomial pieces
// (sums of coefficients common to all lanes times powers of the point's
// offset), all into LDS.
// Phase 2: threads own (cell, slice) pairs; the points reaching cell l are
// those with l - w < l0 <= l, a contiguous range (points are sorted), from a
// list of the first point of every cell (a binary search where the sub-chunk
// spans more than kSpreadSpan cells); slices of one cell are adjacent lanes and are summed with
// cross-lane shuffles after the last sub-chunk.
//
// Where points are sparse an item's cells take several turns of the threads.
// A turn only takes the sub-chunks that reach its cells, and the last one of
// a turn, which also reaches the next turn's, is kept in LDS: every sub-chunk
// goes through phase 1 about once, whatever the number of turns.  (All of an
// item's sub-chunks in every turn took 462 us for the 1e6 log-spaced points of
// order 0, one point a cell, and take 98 so, 73 with the list in place of
// searches; 276, 147 and 145 at the first 1e6 zeros of J_0.)  Where items are
// few, P.spread_turns workgroups share an item, every so many turns each (of
// fewer cells where the item has few): 20000 points of a radial transform 57
// -> 18 us, 5229 of order 18 70 -> 18, 1e5 of order 0 58 -> 35.
// ---------------------------------------------------------------------------
constexpr int kSpreadSub = 256;
constexpr int kSpreadSpan = 512;     // first cells of a sub-chunk that are listed (1 KB; 4 KB cost a workgroup a CU)

// T is the type of the weights, kernel values and channel sums: double, or
// float in the FP32-spreading mode (positions and phases stay double-double
// either way); partials are stored as the matching two-component vector.
// One point of a sub-chunk in LDS: weight (real, imaginary), ratio r0 / r and
// first cell reached, read with two (one for float) 16-byte loads.
template <typename T>
struct alignas(16) SpreadPoint {
    T wr, wi, q;
    int32_t l0;
};

// Dynamic LDS of k_spread: kSpreadSub point records, then w kernel values per point.
template <typename T>
constexpr size_t spread_lds_bytes(int w)
{
    return (size_t)kSpreadSub * (sizeof(SpreadPoint<T>) + (size_t)w * sizeof(T));
}

// One point of a block for spreading: weight c sqrt(r0/r) e^{i D (r - C)}
// (real, imaginary), ratio q = r0 / r, first cell reached l0, and the kernel
// argument s = 2 f - 1 of the polynomial pieces.  The phase is a double-double
// product; the cell position (r - C) / h is formed from the double-double
// difference (the scaling by h is exact).
struct PointEval {
    double wr, wi, q, s;
    int l0;
};

// First cell reached by the point at offset tp = r - C; frac: its distance
// from the cell before.
__device__ __forceinline__ int first_cell(const dd& tp, double inv_h, double hw, double& frac)
{
    // u - w/2 = (tp.hi + tp.lo)/h - w/2
    dd a = two_sum(tp.hi * inv_h, -hw);
    double lo = a.lo + tp.lo * inv_h;
    double fl = floor(a.hi);
    frac = (a.hi - fl) + lo;          // a.hi - fl is exact
    if (frac < 0.0) { fl -= 1.0; frac += 1.0; }
    else if (frac >= 1.0) { fl += 1.0; frac -= 1.0; }
    return (int)fl + 1;
}

__device__ __forceinline__ PointEval eval_point(const ABlock& B, double r, double c, double inv_h, double hw)
{
    dd tp = two_sum(r, -B.C);
    dd ph = two_prod(B.D, tp.hi);
    double cth, sth;
    cis_dd(ph.hi, __builtin_fma(B.D, tp.lo, ph.lo), cth, sth);
    // q = r0 / r in (0, 1] and its square root through the refined hardware
    // estimates (within an ulp or two; no IEEE division or square root)
    const double q = B.r0 * rcp_refined(r);
    const double w0 = c * (q * rsqrt_refined(q));
    double frac;
    const int l0 = first_cell(tp, inv_h, hw, frac);
    PointEval e;
    e.wr = w0 * cth;
    e.wi = w0 * sth;
    e.q = q;
    e.l0 = l0;
    e.s = 1.0 - 2.0 * frac;                  // s = 2 f - 1, f = 1 - frac
    return e;
}

__device__ __forceinline__ double typed_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float typed_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <int NCH, typename T>
__device__ __forceinline__ void spread_body(const PlanDev& P, int bid)
{
    using T2 = typename std::conditional<std::is_same<T, float>::value, float2, double2>::type;
    T2* part = reinterpret_cast<T2*>(P.part);
    const double* __restrict__ cs = P.cs;
    const double* __restrict__ es_poly = P.es_poly;
    extern __shared__ double4 spread_lds[];
    SpreadPoint<T>* s_pt = reinterpret_cast<SpreadPoint<T>*>(spread_lds);
    T* s_k = reinterpret_cast<T*>(s_pt + kSpreadSub);
    // the items not spread on the matrix cores, from the back of the order
    const int share = P.spread_turns;
    const Item I = P.aitems[P.alist[P.n_aitems - 1 - bid / share]];
    const ABlock B = P.ab[I.blk];
    const int tid = threadIdx.x;
    const int w = P.w;
    const double hw = 0.5 * w;
    const double inv_h = 1.0 / B.h;      // exact: h is a power of two
    const int sub_n = I.sub_n;
    int slices = 1;
    // (FP32 sums keep the slices of one workgroup, and so their order)
    const int threads = std::is_same<T, float>::value ? 256 : 256 * share;
    while (slices < 64 && slices * 2 * sub_n <= threads) slices <<= 1;
    const int cells_par = 256 / slices;
    auto cell_of = [&](int k) {
        double frac;
        return first_cell(two_sum(P.rs[k], -B.C), inv_h, hw, frac);
    };
    int k_begin = I.ka, in_lds = -1;     // first sub-chunk that reaches the turn's cells; the one in LDS
    __shared__ uint16_t s_start[kSpreadSpan];
    int l_first = 0, l_last = 0;         // first cells of its first and last point
    for (int cbase = bid % share * cells_par; cbase < sub_n; cbase += share * cells_par) {
        const int l_lo = I.sub_lo + cbase;
        const int l_hi = I.sub_lo + (cbase + cells_par < sub_n ? cbase + cells_par : sub_n) - 1;
        while (k_begin + kSpreadSub < I.kb && cell_of(k_begin + kSpreadSub - 1) <= l_lo - w) k_begin += kSpreadSub;
        const int cell = cbase + tid / slices;
        const int sl = tid & (slices - 1);
        const int l = I.sub_lo + cell;
        T ar[NCH], ai[NCH];
        #pragma unroll
        for (int p = 0; p < NCH; ++p) { ar[p] = T(0); ai[p] = T(0); }
        for (int k0 = k_begin; k0 < I.kb; k0 += kSpreadSub) {
            if (cell_of(k0) > l_hi) break;
            const int np = (I.kb - k0) < kSpreadSub ? (I.kb - k0) : kSpreadSub;
            // every thread evaluates a point (the last one when tid >= np) so
            // that the coefficient loads below stay wave-uniform (scalar)
            if (k0 != in_lds) {
                __syncthreads();
                const bool own = tid < np;
                const int k = k0 + (own ? tid : np - 1);
                const PointEval e = eval_point(B, P.rs[k], cs[k], inv_h, hw);
                if (own) {
                    SpreadPoint<T> rec;
                    rec.wr = (T)e.wr;
                    rec.wi = (T)e.wi;
                    rec.q = (T)e.q;
                    rec.l0 = e.l0;
                    s_pt[tid] = rec;
                }
                const double sv = e.s;
                // powers s^0 .. s^h once per point (h = ceil(kEsDeg / 2));
                // each piece is then sum_{d<=h} c_d s^d + s^h sum_{d>h} c_d
                // s^(d-h), with the (scalar) coefficients as multiplicands
                constexpr int kHalf = (kEsDeg + 1) / 2;
                double spow[kHalf + 1];
                spow[0] = 1.0;
                #pragma unroll
                for (int d = 1; d <= kHalf; ++d) spow[d] = spow[d - 1] * sv;
                T* kv = s_k + tid * w;
                for (int t = 0; t < w; ++t) {
                    const double* cf = es_poly + t * (kEsDeg + 1);
                    double vlo = cf[0], vhi = cf[kHalf + 1] * spow[1];
                    #pragma unroll
                    for (int d = 1; d <= kHalf; ++d) vlo = __builtin_fma(cf[d], spow[d], vlo);
                    #pragma unroll
                    for (int d = kHalf + 2; d <= kEsDeg; ++d) vhi = __builtin_fma(cf[d], spow[d - kHalf], vhi);
                    double v = __builtin_fma(spow[kHalf], vhi, vlo);
                    if (own) kv[t] = (T)v;
                }
                in_lds = k0;
                __syncthreads();
                // the first point from each cell on
                l_first = s_pt[0].l0;
                l_last = s_pt[np - 1].l0;
                if (l_last - l_first < kSpreadSpan) {
                    if (tid < np)
                        for (int a = tid > 0 ? s_pt[tid - 1].l0 + 1 : l_first; a <= s_pt[tid].l0; ++a)
                            s_start[a - l_first] = (uint16_t)tid;
                    __syncthreads();
                }
            }
            if (cell < sub_n) {
                // points with l0 in (l - w, l]
                auto points_to = [&](int b) {            // points with l0 <= b
                    if (b < l_first) return 0;
                    if (b >= l_last) return np;
                    if (l_last - l_first < kSpreadSpan) return (int)s_start[b + 1 - l_first];
                    int lo = 0, hi = np;
                    while (lo < hi) { int mid = (lo + hi) >> 1; if (s_pt[mid].l0 <= b) lo = mid + 1; else hi = mid; }
                    return lo;
                };
                const int first = points_to(l - w), last = points_to(l);
                for (int i = first + sl; i < last; i += slices) {
                    const SpreadPoint<T> rec = s_pt[i];
                    T phi = s_k[i * w + (l - rec.l0)];
                    const T vr = phi * rec.wr, vi = phi * rec.wi;
                    const T q = rec.q;
                    // one chain of powers q^p serves both parts
                    T qp = T(1);
                    #pragma unroll
                    for (int p = 0; p < NCH; ++p) {
                        ar[p] = typed_fma(vr, qp, ar[p]);
                        ai[p] = typed_fma(vi, qp, ai[p]);
                        qp *= q;
                    }
                }
            }
        }
        for (int o = slices >> 1; o >= 1; o >>= 1) {
            #pragma unroll
            for (int p = 0; p < NCH; ++p) {
                ar[p] += __shfl_xor(ar[p], o);
                ai[p] += __shfl_xor(ai[p], o);
            }
        }
        if (cell < sub_n && sl == 0) {
            T2* dst = part + I.off + (int64_t)cell * NCH;
            #pragma unroll
            for (int p = 0; p < NCH; ++p) { dst[p].x = ar[p]; dst[p].y = ai[p]; }
        }
    }
}

template <int NCH, typename T>
__global__ __launch_bounds__(256) void k_spread(PlanDev P)
{
    spread_body<NCH, T>(P, blockIdx.x);
}

template <int NCH, typename T>
__global__ __launch_bounds__(256) void k_spread_many(const PlanDev* __restrict__ plans,
                                                     const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    spread_body<NCH, T>(plan_of(plans, w.t), w.g0);
}

// ---------------------------------------------------------------------------
// Spreading on the matrix cores (FP64), for items whose points reach the grid
// from at most kSpreadAnchors first cells (dense items: many points per cell)
// and, in a launch of their own with room for more cell sums, from at most
// kSpreadAnchorsMed (medium items: tens of points per cell).
// With the points of an item split by their first cell a (anchor), the
// item's partial subgrid is
//   G[a + t][col] = sum over anchors a, over points k with anchor a, of
//                   phi_t(s_k) V_k[col],
// t the tap (0 .. w-1), phi_t the kernel's polynomial piece for tap t and
// V_k[2p + {0,1}] = (re, im) of c_k sqrt(q_k) e^{i D (r_k - C)} q_k^p.  For
// each anchor this is a (16 taps) x (points) x (16 NCT columns) product: one
// v_mfma_f64_16x16x4f64 per four points and column tile.  In an MFMA step,
// lane (row = lane % 16, k = lane / 16) supplies A[row][k] = phi_row(s) of
// point k, evaluated in the lane with the coefficients of piece `row` held in
// its registers, and B[k][col] = V_k[col] (col = lane % 16) from LDS; element
// v of the accumulator is D[lane / 16 + 4 v][lane % 16].
//
// The four waves of a workgroup share one item: wave v takes the steps of 64
// points starting at ka + (4 j + v) 64.  Points are sorted, so the anchors a
// wave meets only increase: it keeps one tile for its current anchor and adds
// it into its own cell sums in LDS when the anchor changes.  At the end the
// four waves' cell sums are added in a fixed order, so the result does not
// depend on timing.
// ---------------------------------------------------------------------------
typedef double v4d __attribute__((ext_vector_type(4)));

// 16-column tiles of the channel columns (re, im of 8 channels each): one
// to four, channel counts up to kMfmaMaxChannels
template <int NCH>
constexpr int kSpreadTiles = (2 * NCH + 15) / 16;

template <int NCH, int ANCH = kSpreadAnchors>
struct SpreadMfma {
    static constexpr int NCT = kSpreadTiles<NCH>;
    static constexpr int NC = 16 * NCT;            // real columns of the tiles (re, im of 8 NCT channels)
    static constexpr int VS = 2 * NCH + 1;         // LDS stride of a point's 2 NCH columns (odd: conflict-free writes)
    static constexpr int GC = ANCH + 15;           // cells an item's anchor tiles reach
    // points per step: 64, 32 with two column tiles, 16 with three or four,
    // so that the wider point records still fit (three workgroups per compute
    // unit at two tiles, two at four)
    static constexpr int WPTS = NCT > 2 ? 16 : NCT > 1 ? 32 : 64;
    // a point: its columns, its s and its anchor
    static constexpr size_t point_bytes = (VS + 1) * sizeof(double) + sizeof(int32_t);
    static constexpr size_t fold_bytes = (size_t)GC * NC * sizeof(double);   // the wave's cell sums
    static constexpr size_t wave_bytes = ((size_t)WPTS * point_bytes + 15) / 16 * 16 + fold_bytes;
    static constexpr size_t lds_bytes = 4 * wave_bytes;   // the workgroup's four waves
};

// Points g_lo .. g_hi-1 of the step (g_lo a multiple of 8) into the tile of
// anchor a, two groups of four points per iteration (two independent kernel
// evaluations).  Lanes past np take B = 0; with MASK, points of other anchors
// take A = 0.
template <int NCH, bool MASK>
__device__ __forceinline__ void spread_mfma_run(v4d (&acc)[kSpreadTiles<NCH>], const double* s_v,
                                                const double* s_s, const int32_t* s_d,
                                                const double (&cf)[kEsDeg + 1], int g_lo, int g_hi, int np,
                                                int col, int kq, int a)
{
    constexpr int NCT = SpreadMfma<NCH>::NCT, VS = SpreadMfma<NCH>::VS;
    for (int g = g_lo; g < g_hi; g += 8) {
        const int i0 = g + kq, i1 = g + 4 + kq;
        const bool v0 = i0 < np, v1 = i1 < np;
        const int j0 = v0 ? i0 : g, j1 = v1 ? i1 : g;
        double b0[NCT], b1[NCT];
        #pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            const bool on = ct * 16 + 16 <= 2 * NCH || ct * 16 + col < 2 * NCH;   // columns past 2 NCH are zero
            b0[ct] = (v0 && on) ? s_v[j0 * VS + ct * 16 + col] : 0.0;
            b1[ct] = (v1 && on) ? s_v[j1 * VS + ct * 16 + col] : 0.0;
        }
        const double s0 = s_s[j0], s1 = s_s[j1];
        double p0 = cf[kEsDeg], p1 = cf[kEsDeg];
        #pragma unroll
        for (int q = kEsDeg - 1; q >= 0; --q) {
            p0 = __builtin_fma(p0, s0, cf[q]);
            p1 = __builtin_fma(p1, s1, cf[q]);
        }
        if (MASK) {
            if (s_d[j0] != a) p0 = 0.0;
            if (s_d[j1] != a) p1 = 0.0;
        }
        #pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(p0, b0[ct], acc[ct], 0, 0, 0);
            acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(p1, b1[ct], acc[ct], 0, 0, 0);
        }
    }
}

// A full step of one anchor: all WPTS points valid and none masked, the same
// products in the same order as spread_mfma_run.  The loop is unrolled, so
// every LDS offset is a constant and no point needs a validity test.
template <int NCH>
__device__ __forceinline__ void spread_mfma_run_full(v4d (&acc)[kSpreadTiles<NCH>], const double* s_v,
                                                     const double* s_s, const double (&cf)[kEsDeg + 1], int col,
                                                     int kq)
{
    constexpr int NCT = SpreadMfma<NCH>::NCT, VS = SpreadMfma<NCH>::VS, WPTS = SpreadMfma<NCH>::WPTS;
    const double* v = s_v + kq * VS + col;
    const double* sp = s_s + kq;
    #pragma unroll
    for (int g = 0; g < WPTS; g += 8) {
        double b0[NCT], b1[NCT];
        #pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            const bool on = ct * 16 + 16 <= 2 * NCH || ct * 16 + col < 2 * NCH;   // columns past 2 NCH are zero
            b0[ct] = on ? v[g * VS + ct * 16] : 0.0;
            b1[ct] = on ? v[(g + 4) * VS + ct * 16] : 0.0;
        }
        const double s0 = sp[g], s1 = sp[g + 4];
        double p0 = cf[kEsDeg], p1 = cf[kEsDeg];
        #pragma unroll
        for (int q = kEsDeg - 1; q >= 0; --q) {
            p0 = __builtin_fma(p0, s0, cf[q]);
            p1 = __builtin_fma(p1, s1, cf[q]);
        }
        #pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(p0, b0[ct], acc[ct], 0, 0, 0);
            acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(p1, b1[ct], acc[ct], 0, 0, 0);
        }
    }
}

// Adds the finished tile of anchor a into the wave's cell sums (row t of the
// tile to cell a + t) and clears it.
template <int NCH>
__device__ __forceinline__ void spread_mfma_flush(v4d (&acc)[kSpreadTiles<NCH>], double* s_g, int col, int kq, int a)
{
    constexpr int NCT = SpreadMfma<NCH>::NCT, NC = SpreadMfma<NCH>::NC;
    #pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        #pragma unroll
        for (int v = 0; v < 4; ++v) s_g[(a + kq + 4 * v) * NC + ct * 16 + col] += acc[ct][v];
        acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
    }
    wave_sync();   // the next anchor's cells overlap this one's in other lanes
}

// Item alist[slot] of the plan, with LDS for anchors up to ANCH.
template <int NCH, int ANCH>
__device__ __forceinline__ void spread_mfma_item(const PlanDev& P, int slot, double4* spread_lds)
{
    const double* __restrict__ cs = P.cs;
    const double* __restrict__ es_poly = P.es_poly;
    double2* __restrict__ part = P.part;
    using SM = SpreadMfma<NCH, ANCH>;
    constexpr int NCT = SM::NCT, NC = SM::NC, VS = SM::VS, WPTS = SM::WPTS, GC = SM::GC;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char* base = reinterpret_cast<char*>(spread_lds) + wave * SM::wave_bytes;
    double* s_v = reinterpret_cast<double*>(base);
    double* s_s = s_v + WPTS * VS;
    int32_t* s_d = reinterpret_cast<int32_t*>(s_s + WPTS);
    double* s_g = reinterpret_cast<double*>(base + SM::wave_bytes - SM::fold_bytes);
    const Item I = P.aitems[P.alist[slot]];
    const ABlock B = P.ab[I.blk];
    const int col = lane & 15, kq = lane >> 4;
    const int w = P.w;
    const double hw = 0.5 * w;
    const double inv_h = 1.0 / B.h;      // exact: h is a power of two
    // polynomial piece of tap `col` (row col of A); rows at or beyond w are zero
    double cf[kEsDeg + 1];
    #pragma unroll
    for (int d = 0; d <= kEsDeg; ++d) cf[d] = col < w ? es_poly[col * (kEsDeg + 1) + d] : 0.0;
    for (int e = lane; e < GC * NC; e += 64) s_g[e] = 0.0;
    v4d acc[NCT];
    #pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
    int cur = -1;                              // anchor of the tile in acc
    // the next step's point and weight are loaded while the current one is
    // multiplied
    int k0 = I.ka + wave * WPTS;
    double r_nx = 0.0, c_nx = 0.0;
    if (k0 + lane < I.kb) { r_nx = P.rs[k0 + lane]; c_nx = cs[k0 + lane]; }
    for (; k0 < I.kb; k0 += 4 * WPTS) {
        const int np = (I.kb - k0) < WPTS ? (I.kb - k0) : WPTS;
        const double r = r_nx, c = c_nx;
        const int kn = k0 + 4 * WPTS + lane;
        if (kn < I.kb) { r_nx = P.rs[kn]; c_nx = cs[kn]; }
        wave_sync();                              // the previous step's reads of the region are done
        int dm = 0;
        if (lane < np) {
            const PointEval e = eval_point(B, r, c, inv_h, hw);
            dm = e.l0 - I.sub_lo;
            s_d[lane] = dm;
            s_s[lane] = e.s;
            double vr = e.wr, vi = e.wi;
            double* v = s_v + lane * VS;
            #pragma unroll
            for (int p = 0; p < NCH; ++p) {
                v[2 * p] = vr;
                v[2 * p + 1] = vi;
                vr *= e.q;
                vi *= e.q;
            }
        }
        wave_sync();
        // the step's anchors run from its first point's to its last point's
        const int a_lo = __builtin_amdgcn_readfirstlane(dm);
        const int a_hi = __builtin_amdgcn_readlane(dm, np - 1);
        if (a_lo == a_hi) {
            if (a_lo != cur) {
                if (cur >= 0) spread_mfma_flush<NCH>(acc, s_g, col, kq, cur);
                cur = a_lo;
            }
            if (np == WPTS) spread_mfma_run_full<NCH>(acc, s_v, s_s, cf, col, kq);
            else spread_mfma_run<NCH, false>(acc, s_v, s_s, s_d, cf, 0, np, np, col, kq, cur);
        } else {
            // the points of anchor a are consecutive lanes (points are sorted):
            // only the groups of eight that hold them are multiplied
            for (int a = a_lo; a <= a_hi; ++a) {
                const uint64_t mine = __ballot(lane < np && dm == a);
                if (mine == 0) continue;
                if (a != cur) {
                    if (cur >= 0) spread_mfma_flush<NCH>(acc, s_g, col, kq, cur);
                    cur = a;
                }
                const int first = __builtin_ctzll(mine), last = 63 - __builtin_clzll(mine);
                spread_mfma_run<NCH, true>(acc, s_v, s_s, s_d, cf, first & ~7, last + 1, np, col, kq, a);
            }
        }
    }
    if (cur >= 0) spread_mfma_flush<NCH>(acc, s_g, col, kq, cur);
    __syncthreads();
    // item partial [cell][channel] (re, im): waves summed in order
    const double* g0 = reinterpret_cast<const double*>(reinterpret_cast<char*>(spread_lds) + SM::wave_bytes -
                                                       SM::fold_bytes);
    constexpr size_t wstride = SM::wave_bytes / sizeof(double);
    double* out = reinterpret_cast<double*>(part + I.off);
    constexpr int row_len = 2 * NCH;
    for (int e = tid; e < I.sub_n * row_len; e += 256) {
        const int cell = e / row_len, c = e - cell * row_len;
        const int k = cell * NC + c;
        out[e] = ((g0[k] + g0[wstride + k]) + g0[2 * wstride + k]) + g0[3 * wstride + k];
    }
}

// Up to 8 channels (one column tile) the dense kernel fits four waves per
// SIMD, with two tiles three.  ANCH = kSpreadAnchors: the dense items, from
// slot 0 of the item list; kSpreadAnchorsMed: the medium ones, after them.
template <int NCH, int ANCH>
__global__ __launch_bounds__(256) void k_spread_mfma(PlanDev P)
{
    __shared__ double4 lds[SpreadMfma<NCH, ANCH>::lds_bytes / sizeof(double4)];
    const int first = ANCH == kSpreadAnchors ? 0 : P.n_adense;
    spread_mfma_item<NCH, ANCH>(P, first + blockIdx.x, lds);
}

template <int NCH, int ANCH>
__global__ __launch_bounds__(256) void k_spread_mfma_many(const PlanDev* __restrict__ plans,
                                                          const WorkSeg* __restrict__ segs, int nseg)
{
    __shared__ double4 lds[SpreadMfma<NCH, ANCH>::lds_bytes / sizeof(double4)];
    const WorkSeg w = find_seg(segs, nseg);
    const PlanDev& P = plan_of(plans, w.t);
    const int first = ANCH == kSpreadAnchors ? 0 : P.n_adense;
    spread_mfma_item<NCH, ANCH>(P, first + w.g0, lds);
}

// ---------------------------------------------------------------------------
// Grid assembly: each grid slot sums the item partials that cover it and
// multiplies channel p by its factor beta_p (the Hankel coefficient
// with the sign and the factor i the combination step gives it), so that the
// row pass only sums the channels weighted by powers of 1/(om r0).
// Direct-sum-path grids are stored cell-major [cell][channel].  FFT
// path: mode l of the spread grid is divided by the inner kernel's transform
// psi^(l) = alpha2 ES^(|l| alpha2), alpha2 = w pi / N2 (the deconvolution of the
// type-2 step) and placed at FFT index l mod N2, channel-major [channel][N2];
// all other FFT inputs are zero (of FFTs above kSmallFft they are not written:
// half of the traffic of the assembly, and of the first pass's reads).
//
// A thread takes a slot with all its channels: the items that cover it are
// found, and the deconvolution computed, once, and a thread's loads and the
// wave's stores are contiguous (101 us at the 1e6 zeros of J_0, 6 channels of
// 2^21 points and less, and 76 without the zeros; 196 with a thread a slot and
// channel).  Where a block's points crowd its cells (grid_crowded) dozens of
// items cover each, and the block's slots take a thread a channel (at 1e6 x 1e6
// uniform points 19 us, 122 without).  A crowded slot of another block is added
// up by the whole wave.
// ---------------------------------------------------------------------------
// Partial i as double2: PT is double2, or float2 in the FP32-spreading mode
// (widened here, so the grids are assembled in FP64).
template <typename PT>
__device__ __forceinline__ double2 load_partial(const double2* __restrict__ part, int64_t i)
{
    PT v = reinterpret_cast<const PT*>(part)[i];
    return make_double2((double)v.x, (double)v.y);
}

constexpr int32_t kSmallFft = 4096;  // FFTs up to this are one kernel (k_fft_small), which reads all inputs
constexpr int kReduceItems = 4;      // items of a slot in flight
constexpr int kReduceLight = 32;     // items of a slot up to which its own thread adds them up
constexpr int kReduceChannels = 8;   // channels of a slot in flight

template <typename PT>
__device__ __forceinline__ void spread_reduce_body(const PlanDev& P, int bid)
{
    const double2* __restrict__ part = P.part;
    double2* __restrict__ grids = P.grids;
    const int nch = P.nch, lane = threadIdx.x & 63;
    const int64_t total = P.grid_units;
    const int64_t unit = (int64_t)bid * blockDim.x + threadIdx.x;
    // Block owning a unit: the last block b with gunit[b] <= unit.  The wave
    // searches once for its first lane's unit (uniform, through the scalar
    // unit), and each lane then steps forward over the few blocks that start
    // inside the wave's 64 units.
    const int64_t unit0 = unit - lane;
    if (unit0 >= total) return;
    int32_t lo = 0, hi = P.n_a - 1;
    const int64_t probe = ((int64_t)__builtin_amdgcn_readfirstlane((int32_t)(unit0 >> 32)) << 32) |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)unit0);
    while (lo < hi) {
        int32_t mid = (lo + hi + 1) >> 1;
        if (P.gunit[mid] <= probe) lo = mid; else hi = mid - 1;
    }
    const bool on = unit < total;
    // when the wave's last unit lies in the same block as the first, the
    // block's fields are read once through the scalar unit
    const int64_t last = unit0 + 63 < total ? unit0 + 63 : total - 1;
    const bool one_block = P.gunit[lo + 1] > last;
    int32_t blk = lo;
    if (!one_block && on)
        while (P.gunit[blk + 1] <= unit) ++blk;
    struct Fields { int64_t grid_off; int32_t fft, N2, llo, N1, item0, nitems; };
    auto fields = [&](const ABlock& B) { return Fields{B.grid_off, B.fft, B.N2, B.llo, B.N1, B.item0, B.nitems}; };
    const Fields B = one_block ? fields(P.ab[__builtin_amdgcn_readfirstlane(lo)]) : fields(P.ab[blk]);
    int64_t local = unit - P.gunit[blk];
    const bool by_channel = nch > 1 && P.gunit[blk + 1] - P.gunit[blk] != P.gslot[blk + 1] - P.gslot[blk];
    int own = 0;                                     // the thread's channel
    if (by_channel) {
        own = (int)(local % nch);
        local /= nch;
    }
    int32_t l;
    if (B.fft) l = local < B.N2 / 2 ? (int32_t)local : (int32_t)(local - B.N2);
    else l = B.llo + (int32_t)local;
    int32_t a = 0, b = 0;
    const bool spread = l >= B.llo && l < B.llo + B.N1;
    // (the first pass of a large FFT takes the other inputs as zero)
    const bool write = on && (spread || !B.fft || B.N2 <= kSmallFft);
    if (on && spread) {
        // Items covering cell l: both ends of the items' cell ranges increase
        // with the item index, so they form one run [a, b): a is the first item
        // ending after l, b the first starting after l.
        const int32_t i0 = B.item0, i1 = B.item0 + B.nitems;
        a = i0;
        int32_t top = i1;
        while (a < top) {
            int32_t mid = (a + top) >> 1;
            const Item& I = P.aitems[mid];
            if (I.sub_lo + I.sub_n <= l) a = mid + 1; else top = mid;
        }
        // b: a few steps forward from a (where points are spread out a cell
        // lies in the subgrids of one or two items), then a binary search
        b = a;
        for (int k = 0; k <= kReduceItems && b < i1 && P.aitems[b].sub_lo <= l; ++k) ++b;
        if (b - a > kReduceItems) {
            top = i1;
            while (b < top) {
                int32_t mid = (b + top) >> 1;
                if (P.aitems[mid].sub_lo <= l) b = mid + 1; else top = mid;
            }
        }
    }
    // 1 / psi^(l) on the FFT path
    double scale = 1.0;
    if (B.fft) {
        const double a2 = P.w * kPi / B.N2;
        scale = 1.0 / (a2 * eshat(P, fabs((double)l) * a2));
    }
    // channel factor: real for even p, i times real for odd p
    auto store = [&](int p, double sr, double si, const Fields& F, int64_t at, double sc) {
        const double f = P.chan[p];
        const double2 v = (p & 1) ? make_double2(-si * f, sr * f) : make_double2(sr * f, si * f);
        if (F.fft) grids[F.grid_off + (int64_t)p * F.N2 + at] = make_double2(v.x * sc, v.y * sc);
        else grids[F.grid_off + at * nch + p] = v;
    };
    if (write && by_channel) {
        // partials several at a time, added in item order
        double sr = 0.0, si = 0.0;
        int32_t it = a;
        auto add = [&](auto count) {
            constexpr int N = decltype(count)::value;
            double2 v[N];
            #pragma unroll
            for (int q = 0; q < N; ++q) {
                const Item& I = P.aitems[it + q];
                v[q] = load_partial<PT>(part, I.off + (int64_t)(l - I.sub_lo) * nch + own);
            }
            #pragma unroll
            for (int q = 0; q < N; ++q) { sr += v[q].x; si += v[q].y; }
            it += N;
        };
        while (it + 16 <= b) add(std::integral_constant<int, 16>());
        while (it + 4 <= b) add(std::integral_constant<int, 4>());
        while (it < b) add(std::integral_constant<int, 1>());
        store(own, sr, si, B, local, scale);
    }
    const bool crowded = !by_channel && b - a > kReduceLight;
    if (write && !by_channel && !crowded) {
        for (int p0 = 0; p0 < nch; p0 += kReduceChannels) {
            double sr[kReduceChannels], si[kReduceChannels];
            #pragma unroll
            for (int u = 0; u < kReduceChannels; ++u) sr[u] = si[u] = 0.0;
            for (int32_t it = a; it < b; it += kReduceItems) {
                int64_t from[kReduceItems];
                #pragma unroll
                for (int k = 0; k < kReduceItems; ++k) {
                    from[k] = 0;
                    if (it + k < b) {
                        const Item& I = P.aitems[it + k];
                        from[k] = I.off + (int64_t)(l - I.sub_lo) * nch;
                    }
                }
                #pragma unroll
                for (int k = 0; k < kReduceItems; ++k)
                    if (it + k < b) {
                        #pragma unroll
                        for (int u = 0; u < kReduceChannels; ++u)
                            if (p0 + u < nch) {
                                const double2 v = load_partial<PT>(part, from[k] + p0 + u);
                                sr[u] += v.x;
                                si[u] += v.y;
                            }
                    }
            }
            #pragma unroll
            for (int u = 0; u < kReduceChannels; ++u)
                if (p0 + u < nch) store(p0 + u, sr[u], si[u], B, local, scale);
        }
    }
    // crowded slots, one after the other: lane (g, p) adds items a + g,
    // a + g + groups, .. of channel p
    const int groups = 64 / nch, g = lane / nch, p = lane - g * nch;
    for (uint64_t left = __ballot(on && crowded); left; left &= left - 1) {
        const int h = __builtin_ctzll(left);
        const int32_t ah = __shfl(a, h), bh = __shfl(b, h), lh = __shfl(l, h);
        double sr = 0.0, si = 0.0;
        if (g < groups) {
            #pragma unroll 4
            for (int32_t it = ah + g; it < bh; it += groups) {
                const Item& I = P.aitems[it];
                const double2 v = load_partial<PT>(part, I.off + (int64_t)(lh - I.sub_lo) * nch + p);
                sr += v.x;
                si += v.y;
            }
        }
        double tr = sr, ti = si;
        for (int q = 1; q < groups; ++q) {
            tr += __shfl(sr, q * nch + p);
            ti += __shfl(si, q * nch + p);
        }
        const Fields F{__shfl(B.grid_off, h), __shfl(B.fft, h), __shfl(B.N2, h), 0, 0, 0, 0};
        const int64_t at = __shfl(local, h);
        const double sc = __shfl(scale, h);
        if (g == 0) store(p, tr, ti, F, at, sc);
    }
}

template <typename PT>
__global__ void k_spread_reduce(PlanDev P)
{
    spread_reduce_body<PT>(P, blockIdx.x);
}

template <typename PT>
__global__ void k_spread_reduce_many(const PlanDev* __restrict__ plans, const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    spread_reduce_body<PT>(plan_of(plans, w.t), w.g0);
}

// Transforms of N <= 4096 points, every size class of the transform in one
// launch (P.small).
__device__ __forceinline__ void fft_small_body(const PlanDev& P, int g)
{
    extern __shared__ double2 sm[];
    const SmallFfts& F = P.small;
    double2* __restrict__ grids = P.grids;
    int c = 0;
    while (c + 1 < F.n && g >= F.wg0[c + 1]) ++c;
    const int logN = F.log2n[c], N = 1 << logN;
    const int nch = P.nch;
    const int loc = g - F.wg0[c];
    const int slot = loc / nch, ch = loc % nch;
    const ABlock B = P.ab[P.fft_list[F.first[c] + slot]];
    double2* x = grids + B.grid_off + (int64_t)ch * N;
    for (int i = threadIdx.x; i < N; i += blockDim.x) sm[i] = x[i];
    __syncthreads();
    lds_fft(sm, N, logN, 1, 0, 1);
    for (int i = threadIdx.x; i < N; i += blockDim.x) x[i] = sm[i];
}

__global__ __launch_bounds__(256) void k_fft_small(PlanDev P) { fft_small_body(P, blockIdx.x); }

__global__ __launch_bounds__(256) void k_fft_small_many(const PlanDev* __restrict__ plans,
                                                        const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    fft_small_body(plan_of(plans, w.t), w.g0);
}

// Transforms of N = 2^13 .. 2^24 points run as two or three passes, each a
// batch of transforms of length L <= 256 done in LDS.  A workgroup holds a
// tile of `lines` batches side by side (lines * L <= kFftTilePts), chosen so
// that every global read and write moves runs of `lines` consecutive elements
// (128 B or more) even where the transform itself is strided.
//
// With n = n1 + N1 n2 and k = k2 + N2 k1 (N = N1 N2),
//   X[k2 + N2 k1] = sum_n1 w_N1^(n1 k1) w_N^(n1 k2) sum_n2 x[n1 + N1 n2] w_N2^(n2 k2),
// w_M = e^(2 pi i / M).  The inner transform over n2 is a column pass (batches
// n1 at unit stride, the transform at stride N1) that also applies
// w_N^(n1 k2); the outer one is a row pass (the transform contiguous, output
// written at stride N2).  When N2 = Na Nb is longer than 256 it is split the
// same way (n2 = na + Na nb, k2 = kb + Nb ka) into two column passes: over nb
// with w_N2^(na kb), in place, then over na, which applies w_N^(n1 k2) and
// writes n1 + N1 k2.  Column passes read the grid and the second writes the
// scratch buffer; the row pass reads the scratch buffer and writes the grid.
constexpr int kFftTilePts = 2048;
constexpr int kFftMaxLines = 16;

// Twiddles, kept per device: entries 0..4095 hold e^(2 pi i j / 4096) and
// entries 4096..8191 hold e^(2 pi i j / 2^24), so that
// w_N^e = T[E >> 12] T[4096 + (E & 4095)] with E = (e mod N) 2^(24 - log2 N).
__device__ __forceinline__ double2 fft_twiddle(const double2* __restrict__ T, int64_t e, int logN)
{
    int64_t E = (e & ((int64_t(1) << logN) - 1)) << (kMaxFftLog2 - logN);
    return cmul(T[E >> 12], T[4096 + (E & 4095)]);
}

// In-LDS transforms of the tile's lines, Stockham radix 4 (one radix-2 stage
// first when log2 L is odd); element (line, n) at sm[line * ls + n].  tw holds
// w_L^j for j < L.
__device__ void lds_fft_lines(double2* sm, int logL, int lines, int ls, const double2* tw)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    const int L = 1 << logL;
    int Ns = 1, logNs = 0;
    if (logL & 1) {
        const int half = L >> 1, nb = lines * half;
        double2 v[kFftTilePts / 2 / 256][2];
        #pragma unroll
        for (int c = 0; c < kFftTilePts / 2 / 256; ++c) {
            int b = tid + c * nt;
            if (b < nb) {
                int line = b >> (logL - 1), j = b & (half - 1);
                v[c][0] = sm[line * ls + j];
                v[c][1] = sm[line * ls + j + half];
            }
        }
        __syncthreads();
        #pragma unroll
        for (int c = 0; c < kFftTilePts / 2 / 256; ++c) {
            int b = tid + c * nt;
            if (b < nb) {
                int line = b >> (logL - 1), j = b & (half - 1);
                double2 a = v[c][0], d = v[c][1];
                sm[line * ls + 2 * j] = make_double2(a.x + d.x, a.y + d.y);
                sm[line * ls + 2 * j + 1] = make_double2(a.x - d.x, a.y - d.y);
            }
        }
        __syncthreads();
        Ns = 2; logNs = 1;
    }
    const int q4 = L >> 2, nb = lines * q4;
    while (Ns < L) {
        double2 v[kFftTilePts / 4 / 256][4];
        #pragma unroll
        for (int c = 0; c < kFftTilePts / 4 / 256; ++c) {
            int b = tid + c * nt;
            if (b < nb) {
                int line = b >> (logL - 2), j = b & (q4 - 1);
                #pragma unroll
                for (int r = 0; r < 4; ++r) v[c][r] = sm[line * ls + j + r * q4];
            }
        }
        __syncthreads();
        #pragma unroll
        for (int c = 0; c < kFftTilePts / 4 / 256; ++c) {
            int b = tid + c * nt;
            if (b < nb) {
                int line = b >> (logL - 2), j = b & (q4 - 1);
                int k = j & (Ns - 1);
                int ti = k << (logL - 2 - logNs);          // w1 = e^(2 pi i k / (4 Ns)) = w_L^ti
                double2 w1 = tw[ti], w2 = tw[2 * ti], w3 = tw[3 * ti];
                double2 x0 = v[c][0];
                double2 x1 = cmul(v[c][1], w1);
                double2 x2 = cmul(v[c][2], w2);
                double2 x3 = cmul(v[c][3], w3);
                double2 a0 = make_double2(x0.x + x2.x, x0.y + x2.y);
                double2 a1 = make_double2(x0.x - x2.x, x0.y - x2.y);
                double2 a2 = make_double2(x1.x + x3.x, x1.y + x3.y);
                double2 a3 = make_double2(-(x1.y - x3.y), x1.x - x3.x);   // i (x1 - x3)
                int d0 = (j - k) * 4 + k;
                sm[line * ls + d0] = make_double2(a0.x + a2.x, a0.y + a2.y);
                sm[line * ls + d0 + Ns] = make_double2(a1.x + a3.x, a1.y + a3.y);
                sm[line * ls + d0 + 2 * Ns] = make_double2(a0.x - a2.x, a0.y - a2.y);
                sm[line * ls + d0 + 3 * Ns] = make_double2(a1.x - a3.x, a1.y - a3.y);
            }
        }
        __syncthreads();
        Ns <<= 2; logNs += 2;
    }
}

// A column pass.  Batch (b_lo, b_hi), b_lo < blo at unit stride; input element
// t at b_lo + b_hi in_hs + t in_es, output element k at
// b_lo + b_hi out_hs + k out_es, multiplied by w_N^e,
// e = (b_lo & lo_mask) (b_hi + kmul k).
struct FftCol {
    int32_t logL, logLines, logBlo, to_scratch;
    int32_t from_grid, pad;  // the pass that reads the assembled grid (written within the spread cells alone)
    int64_t in_es, in_hs, out_es, out_hs, lo_mask, kmul;
};

// One pass over one size class of a transform: the class's first FFT-list
// slot, log2 of its FFT size, its offset in the scratch buffer, and the pass
// (for the row pass only C.logL = log2 N1 and C.logLines are used).
struct FftPass {
    int32_t first, logN;
    int64_t scratch_off;
    FftCol C;
};

// A transform's share of a batched FFT pass launch.
struct FftSeg {
    int32_t t, g0;
    FftPass F;
};

__device__ __forceinline__ void fft_stage_twiddles(double2* tw, const double2* __restrict__ T, int logL)
{
    for (int j = threadIdx.x; j < (1 << logL); j += blockDim.x) tw[j] = T[j << (12 - logL)];
}

__device__ __forceinline__ void fft_col_body(const PlanDev& P, int bid, const FftPass& F)
{
    double2* __restrict__ grids = P.grids;
    double2* __restrict__ scratch = P.scratch;
    const double2* __restrict__ T = P.fft_tw;
    const int first = F.first, logN = F.logN;
    const int64_t scratch_off = F.scratch_off;
    const FftCol& C = F.C;
    extern __shared__ double2 sm[];
    const int L = 1 << C.logL, lines = 1 << C.logLines, ls = L + 1;
    double2* tw = sm + lines * ls;
    const int tile = lines << C.logL;
    const int64_t N = int64_t(1) << logN;
    const int groups = (int)(N >> (C.logL + C.logLines));
    const int nch = P.nch;
    int tr = bid / groups, grp = bid - tr * groups;
    int slot = tr / nch, ch = tr - slot * nch;
    const ABlock B = P.ab[P.fft_list[first + slot]];
    const double2* x = grids + B.grid_off + (int64_t)ch * N;
    double2* y = C.to_scratch ? scratch + scratch_off + (int64_t)tr * N : grids + B.grid_off + (int64_t)ch * N;
    const int64_t bb = (int64_t)grp << C.logLines;
    const int64_t blo0 = bb & ((int64_t(1) << C.logBlo) - 1), bhi = bb >> C.logBlo;
    const double2* xs = x + blo0 + bhi * C.in_hs;
    constexpr int kPer = kFftTilePts / 256;
    double2 v[kPer];
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        int e = threadIdx.x + u * 256;
        const int64_t at = (int64_t)(e >> C.logLines) * C.in_es + (e & (lines - 1));
        v[u] = make_double2(0.0, 0.0);
        if (e < tile) {
            const int64_t i = blo0 + bhi * C.in_hs + at;
            if (!C.from_grid || i < B.llo + B.N1 || i >= N + B.llo) v[u] = xs[at];
        }
    }
    fft_stage_twiddles(tw, T, C.logL);
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        int e = threadIdx.x + u * 256;
        if (e < tile) sm[(e & (lines - 1)) * ls + (e >> C.logLines)] = v[u];
    }
    __syncthreads();
    lds_fft_lines(sm, C.logL, lines, ls, tw);
    double2* ys = y + blo0 + bhi * C.out_hs;
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        int e = threadIdx.x + u * 256;
        if (e < tile) {
            int k = e >> C.logLines, li = e & (lines - 1);
            double2 w = fft_twiddle(T, ((blo0 + li) & C.lo_mask) * (bhi + C.kmul * k), logN);
            ys[(int64_t)k * C.out_es + li] = cmul(sm[li * ls + k], w);
        }
    }
}

__global__ __launch_bounds__(256) void k_fft_col(PlanDev P, FftPass F) { fft_col_body(P, blockIdx.x, F); }

__global__ __launch_bounds__(256) void k_fft_col_many(const PlanDev* __restrict__ plans,
                                                      const FftSeg* __restrict__ segs, int nseg)
{
    const int s = find_seg_index(segs, nseg);
    fft_col_body(plan_of(plans, segs[s].t), (int)blockIdx.x - segs[s].g0, segs[s].F);
}

// The row pass: batch k2 < N2 of length L = N1 read contiguously at k2 N1 from
// the scratch buffer; output k1 written to the grid at k2 + N2 k1.
__device__ __forceinline__ void fft_row_body(const PlanDev& P, int bid, const FftPass& F)
{
    double2* __restrict__ grids = P.grids;
    const double2* __restrict__ scratch = P.scratch;
    const double2* __restrict__ T = P.fft_tw;
    const int first = F.first, logN = F.logN, logL = F.C.logL, logLines = F.C.logLines;
    const int64_t scratch_off = F.scratch_off;
    extern __shared__ double2 sm[];
    const int L = 1 << logL, lines = 1 << logLines, ls = L + 1;
    double2* tw = sm + lines * ls;
    const int tile = lines << logL;
    const int64_t N = int64_t(1) << logN, N2 = N >> logL;
    const int groups = (int)(N2 >> logLines);
    const int nch = P.nch;
    int tr = bid / groups, grp = bid - tr * groups;
    int slot = tr / nch, ch = tr - slot * nch;
    const ABlock B = P.ab[P.fft_list[first + slot]];
    const int64_t k20 = (int64_t)grp << logLines;
    // the cells that the block's frequencies reach (half of them or fewer: the
    // grid is twice as fine as they need); the others are not written
    const double span = fmax(P.ws[B.j1] - B.D, B.D - P.ws[B.j0]) * B.Khi;
    const int64_t reach = (int64_t)ceil(span) + P.w + 2;
    const double2* xs = scratch + scratch_off + (int64_t)tr * N + (k20 << logL);
    double2* ys = grids + B.grid_off + (int64_t)ch * N + k20;
    constexpr int kPer = kFftTilePts / 256;
    double2 v[kPer];
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        int e = threadIdx.x + u * 256;
        if (e < tile) v[u] = xs[e];
    }
    fft_stage_twiddles(tw, T, logL);
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        int e = threadIdx.x + u * 256;
        if (e < tile) sm[(e >> logL) * ls + (e & (L - 1))] = v[u];
    }
    __syncthreads();
    lds_fft_lines(sm, logL, lines, ls, tw);
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        int e = threadIdx.x + u * 256;
        if (e < tile) {
            int k1 = e >> logLines, li = e & (lines - 1);
            const int64_t k = k20 + li + (int64_t)k1 * N2;
            if (k <= reach || k >= N - reach) ys[(int64_t)k1 * N2 + li] = sm[li * ls + k1];
        }
    }
}

__global__ __launch_bounds__(256) void k_fft_row(PlanDev P, FftPass F) { fft_row_body(P, blockIdx.x, F); }

__global__ __launch_bounds__(256) void k_fft_row_many(const PlanDev* __restrict__ plans,
                                                      const FftSeg* __restrict__ segs, int nseg)
{
    const int s = find_seg_index(segs, nseg);
    fft_row_body(plan_of(plans, segs[s].t), (int)blockIdx.x - segs[s].g0, segs[s].F);
}

// ---------------------------------------------------------------------------
// Row side.
// ---------------------------------------------------------------------------

// Local block contribution at frequency om:  sum_{l=0}^{L} C_l(om R) t_l with
//   C_l(x) = delta_l J_{nu/2+l}(x/2) J_{nu/2-l}(x/2)        (nu even, reading x/2)
//   C_l(x) = 2 J_{(nu+1)/2+l}(x/2) J_{(nu-1)/2-l}(x/2)       (nu odd)
// J_k(y), y = om R / 2, comes from Miller's backward recurrence, started at N
// and normalised at the end by J_0^2 + 2 sum_k J_k^2 = 1.  Written with
// J_{-i} = (-1)^i J_i, the sum pairs index i with i + nu (the terms l > a,
// a = floor(nu/2), sign (-1)^i) and with nu - i (the terms l <= a).
//   MODE 0 (nu = 0): the products are J_i^2;
//   MODE 1 (nu = 1): J_i J_{i+1}, i.e. the current and the previous value;
//   MODE 2 (any nu): the partner nu steps back from a second copy of the
//   recurrence running behind the first; the floor(nu/2) + 1 partners of the
//   l <= a terms from LDS.
// In every mode the recurrence first runs alone down to the highest index a
// product needs, then continues with the products.
__device__ __forceinline__ void miller_rescale(double& yk, double& yk1, double& S2, double& dot)
{
    if (fabs(yk) > 1e100) { yk *= 1e-100; yk1 *= 1e-100; S2 *= 1e-200; dot *= 1e-200; }
}

// Once per four steps, for waves whose arguments are all >= kMillerGroupY: a
// step multiplies the values by at most 2N / y + 1 < 4.2e6 (start N <= 2048,
// the largest local rank allowed plus one), four steps by less than 3.1e26,
// so the values stay below 3.1e126 and their squares and sums finite.
constexpr double kMillerGroupY = 1e-3;
__device__ __forceinline__ void miller_rescale_group(double& yk, double& yk1, double& S2, double& dot)
{
    if (fmax(fabs(yk), fabs(yk1)) > 1e100) { yk *= 1e-100; yk1 *= 1e-100; S2 *= 1e-200; dot *= 1e-200; }
}

// Four consecutive local moments (8-byte aligned, read as one block).
struct Moments4 {
    double v[4];
};

template <int MODE>
__device__ double local_eval(const PlanDev& P, int lblk, double om, const double* __restrict__ lmom,
                             double* __restrict__ ring, int stride)
{
    const LBlock B = P.lb[lblk];
    double y = 0.5 * (om * B.R);
    const double* t = lmom + (int64_t)lblk * (P.L + 1);
    const int nu = MODE == 0 ? 0 : (MODE == 1 ? 1 : P.nu), L = P.L;
    if (y < 1e-30) return nu == 0 ? t[0] : 0.0;
    // the pairing reads J_{nu-i} for i <= nu/2, so the recurrence must have
    // produced every index up to nu; it also starts above every index a
    // product needs, so that the product phase runs over the same indices in
    // every lane (its index, and with it the moment loads, stay wave-uniform;
    // a higher start only makes the recurrence more accurate)
    int N = miller_start(y);
    if (N < nu + 1) N = nu + 1;
    {
        const int a_ = (MODE == 2 && (nu & 1)) ? (nu - 1) >> 1 : nu >> 1;
        const int top_ = MODE == 2 ? ((L - a_) > a_ ? (L - a_) : a_) : L;
        if (N < top_ + 1) N = top_ + 1;
    }
    const double rec = 2.0 / y;
    double yk1 = 0.0, yk = 1e-100, S2 = 0.0, dot = 0.0;
    if (MODE == 0) {
        // J_0^2 t_0 + sum_{i=1}^{L} 2 (-1)^i t_i J_i^2
        int i = N;
        // above L: the recurrence alone, with one rescale test per four
        // steps where the wave's arguments allow it (as in the grouped
        // steps below)
        auto lead = [&](int k) {
            S2 = __builtin_fma(2.0 * yk, yk, S2);
            double ykm1 = __builtin_fma((double)k * rec, yk, -yk1);
            yk1 = yk; yk = ykm1;
        };
        if (__all(y >= kMillerGroupY)) {
            for (; i - 3 > L; i -= 4) {
                lead(i); lead(i - 1); lead(i - 2); lead(i - 3);
                miller_rescale_group(yk, yk1, S2, dot);
            }
        }
        for (; i > L; --i) {
            lead(i);
            miller_rescale(yk, yk1, S2, dot);
        }
        i = L;   // where every lane left the loop (N > L): the index is now wave-uniform
        // i = L .. 1 in every lane (the start is above L): L mod 4 single
        // steps, then groups of four whose moments u[i-3 .. i] are read
        // together (u_i = 2 (-1)^i t_i)
        auto step = [&](int k, double uk, bool check) {
            double q = yk * yk;
            S2 = __builtin_fma(2.0, q, S2);
            dot = __builtin_fma(uk, q, dot);
            double ykm1 = __builtin_fma((double)k * rec, yk, -yk1);
            yk1 = yk; yk = ykm1;
            if (check) miller_rescale(yk, yk1, S2, dot);
        };
        for (int u = L & 3; u > 0; --u, --i) step(i, t[i], true);
        if (__all(y >= kMillerGroupY)) {
            // four steps grow the values by less than 1e27: one rescale test
            // per group, and the next group's moments in flight
            Moments4 nx;
            if (i >= 4) __builtin_memcpy(&nx, t + i - 3, sizeof nx);
            for (; i >= 4; i -= 4) {
                const Moments4 q = nx;
                if (i >= 8) __builtin_memcpy(&nx, t + i - 7, sizeof nx);
                step(i, q.v[3], false); step(i - 1, q.v[2], false);
                step(i - 2, q.v[1], false); step(i - 3, q.v[0], false);
                miller_rescale_group(yk, yk1, S2, dot);
            }
        } else {
            for (; i >= 4; i -= 4) {
                Moments4 q;
                __builtin_memcpy(&q, t + i - 3, sizeof q);
                step(i, q.v[3], true); step(i - 1, q.v[2], true); step(i - 2, q.v[1], true); step(i - 3, q.v[0], true);
            }
        }
        S2 = __builtin_fma(yk, yk, S2);
        dot = __builtin_fma(t[0] * yk, yk, dot);
        return dot / S2;
    } else if (MODE == 1) {
        // 2 t_0 J_0 J_1 + sum_{i=1}^{L} 2 (-1)^i t_i J_i J_{i+1}; yk1 = J_{i+1}
        int i = N;
        // above L: the recurrence alone, with one rescale test per four
        // steps where the wave's arguments allow it (as in the grouped
        // steps below)
        auto lead = [&](int k) {
            S2 = __builtin_fma(2.0 * yk, yk, S2);
            double ykm1 = __builtin_fma((double)k * rec, yk, -yk1);
            yk1 = yk; yk = ykm1;
        };
        if (__all(y >= kMillerGroupY)) {
            for (; i - 3 > L; i -= 4) {
                lead(i); lead(i - 1); lead(i - 2); lead(i - 3);
                miller_rescale_group(yk, yk1, S2, dot);
            }
        }
        for (; i > L; --i) {
            lead(i);
            miller_rescale(yk, yk1, S2, dot);
        }
        i = L;   // where every lane left the loop (N > L): the index is now wave-uniform
        auto step = [&](int k, double uk, bool check) {
            S2 = __builtin_fma(2.0 * yk, yk, S2);
            dot = __builtin_fma(uk * yk, yk1, dot);
            double ykm1 = __builtin_fma((double)k * rec, yk, -yk1);
            yk1 = yk; yk = ykm1;
            if (check) miller_rescale(yk, yk1, S2, dot);
        };
        for (int u = L & 3; u > 0; --u, --i) step(i, t[i], true);
        if (__all(y >= kMillerGroupY)) {
            Moments4 nx;
            if (i >= 4) __builtin_memcpy(&nx, t + i - 3, sizeof nx);
            for (; i >= 4; i -= 4) {
                const Moments4 q = nx;
                if (i >= 8) __builtin_memcpy(&nx, t + i - 7, sizeof nx);
                step(i, q.v[3], false); step(i - 1, q.v[2], false);
                step(i - 2, q.v[1], false); step(i - 3, q.v[0], false);
                miller_rescale_group(yk, yk1, S2, dot);
            }
        } else {
            for (; i >= 4; i -= 4) {
                Moments4 q;
                __builtin_memcpy(&q, t + i - 3, sizeof q);
                step(i, q.v[3], true); step(i - 1, q.v[2], true); step(i - 2, q.v[1], true); step(i - 3, q.v[0], true);
            }
        }
        S2 = __builtin_fma(yk, yk, S2);
        dot = __builtin_fma(2.0 * t[0] * yk, yk1, dot);
        return dot / S2;
    } else {
        // Part one pairs i with i + nu (1 <= i <= L - a, weight 2 (-1)^i t_{a+i});
        // part two pairs i with nu - i (0 <= i <= a, weight t_{a-i}, doubled
        // except the l = 0 term of an even order).  J_{i+nu} comes from a second
        // copy of the recurrence run nu steps behind the first: the same
        // operations on the same state give the same values, so the lagging
        // copy is started from the leading copy's state at s0 = min(N, L-a+nu)
        // and the two run as independent chains.  Part two's partners
        // J_{a2..nu} (a2 = nu - a) are kept per thread in LDS as the leading
        // copy passes them.  Both copies rescale by exact powers of two; the
        // leading copy's rescales since the lagging copy's state (d) set the
        // factor 2^(-332 d) between the two scales.
        const int odd = nu & 1;
        const int a = nu >> 1;
        const int a2 = nu - a;
        const double sa = (a & 1) ? -1.0 : 1.0;
        const int hi1 = L - a;
        const int top = hi1 > nu ? hi1 : nu;
        const int s0 = N < hi1 + nu ? N : hi1 + nu;
        const int act = s0 - nu;
        const double up = 0x1p332, down = 0x1p-332, down2 = 0x1p-664;
        // Here S2 holds half the normalising sum (J_0^2 / 2 + sum_{i>=1} J_i^2),
        // one FMA per step; the lagging copy starts (i == act) at one or two
        // steps of a wave, so that test is a wave vote first.
        double syk = yk, syk1 = 0.0;          // leading copy's state at s0
        double lyk = 0.0, lyk1 = 0.0, lsc = sa;   // lsc: (-1)^a 2^(-332 d)
        int d = 0;
        int i = N;
        auto lead = [&](int k) {
            if (k == s0) { syk = yk; syk1 = yk1; d = 0; lsc = sa; }
            S2 = __builtin_fma(yk, yk, S2);
            double ykm1 = __builtin_fma((double)k * rec, yk, -yk1);
            yk1 = yk; yk = ykm1;
        };
        auto lead_rescale = [&](bool group) {
            if ((group ? fmax(fabs(yk), fabs(yk1)) : fabs(yk)) > up) {
                yk *= down; yk1 *= down; S2 *= down2; dot *= down2;
                ++d; lsc = __builtin_amdgcn_ldexp(sa, -332 * d);
            }
        };
        if (__all(y >= kMillerGroupY)) {
            // one rescale test per four steps, as in the grouped steps below
            for (; i - 3 > top; i -= 4) {
                lead(i); lead(i - 1); lead(i - 2); lead(i - 3);
                lead_rescale(true);
            }
        }
        for (; i > top; --i) {
            lead(i);
            lead_rescale(false);
        }
        i = top;   // where every lane left the loop (N > top): the index is now wave-uniform
        // i = top .. 0 in every lane.  stepB takes the products at index i and
        // (i > 0) moves both copies one index down; rescaleB follows a step
        // whose last products were at index il (stored partners: indices il .. nu).
        auto stepB = [&](int i) {
            if (__any(i == act)) {
                if (i == act) { lyk = syk; lyk1 = syk1; }
            }
            S2 = __builtin_fma(i == 0 ? 0.5 * yk : yk, yk, S2);
            if (i >= a2 && i <= nu) ring[(i - a2) * stride] = yk;
            if (i >= 1 && i <= hi1) {
                // 2 (-1)^i t_{a+i} = (-1)^a u_{a+i}
                dot = __builtin_fma(t[a + i] * yk, lyk * lsc, dot);
            }
            if (i <= a && a - i <= L) {
                int l2 = a - i;
                double pv = ring[(nu - i - a2) * stride];
                // 2 t_l2 = (-1)^l2 u_l2 (l2 >= 1); t_0 = u_0
                double coef = l2 == 0 ? (odd ? 2.0 * t[0] : t[0]) : ((l2 & 1) ? -t[l2] : t[l2]);
                dot = __builtin_fma(coef * yk, pv, dot);
            }
            if (i > 0) {
                double ykm1 = __builtin_fma((double)i * rec, yk, -yk1);
                yk1 = yk; yk = ykm1;
                double lykm1 = __builtin_fma((double)(i + nu) * rec, lyk, -lyk1);
                lyk1 = lyk; lyk = lykm1;
            }
        };
        auto rescaleB = [&](int il, bool group) {
            const double ml = group ? fmax(fabs(yk), fabs(yk1)) : fabs(yk);
            if (ml > up) {
                yk *= down; yk1 *= down; S2 *= down2; dot *= down2;
                ++d; lsc = __builtin_amdgcn_ldexp(sa, -332 * d);
                for (int q = (il > a2 ? il : a2) - a2; q <= nu - a2; ++q) ring[q * stride] *= down;
            }
            const double mg = group ? fmax(fabs(lyk), fabs(lyk1)) : fabs(lyk);
            if (mg > up) {
                lyk *= down; lyk1 *= down;
                --d; lsc = __builtin_amdgcn_ldexp(sa, -332 * d);
            }
        };
        // Above nu (i = top .. nu + 1, present when hi1 > nu) a step has no
        // partner to store or read: only part one's product and the two
        // recurrences, so these steps skip stepB's index tests, and their
        // moments t[a + i] (contiguous, wave-uniform) come four at a time.
        auto stepA = [&](int i, double ti) {
            if (__any(i == act)) {
                if (i == act) { lyk = syk; lyk1 = syk1; }
            }
            S2 = __builtin_fma(yk, yk, S2);
            dot = __builtin_fma(ti * yk, lyk * lsc, dot);
            double ykm1 = __builtin_fma((double)i * rec, yk, -yk1);
            yk1 = yk; yk = ykm1;
            double lykm1 = __builtin_fma((double)(i + nu) * rec, lyk, -lyk1);
            lyk1 = lyk; lyk = lykm1;
        };
        const bool group = __all(y >= kMillerGroupY);
        if (group) {
            // one rescale test per four steps (growth below 3.1e26 per group);
            // the copies may rescale at different indices, d counts both
            Moments4 nx;
            if (i - 3 > nu) __builtin_memcpy(&nx, t + a + i - 3, sizeof nx);
            for (; i - 3 > nu; i -= 4) {
                const Moments4 q = nx;
                if (i - 7 > nu) __builtin_memcpy(&nx, t + a + i - 7, sizeof nx);
                stepA(i, q.v[3]); stepA(i - 1, q.v[2]); stepA(i - 2, q.v[1]); stepA(i - 3, q.v[0]);
                rescaleB(i - 3, true);
            }
        }
        for (; i > nu; --i) {
            stepA(i, t[a + i]);
            rescaleB(i, false);
        }
        if (group) {
            for (; i >= 4; i -= 4) {
                stepB(i); stepB(i - 1); stepB(i - 2); stepB(i - 3);
                rescaleB(i - 3, true);
            }
        }
        for (; i >= 0; --i) {
            stepB(i);
            if (i == 0) break;
            rescaleB(i, false);
        }
        return dot / (2.0 * S2);
    }
}

// Local block contribution at a half-integer order nu = n + 1/2, x = om R in
// [0, z]: from J_{n+1/2}(x y) = sqrt(y) sqrt(2x/pi) sum_l beta_{e+2l}(x) T_{e+2l}(y),
//   sqrt(2x/pi) sum_{l=0}^{L} beta_{e+2l}(x) t_l,   t_l = sum_k c_k sqrt(y_k) T_{e+2l}(y_k),
// with beta from the plan's table: panel p = floor(x / h), Horner's rule in the
// panel variable tau = 2 (x / h - p) - 1 for each l; the leading panels
// (below x = n + 10) hold beta / x^n, accurate relative to beta itself there.
// The factor sqrt(2x/pi), not smooth at 0, is left to the row pass.
__device__ double local_eval_half(const PlanDev& P, int lblk, double om, const double* __restrict__ lmom)
{
    const LBlock B = P.lb[lblk];
    const double x = om * B.R;
    const double* t = lmom + (int64_t)lblk * (P.L + 1);
    const double u = x * P.half_inv_h;
    int pn = (int)u;
    if (pn > P.half_np - 1) pn = P.half_np - 1;
    const double tau = 2.0 * (u - pn) - 1.0;
    const double* tab = P.half_tab + (int64_t)pn * (P.L + 1) * (kHalfDeg + 1);
    double acc = 0.0;
    for (int l = 0; l <= P.L; ++l) {
        const double* cf = tab + l * (kHalfDeg + 1);
        double b = cf[kHalfDeg];
        #pragma unroll
        for (int d = kHalfDeg - 1; d >= 0; --d) b = __builtin_fma(b, tau, cf[d]);
        acc = __builtin_fma(b, t[l], acc);
    }
    if (pn < P.half_ns && P.nu > 0) acc *= pow(x, (double)P.nu);
    return acc;
}

// Asymptotic block contribution at frequency om (Sec. 3.2):
//   sqrt(2/pi) Re( e^{i phi} sum_p beta_p om^(-p-1/2) y_p ),
//   beta_{2l} = (-1)^l a_{2l},  beta_{2l+1} = i (-1)^l a_{2l+1},
// where y_p = sum_k x_k^(p) e^{i om r_k} is the type-3 sum of channel p.  With
// s' = om - D and theta = s' h:  y_p = e^{i om C} h F_p(theta) / phi^(s'),
// F_p(theta) = sum_l b_l^(p) e^{i l theta} evaluated directly over the cells
// (direct-sum path) or from the FFT by ES interpolation (FFT path).  The grids
// already hold beta_p b_l^(p), so with gamma = 1/(om r0) each cell (or tap)
// needs the single value sum_p gamma^p beta_p b_l^(p): two multiply-adds per
// channel.  On the direct-sum path the powers gamma^p are kept in registers
// (the grid value, when it comes through the scalar unit, is then a
// multiplicand and needs no copy into vector registers); on the FFT path the
// sum is Horner's rule in gamma.  One complex product per cell or tap.
// Called with a wave-uniform block index whenever every active lane of the
// wave is in the same block (the usual case, frequencies being sorted); the
// block's fields and its direct-sum grid are then read through the scalar
// unit and broadcast to all lanes.
// One Horner step of a direct-sum cell sum with the cell's channel-0 value
// (g0r, g0i) in scalar registers:
//   (ar, ai) <- (ar, ai) e^{i theta} + (g0r, g0i)
// in four FMAs, the scalar values as addends and ar, ai updated in place.
// The compiler would copy the two scalar values into vector registers first
// and move the results back into ar, ai (six more instructions per cell);
// the step is written out so that it does not.  Callers pass values that are
// the same in every lane.
__device__ __forceinline__ void rotate_add_uniform(double& ar, double& ai, double er, double ei, double g0r, double g0i)
{
    double t;
    asm("v_fma_f64 %2, %0, %4, %6\n\t"     // t  = ar ei + g0i
        "v_fma_f64 %0, %0, %3, %5\n\t"     // ar = ar er + g0r
        "v_fma_f64 %0, -%1, %4, %0\n\t"    // ar -= ai ei
        "v_fma_f64 %1, %1, %3, %2"           // ai = ai er + t
        : "+v"(ar), "+v"(ai), "=&v"(t)
        : "v"(er), "v"(ei), "s"(g0r), "s"(g0i));
}

// UNI: the block index, and so the block's fields and grid, is the same in
// every lane of the wave.
template <int NCH, bool UNI>
__device__ double asym_eval(const PlanDev& P, int ablk, double om, const double2* __restrict__ grids)
{
    const ABlock B = P.ab[ablk];
    if (B.rK > 0) return rank_eval<UNI>(P, B, om);
    const int w = P.w;
    // gamma = 1/(om r0) and its square root (om r0 > z > 0 on an asymptotic block)
    const double rs = rsqrt_refined(om * B.r0);
    const double gam = rs * rs;
    double gpow[NCH];
    gpow[0] = 1.0;
    #pragma unroll
    for (int p = 1; p < NCH; ++p) gpow[p] = gpow[p - 1] * gam;
    dd sp = two_sum(om, -B.D);
    double ar = 0.0, ai = 0.0;
    // final phase om C + phi (+ llo theta on the direct-sum path), double-double
    dd pc = two_prod(om, B.C);
    dd ph = two_sum(pc.hi, P.phi_hi);
    double ph_lo = ph.lo + pc.lo + P.phi_lo;
    if (!B.fft) {
        const double2* G = grids + B.grid_off;
        double th = sp.hi * B.h, tl = sp.lo * B.h;
        // the cell sum starts at l = llo: its factor e^{i llo theta} joins the
        // final phase, and the rotation starts at 1
        dd a0 = two_prod((double)B.llo, th);
        dd q = two_sum(ph.hi, a0.hi);
        ph.hi = q.hi;
        ph_lo += q.lo + __builtin_fma((double)B.llo, tl, a0.lo);
        double s1, c1;
        sincos_small(th, &s1, &c1);
        const double er = c1 - tl * s1, ei = s1 + tl * c1;
        // Horner's rule in e^{i theta} from the last cell down
        for (int cix = B.N1 - 1; cix >= 0; --cix) {
            // the channel sum with the powers of gamma as multiplicands (where
            // the block is uniform across the wave the grid values come in
            // scalar registers, and a scalar operand fits an FMA's
            // multiplicand with no copy)
            const double2* gp = G + (int64_t)cix * NCH;
            double2 gv[NCH];
            #pragma unroll
            for (int p = 0; p < NCH; ++p) gv[p] = gp[p];
            if constexpr (UNI) {
                // the rotation first, channel 0 its addend, then the other
                // channels straight into ar, ai
                rotate_add_uniform(ar, ai, er, ei, gv[0].x, gv[0].y);
                #pragma unroll
                for (int p = 1; p < NCH; ++p) {
                    ar = __builtin_fma(gv[p].x, gpow[p], ar);
                    ai = __builtin_fma(gv[p].y, gpow[p], ai);
                }
            } else {
                double br = gv[0].x, bi = gv[0].y;
                #pragma unroll
                for (int p = 1; p < NCH; ++p) {
                    br = __builtin_fma(gv[p].x, gpow[p], br);
                    bi = __builtin_fma(gv[p].y, gpow[p], bi);
                }
                const double tr = __builtin_fma(ar, er, __builtin_fma(-ai, ei, br));
                ai = __builtin_fma(ar, ei, __builtin_fma(ai, er, bi));
                ar = tr;
            }
        }
    } else {
        const double2* Aq = grids + B.grid_off;
        dd v = two_prod(sp.hi, B.Khi);
        double vl = v.lo + (sp.lo * B.Khi + sp.hi * B.Klo);
        int q0 = (int)ceil(v.hi - 0.5 * w);
        const int mask = B.N2 - 1;
        // Tap t sits at offset t + f0 - w/2 from the target, f0 in [0, 1).  Its
        // kernel value is piece t of the ES kernel at f0 (the pieces the
        // spreading uses, w x (kEsDeg + 1) monomial coefficients in 2 f - 1,
        // the same for every lane: each enters its FMA as the scalar addend).
        // Against exp and sqrt per tap this is a third of the instructions and
        // fewer registers.
        const double* __restrict__ es_poly = P.es_poly;
        const double sf = 2.0 * ((((double)q0 - v.hi) - vl) + 0.5 * w) - 1.0;
        for (int tap = 0; tap < w; ++tap) {
            int q = q0 + tap;
            int qi = q & mask;
            // the tap's channel values first, all loads in flight while the
            // kernel value is computed
            double2 gv[NCH];
            #pragma unroll
            for (int p = 0; p < NCH; ++p) gv[p] = Aq[(int64_t)p * B.N2 + qi];
            const double* cf = es_poly + tap * (kEsDeg + 1);
            double psi = cf[kEsDeg];
            #pragma unroll
            for (int d = kEsDeg - 1; d >= 0; --d) psi = fma_uniform_addend(psi, sf, cf[d]);
            // Horner's rule in gamma from the highest channel: the loaded values
            // (vector registers here) are the addends
            double br = gv[NCH - 1].x, bi = gv[NCH - 1].y;
            #pragma unroll
            for (int p = NCH - 2; p >= 0; --p) {
                br = __builtin_fma(br, gam, gv[p].x);
                bi = __builtin_fma(bi, gam, gv[p].y);
            }
            ar = __builtin_fma(psi, br, ar);
            ai = __builtin_fma(psi, bi, ai);
        }
        double sc = 2.0 * kPi / B.N2;
        ar *= sc;
        ai *= sc;
    }
    double kap = fabs(sp.hi) * B.alpha;
    double scale = B.h * rcp_refined(B.alpha * eshat(P, kap));
    double cr, ci;
    cis_dd(ph.hi, ph_lo, cr, ci);
    double amp = rs * scale;
    return kSqrt2OverPi * amp * __builtin_fma(cr, ar, -ci * ai);
}

// ---------------------------------------------------------------------------
// Rows of FFT-path blocks through expansions.  Where a block has many more
// rows than degrees of freedom, its part at frequency omega, without the
// phase e^{i omega C}, is a K-term Chebyshev expansion on each of its panels
// of frequencies (as in the rank blocks): the transform is interpolated at
// the K nodes of a panel, and a row adds up a series instead of reading w
// cells of every channel.  A node's loads, w neighbouring cells of a channel
// at a time, are a chain of latencies over the channels, so four lanes share
// a node, every fourth channel and tap each: a wave takes one of the four
// shares of two neighbouring panels, kRankK lanes a panel.
// 34 us for 6600 panels (1e6 x 1e6, order 0, 8 channels), where the row pass
// falls from 123 to 73 us; at order 10 (12 channels) 41, and 138 to 74.
// ---------------------------------------------------------------------------
constexpr int kFftShares = 4;        // waves
constexpr int kFftTaps = 8;          // taps loaded at once

__device__ __forceinline__ void fft_nodes_body(const PlanDev& P, int bid)
{
    constexpr int kTaps = (kMaxEsWidth + kFftTaps - 1) / kFftTaps * kFftTaps;
    __shared__ double s_psi[kTaps][64];
    __shared__ double2 s_f[kFftShares][64];
    const int lane = threadIdx.x & 63, share = threadIdx.x >> 6, g = lane / kRankK, x = lane - g * kRankK;
    const Panel T = P.flist[bid];
    const ABlock& B = P.ab[T.blk];
    const int K = B.rK, q = T.q + g;
    const bool on = g < kFftPanels && q < B.pr;
    const double* __restrict__ tab = P.rank_tab + rank_tab_off(K);
    // the share's cosines of coefficient x (of the panel's first node in lanes
    // without one), loaded ahead
    const int quarter = K / kFftShares, xc = x < K ? x : 0;
    double cosine[kRankK / kFftShares];
    #pragma unroll
    for (int u = 0; u < kRankK / kFftShares; ++u)
        cosine[u] = u < quarter ? tab[K * K + (share * quarter + u) * K + xc] : 0.0;
    const int w = P.w, mask = B.N2 - 1;
    const dd sp = two_sum(rank_mid(q, B.pr, B.rw), B.rw * tab[K + xc]);
    const dd v = two_prod(sp.hi, B.Khi);
    const double vl = v.lo + (sp.lo * B.Khi + sp.hi * B.Klo);
    const int q0 = (int)ceil(v.hi - 0.5 * w);
    const double sf = 2.0 * ((((double)q0 - v.hi) - vl) + 0.5 * w) - 1.0;
    for (int tap = share; tap < kTaps; tap += kFftShares) {
        double psi = 0.0;
        if (tap < w) {
            const double* cf = P.es_poly + tap * (kEsDeg + 1);
            psi = cf[kEsDeg];
            #pragma unroll
            for (int d = kEsDeg - 1; d >= 0; --d) psi = __builtin_fma(psi, sf, cf[d]);
        }
        s_psi[tap][lane] = psi;
    }
    __syncthreads();
    {
        const double rs = rsqrt_refined((B.D + sp.hi) * B.r0), gam = rs * rs, gam2 = gam * gam, gam4 = gam2 * gam2;
        double ar = 0.0, ai = 0.0;
        for (int p = (P.nch - 1 - share) / kFftShares * kFftShares + share; p >= 0 && P.nch > share; p -= kFftShares) {
            const double2* __restrict__ A = P.grids + B.grid_off + (int64_t)p * B.N2;
            double br = 0.0, bi = 0.0;
            for (int t0 = 0; t0 < w; t0 += kFftTaps) {
                double2 c[kFftTaps];
                #pragma unroll
                for (int u = 0; u < kFftTaps; ++u) c[u] = A[(q0 + t0 + u) & mask];
                #pragma unroll
                for (int u = 0; u < kFftTaps; ++u) {
                    const double psi = s_psi[t0 + u][lane];
                    br = __builtin_fma(psi, c[u].x, br);
                    bi = __builtin_fma(psi, c[u].y, bi);
                }
            }
            ar = __builtin_fma(ar, gam4, br);
            ai = __builtin_fma(ai, gam4, bi);
        }
        const double kap = fabs(sp.hi) * B.alpha;
        const double own = (share & 1 ? gam : 1.0) * (share & 2 ? gam2 : 1.0);
        const double sc = own * (2.0 * kPi / B.N2 * (B.h * rcp_refined(B.alpha * eshat(P, kap))));
        s_f[share][lane] = make_double2(ar * sc, ai * sc);
    }
    __syncthreads();
    // coefficient x, as rank_store_coefs, the shares a quarter of the nodes each
    double vr = 0.0, vi = 0.0;
    #pragma unroll
    for (int u = 0; u < kRankK / kFftShares; ++u) {
        const int h = g * kRankK + share * quarter + (u < quarter ? u : 0);
        double fr = 0.0, fi = 0.0;
        #pragma unroll
        for (int e = 0; e < kFftShares; ++e) {
            const double2 f = s_f[e][h & 63];
            fr += f.x;
            fi += f.y;
        }
        vr = __builtin_fma(fr, cosine[u], vr);
        vi = __builtin_fma(fi, cosine[u], vi);
    }
    __syncthreads();
    s_f[share][lane] = make_double2(vr, vi);
    __syncthreads();
    if (share == 0 && on && x < K) {
        const double2 a = s_f[0][lane], b = s_f[1][lane], c = s_f[2][lane], d = s_f[3][lane];
        static_assert(kFftShares == 4, "four shares added up");
        const double f = (x == 0 ? 1.0 : 2.0) / K;
        P.rcoef[(int64_t)(B.rpan0 + q) * kRankK + x] =
            make_double2(((a.x + b.x) + (c.x + d.x)) * f, ((a.y + b.y) + (c.y + d.y)) * f);
    }
}

__global__ __launch_bounds__(256) void k_fft_nodes(PlanDev P) { fft_nodes_body(P, blockIdx.x); }

__global__ __launch_bounds__(256) void k_fft_nodes_many(const PlanDev* __restrict__ plans,
                                                        const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    fft_nodes_body(plan_of(plans, w.t), w.g0);
}

// ---------------------------------------------------------------------------
// J_nu for the direct blocks.  Their entries lie along the curve omega r = z
// (every direct block straddles it at the finest subdivision level), so the
// plan carries a table of J_nu on panels of width kJtabWidth around z (built
// on the host in extended precision): per panel the degree-15 Chebyshev
// interpolant at the 16 Chebyshev points, stored as monomial coefficients in
// the panel coordinate u in [-1, 1].  Arguments outside the table take
// besselj_full.
// ---------------------------------------------------------------------------
// J_nu(xh + xl) from the table where it covers xh, else besselj_full.
__device__ __forceinline__ double besselj_direct(const PlanDev& P, double xh, double xl)
{
    const double t = (xh - P.jtab_x0) * (1.0 / kJtabWidth);
    if (t >= 0.0 && t < (double)P.jtab_np) {
        const int p = (int)t;
        // the panel's left end (exact), and xh - xs exactly (xs = 0 or xs <= xh <= 2 xs)
        const double xs = __builtin_fma((double)p, kJtabWidth, P.jtab_x0);
        const double u = ((xh - xs) - 1.0) + xl;
        const double2* __restrict__ c = (const double2*)(P.jtab + (int64_t)p * kJtabCoef);
        double2 a[kJtabCoef / 2];
        #pragma unroll
        for (int q = 0; q < kJtabCoef / 2; ++q) a[q] = c[q];
        double v = a[kJtabCoef / 2 - 1].y;
        #pragma unroll
        for (int q = kJtabCoef / 2 - 1; q >= 0; --q) {
            if (q < kJtabCoef / 2 - 1) v = __builtin_fma(v, u, a[q].y);
            v = __builtin_fma(v, u, a[q].x);
        }
        return v;
    }
    return besselj_full(P, xh, xl);
}

// Two entries' table values at once (both arguments on the table): the two
// panels' loads issue together and the two Horner chains interleave.
__device__ __forceinline__ bool on_jtab(const PlanDev& P, double xh)
{
    const double t = (xh - P.jtab_x0) * (1.0 / kJtabWidth);
    return t >= 0.0 && t < (double)P.jtab_np;
}

// The table's panels as (kJtabCoef / 2) double2 records, read from `tab`
// with a stride of STRIDE double2 per panel (global memory, or the LDS copy
// whose padded stride spreads consecutive panels over the banks).
template <int STRIDE, typename Tab>
__device__ __forceinline__ void besselj_table2(const PlanDev& P, Tab tab, double xh1, double xl1, double xh2,
                                               double xl2, double& j1, double& j2)
{
    const int p1 = (int)((xh1 - P.jtab_x0) * (1.0 / kJtabWidth));
    const int p2 = (int)((xh2 - P.jtab_x0) * (1.0 / kJtabWidth));
    const double u1 = ((xh1 - __builtin_fma((double)p1, kJtabWidth, P.jtab_x0)) - 1.0) + xl1;
    const double u2 = ((xh2 - __builtin_fma((double)p2, kJtabWidth, P.jtab_x0)) - 1.0) + xl2;
    const auto c1 = tab + p1 * STRIDE;
    const auto c2 = tab + p2 * STRIDE;
    double2 a[kJtabCoef / 2], b[kJtabCoef / 2];
    #pragma unroll
    for (int q = 0; q < kJtabCoef / 2; ++q) { a[q] = c1[q]; b[q] = c2[q]; }
    double v = a[kJtabCoef / 2 - 1].y, w = b[kJtabCoef / 2 - 1].y;
    #pragma unroll
    for (int q = kJtabCoef / 2 - 1; q >= 0; --q) {
        if (q < kJtabCoef / 2 - 1) {
            v = __builtin_fma(v, u1, a[q].y);
            w = __builtin_fma(w, u2, b[q].y);
        }
        v = __builtin_fma(v, u1, a[q].x);
        w = __builtin_fma(w, u2, b[q].x);
    }
    j1 = v;
    j2 = w;
}

// Direct blocks (entry by entry, J_nu to full precision).  One workgroup of
// kDirectThreads lanes per block: each row of the block is given G lanes (G a
// power of two up to 64, as many as fit), the lanes of a row sum strided
// entries and combine by shuffles.  A
// row lies in at most one direct block (the last block of its path down the
// subdivision tree), so the per-row sums are stored, not accumulated; rows in
// none are never read, and gd needs no clearing.
constexpr int kDirectThreads = 256;
// The panels that a block's arguments lie on, where they are at most
// kJtabLdsPanels, are copied into LDS by its workgroup and read from there:
// shorter latency than the cache hierarchy for the eight 16-byte loads per
// entry.  A panel takes kJtabLdsStride double2 (one more than its
// coefficients), so that lanes on neighbouring panels read different banks.
constexpr int kJtabLdsPanels = 64;
constexpr int kJtabLdsStride = kJtabCoef / 2 + 1;

template <bool LDS>
__device__ __forceinline__ void direct_rows(const PlanDev& P, const DBlock& D, const double2* s_tab)
{
    const double* __restrict__ cs = P.cs;
    double* __restrict__ gd = P.gd;
    const int mb = D.j1 - D.j0 + 1, nb = D.k1 - D.k0 + 1;
    int G = 1;
    while (G < 64 && 2 * G * mb <= kDirectThreads) G <<= 1;
    const int rows_per_pass = kDirectThreads / G;
    const int lane = threadIdx.x;
    const int grp = lane / G, gl = lane & (G - 1);
    for (int r0 = 0; r0 < mb; r0 += rows_per_pass) {
        int i = r0 + grp;
        double acc = 0.0;
        if (i < mb) {
            double om = P.ws[D.j0 + i];
            // two entries per step (the lane's next two, in order): when both
            // arguments are on the table their evaluations interleave
            for (int k = gl; k < nb; k += 2 * G) {
                const bool two = k + G < nb;
                const int k2 = two ? k + G : k;
                const dd x1 = two_prod(om, P.rs[D.k0 + k]), x2 = two_prod(om, P.rs[D.k0 + k2]);
                const double c1 = cs[D.k0 + k], c2 = two ? cs[D.k0 + k2] : 0.0;
                double j1, j2;
                if (on_jtab(P, x1.hi) && on_jtab(P, x2.hi)) {
                    if constexpr (LDS)
                        besselj_table2<kJtabLdsStride>(P, s_tab, x1.hi, x1.lo, x2.hi, x2.lo, j1, j2);
                    else
                        besselj_table2<kJtabCoef / 2>(P, (const double2*)P.jtab, x1.hi, x1.lo, x2.hi, x2.lo, j1, j2);
                } else {
                    j1 = besselj_direct(P, x1.hi, x1.lo);
                    j2 = two ? besselj_direct(P, x2.hi, x2.lo) : 0.0;
                }
                acc = __builtin_fma(c1, j1, acc);
                acc = __builtin_fma(c2, j2, acc);
            }
        }
        for (int o = G >> 1; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
        if (i < mb && gl == 0) gd[D.j0 + i] = acc;
    }
}

// A direct block through expansions, a wave: with x = omega r its kernel
// J_nu(x) (x^{-1/2} J_nu(x) at half-integer orders, the square roots going to
// the weights and the rows) is entire in r and in omega, and the blocks lie so
// close to the curve omega r = z that a few terms give it to full precision.
// Moments of the weights, nodal weights, the kernel at K x K node pairs (to
// full precision, as an entry), coefficients of the rows' series.
template <int KC>
__device__ __forceinline__ void direct_expand(const PlanDev& P, int d, double* s)
{
    const DBlock& B = P.db[d];
    const int lane = threadIdx.x & 63, K = B.K;
    const double inv = B.cw > 0.0 ? rcp_refined(B.cw) : 0.0;
    double acc[KC];
    #pragma unroll
    for (int m = 0; m < KC; ++m) acc[m] = 0.0;
    const int kb = B.k1 + 1;
    double r_nx = B.C, c_nx = 0.0;
    if (B.k0 + lane < kb) { r_nx = P.rs[B.k0 + lane]; c_nx = P.cs[B.k0 + lane]; }
    for (int k0 = B.k0; k0 < kb; k0 += 64) {
        const double r = r_nx;
        double c = c_nx;
        const int k = k0 + 64 + lane;
        r_nx = B.C; c_nx = 0.0;
        if (k < kb) { r_nx = P.rs[k]; c_nx = P.cs[k]; }
        if (P.half) c *= sqrt(r);
        const dd b = two_sum(r, -B.C);
        const double y = (b.hi + b.lo) * inv, y2 = y + y;
        double t0 = 1.0, t1 = y;
        #pragma unroll
        for (int m = 0; m < KC; ++m) {
            acc[m] = __builtin_fma(c, t0, acc[m]);
            const double t2 = __builtin_fma(y2, t1, -t0);
            t0 = t1;
            t1 = t2;
        }
    }
    const double tm = wave_sums<KC>(acc, s, lane);
    const double* __restrict__ tab = P.rank_tab + rank_tab_off(K);
    double w = 0.0;
    {
        const int q = lane < K ? lane : K - 1;
        for (int m0 = 0; m0 < K; m0 += 4) {
            double c[4];
            #pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = tab[(m0 + i) * K + q];
            #pragma unroll
            for (int i = 0; i < 4; ++i) w = __builtin_fma(read_lane(tm, m0 + i), c[i], w);
        }
        w = (w + w - read_lane(tm, 0)) / K;
    }
    const int logt = K <= 8 ? 3 : K <= 16 ? 4 : 5, groups = 64 >> logt;
    const int t = lane & ((1 << logt) - 1), g = lane >> logt;
    const dd om = two_sum(B.D, B.rw * tab[K + (t < K ? t : K - 1)]);
    double u = 0.0;
    for (int s0 = 0; s0 < K; s0 += groups) {
        const int q = s0 + g < K ? s0 + g : K - 1;
        const double wq = __shfl(w, q);
        const dd r = two_sum(B.C, B.cw * tab[K + q]);
        const dd x = two_prod(om.hi, r.hi);
        const double xl = __builtin_fma(om.hi, r.lo, __builtin_fma(om.lo, r.hi, x.lo));
        double v = 0.0;
        if (x.hi > 0.0) {
            v = besselj_direct(P, x.hi, xl);
            if (P.half) v *= rsqrt_refined(x.hi);
        } else if (P.nu == 0 && !P.half) {
            v = 1.0;
        }
        u = __builtin_fma(s0 + g < K ? wq : 0.0, v, u);
    }
    for (int o = 32; o >= (1 << logt); o >>= 1) u += __shfl_xor(u, o);
    const int m = lane < K ? lane : K - 1;
    const double* __restrict__ col = tab + K * K + m;
    double v = 0.0;
    for (int h0 = 0; h0 < K; h0 += 4) {
        double c[4];
        #pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = col[(h0 + i) * K];
        #pragma unroll
        for (int i = 0; i < 4; ++i) v = __builtin_fma(read_lane(u, h0 + i), c[i], v);
    }
    if (lane < K) P.dcoef[(int64_t)d * kRankK + lane] = v * ((m == 0 ? 1.0 : 2.0) / K);
}

// Workgroups 0 .. n_dentry - 1: a block entry by entry each; then four blocks
// through expansions each, one per wave.
__device__ __forceinline__ void direct_body(const PlanDev& P, int bid)
{
    constexpr int kWaveSums = kRankK / 4 * 64;
    __shared__ double2 s_tab[kJtabLdsPanels * kJtabLdsStride];
    static_assert(sizeof(s_tab) >= sizeof(double) * kWaveSums * (kDirectThreads / 64) / 2, "LDS of the waves' sums");
    __shared__ double s_more[kWaveSums * (kDirectThreads / 64) / 2];
    if (bid >= P.n_dentry) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int i = (bid - P.n_dentry) * (kDirectThreads / 64) + wave;
        if (i >= P.n_drank) return;
        const int d = P.dlist[P.n_d - 1 - i];
        double* s = (wave < 2 ? reinterpret_cast<double*>(s_tab) : s_more) + (wave & 1) * kWaveSums;
        const int K = P.db[d].K;
        if (K <= 8) direct_expand<8>(P, d, s);
        else if (K <= 16) direct_expand<16>(P, d, s);
        else direct_expand<24>(P, d, s);
        return;
    }
    const DBlock D = P.db[P.dlist[bid]];
    // the panels of the table that the block's arguments can lie on
    const double x0 = P.ws[D.j0] * P.rs[D.k0], x1 = P.ws[D.j1] * P.rs[D.k1];
    const int p0 = (int)fmax(fmin((x0 - P.jtab_x0) * (1.0 / kJtabWidth) - 1e-6, (double)P.jtab_np), 0.0);
    const int p1 = (int)fmax(fmin((x1 - P.jtab_x0) * (1.0 / kJtabWidth) + 1e-6, (double)(P.jtab_np - 1)), -1.0) + 1;
    if (p0 < p1 && p1 - p0 <= kJtabLdsPanels) {
        const double2* __restrict__ g = (const double2*)P.jtab + (int64_t)p0 * (kJtabCoef / 2);
        constexpr int per = kJtabCoef / 2;
        for (int e = threadIdx.x; e < (p1 - p0) * per; e += kDirectThreads) {
            const int pn = e / per;
            s_tab[pn * kJtabLdsStride + (e - pn * per)] = g[e];
        }
        __syncthreads();
        direct_rows<true>(P, D, s_tab - p0 * kJtabLdsStride);
    } else {
        direct_rows<false>(P, D, nullptr);
    }
}

static inline int direct_workgroups(const Summary& S)
{
    return S.n_dentry + (S.n_drank + kDirectThreads / 64 - 1) / (kDirectThreads / 64);
}

__global__ __launch_bounds__(kDirectThreads) void k_direct_blocks(PlanDev P) { direct_body(P, blockIdx.x); }

__global__ __launch_bounds__(kDirectThreads) void k_direct_blocks_many(const PlanDev* __restrict__ plans,
                                                                       const WorkSeg* __restrict__ segs, int nseg)
{
    const WorkSeg w = find_seg(segs, nseg);
    direct_body(plan_of(plans, w.t), w.g0);
}

// The local blocks' rows.  In omega a block's sum sum_l C_l(omega R) t_l is
// entire and no wider than R, so on a panel of frequencies its Chebyshev
// interpolant of K terms stands for it: k_local_nodes evaluates the sum at
// each panel's K nodes (Miller's recurrence, or the half-integer table), a
// wave per 64 / K panels of a block, and turns the values into coefficients;
// the row pass then spends 2 K operations on a row instead of a recurrence
// of tens of steps with its products.  A block with fewer rows than nodes has
// the sum evaluated at its rows and the values kept.
template <int MODE>
__device__ __forceinline__ void local_nodes_body(const PlanDev& P, int bid, double* ring_all)
{
    const LocalWork W = P.lwork[bid];
    const LBlock& B = P.lb[W.blk];
    const int lane = threadIdx.x;
    const int K = B.K, per = local_wave_slots(K), slots = local_slots(B);
    const int n = slots - W.q < per ? slots - W.q : per;       // slots of this wave
    double* __restrict__ out = P.lcoef + (int64_t)(B.slot0 + W.q) * kRankK;
    int rows = 0, p = 0, t = 0;
    double om;
    const double* __restrict__ tab = P.rank_tab + rank_tab_off(K > 0 ? K : 4);
    if (K > 0) {
        p = lane / K;
        t = lane - p * K;
        if (p >= n) { p = n - 1; t = K - 1; }
        om = B.D + (rank_mid(W.q + p, B.pr, B.rw) + B.rw * tab[K + t]);
        if (om < 0.0) om = 0.0;                                 // the lowest node at omega = 0, rounded
    } else {
        rows = B.j1 - B.j0 + 1 - W.q * kRankK;
        if (rows > n * kRankK) rows = n * kRankK;
        om = P.ws[B.j0 + W.q * kRankK + (lane < rows ? lane : rows - 1)];
    }
    double v;
    if constexpr (MODE == 3) v = local_eval_half(P, W.blk, om, P.lmom);
    else v = local_eval<MODE>(P, W.blk, om, P.lmom, ring_all + lane, 64);
    if (K == 0) {
        if (lane < rows) out[lane] = v;
        return;
    }
    // lane p K + m: coefficient m = t of panel p
    const double* __restrict__ col = tab + K * K + t;
    double c = 0.0;
    for (int h = 0; h < K; ++h) c = __builtin_fma(__shfl(v, p * K + h), col[h * K], c);
    if (lane < n * K) out[p * kRankK + t] = c * ((t == 0 ? 1.0 : 2.0) / K);
}

template <int MODE>
__global__ __launch_bounds__(64) void k_local_nodes(PlanDev P)
{
    extern __shared__ double ring_all[];
    local_nodes_body<MODE>(P, blockIdx.x, ring_all);
}

template <int MODE>
__global__ __launch_bounds__(64) void k_local_nodes_many(const PlanDev* __restrict__ plans,
                                                         const WorkSeg* __restrict__ segs, int nseg)
{
    extern __shared__ double ring_all[];
    const WorkSeg w = find_seg(segs, nseg);
    local_nodes_body<MODE>(plan_of(plans, w.t), w.g0, ring_all);
}

__device__ __forceinline__ double local_series(const double* __restrict__ v, int K, double eta)
{
    double t0 = 1.0, t1 = eta, a = 0.0;
    const double e2 = eta + eta;
    for (int m = 0; m < K; m += 4) {
        #pragma unroll
        for (int u = 0; u < 4; ++u) {
            a = __builtin_fma(v[m + u], t0, a);
            const double t2 = __builtin_fma(e2, t1, -t0);
            t0 = t1;
            t1 = t2;
        }
    }
    return a;
}

// Local block lb's contribution at row j, frequency om (lb the same in every
// lane with UNI).
template <bool UNI>
__device__ __forceinline__ double local_row(const PlanDev& P, int lb, int j, double om)
{
    const LBlock& B = P.lb[lb];
    const double* __restrict__ slots = P.lcoef + (int64_t)B.slot0 * kRankK;
    double v;
    if (B.K == 0) {
        v = slots[j - B.j0];
    } else {
        const double inv = B.rw > 0.0 ? rcp_refined(B.rw) : 0.0;
        const dd a = two_sum(om, -B.D);
        int q = (int)(0.5 * __builtin_fma(a.hi, inv, (double)B.pr));
        q = q < 0 ? 0 : q > B.pr - 1 ? B.pr - 1 : q;
        const double eta = ((a.hi - rank_mid(q, B.pr, B.rw)) + a.lo) * inv;
        if constexpr (UNI) {
            const int qu = __builtin_amdgcn_readfirstlane(q);
            if (__all(q == qu)) v = local_series(slots + qu * kRankK, B.K, eta);
            else v = local_series(slots + q * kRankK, B.K, eta);
        } else {
            v = local_series(slots + q * kRankK, B.K, eta);
        }
    }
    if (P.half) v *= sqrt(2.0 / kPi * (om * B.R));
    return v;
}

// The direct block's contribution at row j, frequency om.
__device__ __forceinline__ double direct_row(const PlanDev& P, int d, int j, double om)
{
    const DBlock& B = P.db[d];
    if (B.K == 0) return P.gd[j];
    const dd a = two_sum(om, -B.D);
    const double eta = (a.hi + a.lo) * (B.rw > 0.0 ? rcp_refined(B.rw) : 0.0);
    const double v = local_series(P.dcoef + (int64_t)d * kRankK, B.K, eta);
    return P.half ? v * sqrt(om) : v;
}

// Row pass: one thread per sorted frequency walks the block tree from the
// root.  At a node the row lies either in the local side (rows j0..js) --
// local block, then the upper-right child -- or in the asymptotic side --
// asymptotic block, then the lower-left child; a direct child ends the walk
// and adds the row's part from k_direct_blocks.  g is written once, in the
// caller's order.
// NCH: the plan's channels, or 0 where the rows of every asymptotic block go
// through expansions (no row reads a grid): then one instance serves every
// order, so that a batch's transforms share a launch.
// direct = false leaves the direct blocks to k_direct_rows.
template <int NCH>
__device__ __forceinline__ void rows_body(const PlanDev& P, int bid, double* g, bool direct)
{
    const double2* __restrict__ grids = P.grids;
    const int j = bid * blockDim.x + threadIdx.x;
    if (j >= P.m) return;
    const double om = P.ws[j];
    double acc = 0.0;
    int node = P.n_nodes > 0 ? 0 : -1;
    while (node >= 0) {
        const Node nd = P.nodes[node];
        int child;
        if (j <= nd.js) {
            if (nd.lblk >= 0) {
                const int lb = nd.lblk, lbu = __builtin_amdgcn_readfirstlane(lb);
                if (__all(lb == lbu)) acc += local_row<true>(P, lbu, j, om);
                else acc += local_row<false>(P, lb, j, om);
            }
            child = nd.ur;
        } else {
            if (nd.ablk >= 0) {
                const int ab = nd.ablk, abu = __builtin_amdgcn_readfirstlane(ab);
                if constexpr (NCH == 0) {
                    if (__all(ab == abu)) acc += rank_eval<true>(P, P.ab[abu], om);
                    else acc += rank_eval<false>(P, P.ab[ab], om);
                } else {
                    if (__all(ab == abu)) acc += asym_eval<NCH, true>(P, abu, om, grids);
                    else acc += asym_eval<NCH, false>(P, ab, om, grids);
                }
            }
            child = nd.ll;
        }
        if (child <= -2) {
            if (direct) acc += direct_row(P, decode_direct(child), j, om);
            break;
        }
        node = child;
    }
    g[P.perm_w[j]] = P.sign * acc;
}

template <int NCH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_rows(PlanDev P, double* g,
                                                                                     double* const* g_slot, int direct)
{
    rows_body<NCH>(P, blockIdx.x, g_slot ? *g_slot : g, direct != 0);
}

// The rows' parts from the direct blocks, added to what k_rows wrote without
// them (the last term of a row's sum, so the same result), a workgroup a block.
__global__ __launch_bounds__(256) void k_direct_rows(PlanDev P, double* g, double* const* g_slot)
{
    double* out = g_slot ? *g_slot : g;
    const int32_t j0 = P.db[blockIdx.x].j0, j1 = P.db[blockIdx.x].j1;
    for (int32_t j = j0 + (int32_t)threadIdx.x; j <= j1; j += blockDim.x)
        out[P.perm_w[j]] += P.sign * direct_row(P, blockIdx.x, j, P.ws[j]);
}

template <int NCH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_rows_many(
    const PlanDev* __restrict__ plans, const WorkSeg* __restrict__ segs, int nseg, double* const* g_table)
{
    const WorkSeg w = find_seg(segs, nseg);
    rows_body<NCH>(plan_of(plans, w.t), w.g0, g_table[w.t], true);
}

// Brute-force reference: one thread per frequency, all points.
__global__ void k_direct_all(PlanDev P, const double* __restrict__ r, const double* __restrict__ c, int32_t n,
                             const double* __restrict__ w, int32_t m, double* __restrict__ g)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    double om = w[j];
    double acc = 0.0;
    for (int k = 0; k < n; ++k) {
        dd x = two_prod(om, r[k]);
        acc = __builtin_fma(c[k], besselj_full(P, x.hi, x.lo), acc);
    }
    g[j] = P.sign * acc;
}

// ---------------------------------------------------------------------------
static inline int cdiv64(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

template <int NCH>
static void launch_spread(const PlanDev& P, const Summary& S, hipStream_t s)
{
    const int32_t n_dense = S.n_adense, n_med = S.n_amed, n_rest = S.n_aspread - S.n_adense - S.n_amed;
    if constexpr (NCH <= kMfmaMaxChannels) {
        if (n_dense > 0)
            hipLaunchKernelGGL((k_spread_mfma<NCH, kSpreadAnchors>), dim3(n_dense), dim3(256), 0, s, P);
    }
    if constexpr (NCH <= kMfmaMedMaxChannels) {
        if (n_med > 0)
            hipLaunchKernelGGL((k_spread_mfma<NCH, kSpreadAnchorsMed>), dim3(n_med), dim3(256), 0, s, P);
    }
    if (n_rest > 0) {
        if (P.fp32)
            hipLaunchKernelGGL((k_spread<NCH, float>), dim3(n_rest * P.spread_turns), dim3(256), spread_lds_bytes<float>(P.w), s, P);
        else
            hipLaunchKernelGGL((k_spread<NCH, double>), dim3(n_rest * P.spread_turns), dim3(256), spread_lds_bytes<double>(P.w), s, P);
    }
}

// local_eval keeps J_{nu-a .. nu}, a = floor(nu/2), per lane in LDS at orders
// 2 and up.
static size_t local_nodes_lds(const PlanDev& P)
{
    return P.half || P.nu <= 1 ? 0 : (size_t)((P.nu >> 1) + 1) * 64 * sizeof(double);
}

// The instance of k_local_nodes: orders 0 and 1, the general one, half-integer
// orders.
static int local_mode(const PlanDev& P) { return P.half ? 3 : P.nu <= 1 ? P.nu : 2; }

static void launch_local_nodes(const PlanDev& P, hipStream_t s)
{
    const int mode = local_mode(P);
    auto k = mode == 0 ? k_local_nodes<0> : mode == 1 ? k_local_nodes<1> : mode == 2 ? k_local_nodes<2> : k_local_nodes<3>;
    hipLaunchKernelGGL(k, dim3(P.n_lwork), dim3(64), local_nodes_lds(P), s, P);
}

// Calls f with std::integral_constant<int, nch>; nch is one of the instantiated
// channel counts (every even count up to 16, multiples of 4 up to 40).
template <class F>
static void dispatch_channels(int nch, F&& f)
{
    switch (nch) {
    case 2: f(std::integral_constant<int, 2>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 6: f(std::integral_constant<int, 6>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    case 10: f(std::integral_constant<int, 10>()); break;
    case 12: f(std::integral_constant<int, 12>()); break;
    case 14: f(std::integral_constant<int, 14>()); break;
    case 16: f(std::integral_constant<int, 16>()); break;
    case 20: f(std::integral_constant<int, 20>()); break;
    case 24: f(std::integral_constant<int, 24>()); break;
    case 28: f(std::integral_constant<int, 28>()); break;
    case 32: f(std::integral_constant<int, 32>()); break;
    case 36: f(std::integral_constant<int, 36>()); break;
    default: f(std::integral_constant<int, 40>()); break;
    }
}

// The row pass's channel count: 0 where no row reads a grid.
static int rows_channels(const PlanDev& P) { return P.n_gridrows > 0 ? P.nch : 0; }

template <class F>
static void dispatch_rows(int nch, F&& f)
{
    if (nch == 0) f(std::integral_constant<int, 0>());
    else dispatch_channels(nch, f);
}

static inline void mark(hipEvent_t* marks, int i, hipStream_t s)
{
    if (marks && marks[i]) (void)hipEventRecord(marks[i], s);
}

hipError_t launch_fill(double* x, int64_t n, double v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_value, dim3(cdiv64(n, 256)), dim3(256), 0, s, x, n, v);
    return hipGetLastError();
}

hipError_t launch_set_pointers(void** table, const void* const* ptrs, int count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    if (count > 224) return hipErrorInvalidValue;
    PtrArgs a;
    for (int i = 0; i < count; ++i) a.p[i] = const_cast<void*>(ptrs[i]);
    hipLaunchKernelGGL(k_set_pointers, dim3(1), dim3(256), 0, s, table, a, count);
    return hipGetLastError();
}

// Lines per tile for transforms of length 2^logL.
static int fft_log_lines(int logL)
{
    int l = 0;
    while ((1 << (l + 1)) <= kFftMaxLines && (1 << (l + 1 + logL)) <= kFftTilePts) ++l;
    return l;
}

static size_t fft_lds_bytes(int logL, int logLines)
{
    return sizeof(double2) * ((size_t)((1 << logL) + 1) * (1 << logLines) + (1 << logL));
}

// Two passes for N <= 2^16 (N1 = 2^floor(logN/2)), three beyond; every pass
// length is at most 2^8 and at least 2^6 for the sizes that reach here.
// pass 0: the inner column pass over nb (three-pass sizes only), 1: the
// column pass over na, 2: the row pass.  Returns false when the size class
// has no such pass; else its arguments, workgroups and LDS bytes.
static bool fft_pass(const FftClass& K, int nch, int pass, FftPass& F, int& blocks, size_t& lds)
{
    const int logN = K.log2n;
    const int ntr = K.count * nch;
    int logN1, logNa, logNb;
    if (logN <= 16) {
        logN1 = logN / 2; logNa = logN - logN1; logNb = 0;
    } else {
        logN1 = logN / 3; logNa = (logN - logN1) / 2; logNb = logN - logN1 - logNa;
    }
    const int64_t N1 = int64_t(1) << logN1, Na = int64_t(1) << logNa, Nb = int64_t(1) << logNb;
    F = FftPass{};
    F.first = K.first;
    F.logN = logN;
    F.scratch_off = K.scratch_off;
    FftCol& c = F.C;
    if (pass == 0) {
        if (logNb == 0) return false;
        c.logL = logNb; c.logLines = fft_log_lines(logNb); c.logBlo = logN1 + logNa; c.to_scratch = 0;
        c.in_es = N1 * Na; c.in_hs = 0; c.out_es = N1 * Na; c.out_hs = 0;
        c.lo_mask = ~(N1 - 1); c.kmul = 1; c.from_grid = 1;
    } else if (pass == 1) {
        c.logL = logNa; c.logLines = fft_log_lines(logNa); c.logBlo = logN1; c.to_scratch = 1;
        c.in_es = N1; c.in_hs = N1 * Na; c.out_es = N1 * Nb; c.out_hs = N1;
        c.lo_mask = ~int64_t(0); c.kmul = Nb; c.from_grid = logNb == 0 ? 1 : 0;
    } else {
        c.logL = logN1; c.logLines = fft_log_lines(logN1);
        blocks = ntr * (int)((int64_t(1) << (logN - logN1)) >> c.logLines);
        lds = fft_lds_bytes(c.logL, c.logLines);
        return true;
    }
    blocks = ntr * (int)((int64_t(1) << logN) >> (c.logL + c.logLines));
    lds = fft_lds_bytes(c.logL, c.logLines);
    return true;
}

static void launch_fft_large(const PlanDev& P, const FftClass& K, hipStream_t s)
{
    for (int pass = 0; pass < 3; ++pass) {
        FftPass F;
        int blocks = 0;
        size_t lds = 0;
        if (!fft_pass(K, P.nch, pass, F, blocks, lds)) continue;
        if (pass < 2) hipLaunchKernelGGL(k_fft_col, dim3(blocks), dim3(256), lds, s, P, F);
        else hipLaunchKernelGGL(k_fft_row, dim3(blocks), dim3(256), lds, s, P, F);
    }
}

// Transforms of at most this many points and frequencies run on one stream.
// At half-integer orders z is so small that the direct entries lie below the
// table of J_nu and run a recurrence each, so the fork pays earlier: 155 us a
// pass on one stream and 116 forked at 2500 x 400, order 1.5, but 86 and 93 at
// 300 x 300, where the host's launches are the longer.
constexpr int64_t kForkMin = 1 << 13, kHalfForkMin = 1 << 11;
// Above this many, and where there are grids, the rank blocks leave the main
// stream too.
constexpr int64_t kRankForkMin = 1 << 14;
// A direct block of more than this many entries below the table of J_nu, a
// recurrence each (half-integer orders and high ones), keeps k_direct_blocks
// busy for longer than the other stages of most transforms, 100 to 280 us: then
// the rank blocks stay on the main stream whatever the sizes, and the rows do
// not wait for the direct blocks.
constexpr int32_t kDirectHeavy = 2048;
// The other executions whose rows do not wait for the direct blocks: few rows,
// whose pass is a chain of latencies as long as the main stream's whole work
// where that has no FFT, of this many points and frequencies or more (without
// rank blocks, with them).
constexpr int64_t kLateRows = 1024, kLateMin = 1 << 14, kLateRankMin = 1 << 17;

hipError_t launch_execute(const PlanDev& P, const Summary& S, const ExecBuffers& B, const FftClass* cls, int ncls,
                          const IoArgs& io, hipStream_t s, hipEvent_t* marks, const ExecFork* fork)
{
    if (P.m == 0) return hipSuccess;
    if (P.n == 0) {   // a fill kernel, not a memset node, so the call can be captured in a graph
        hipLaunchKernelGGL(k_zero_output, dim3(cdiv64(P.m, 256)), dim3(256), 0, s, io.g, io.g_slot, (int64_t)P.m);
        return hipGetLastError();
    }
    mark(marks, 0, s);
    hipLaunchKernelGGL(k_gather, dim3(cdiv64(P.n, 256)), dim3(256), 0, s, P, io.c, io.c_slot,
                       io.scale_by_points ? 1 : 0);
    mark(marks, 1, s);
    // the local moments, the rank blocks and the direct blocks read only the
    // gathered weights and run beside the grids' kernels.  A small transform's
    // kernels are shorter than the fork's events and waits take the host: plan
    // and pass at 2000 x 2000 173 us on one stream, 220 forked; passes of
    // 5229 x 10761 and back, order 18, 277 and 222, but 244 with the rank
    // blocks on the side stream (the host's launches of which hold the grids'
    // up); passes of 20000 x 20000 and back 268 us with those on the main
    // stream, 233 on the side one.  Without grids the rank blocks are the main
    // stream's work.
    const bool forked = fork && fork->side && (S.n_litems > 0 || P.n_d > 0) &&
                        (int64_t)P.n + P.m > (P.half ? kHalfForkMin : kForkMin);
    // The rows wait for the local rows' expansions and, as a rule, for the
    // direct blocks.  Where those are the side stream's long work, the rows run
    // beside them instead and the direct blocks' parts are added at the end.
    // Microseconds a pass with rows that wait, and with rows that do not:
    //   order 5.5, radial, 30000 x 500 (direct blocks 236)   359   286
    //   order 3/2, uniform, 100000 x 100000                  342   299
    //   order 40, radial, 30000 x 500                        441   306
    //   order 0, radial, 300000 x 500, at 1e-6               143   115
    // Elsewhere the addition only costs its launch:
    //   order 0, uniform, 500 x 300000, at 1e-6              101   107
    //   order 0, uniform, 30000 x 30000, at 1e-6             130   143
    const bool heavy = forked && S.d_area > kDirectHeavy;
    const bool rank_aside = forked && !heavy && P.grid_cells > 0 && (int64_t)P.n + P.m > kRankForkMin;
    const bool late = heavy || (forked && P.n_d > 0 && S.n_fft == 0 && P.m <= kLateRows &&
                                (int64_t)P.n + P.m > (P.rank ? kLateRankMin : kLateMin));
    const hipStream_t ls = forked ? fork->side : s, ks = rank_aside ? fork->side : s;
    auto launch_local = [&] {
        if (S.n_litems == 0) return;
        if (lmom_width(P.L) == 32) hipLaunchKernelGGL(k_lmom<32>, dim3(S.n_litems), dim3(64), 0, ls, P);
        else hipLaunchKernelGGL(k_lmom<64>, dim3(S.n_litems), dim3(64), 0, ls, P);
        if (S.n_litems > S.n_l)   // some block has several items
            hipLaunchKernelGGL(k_lmom_reduce, dim3(lmom_reduce_blocks(S.n_l, P.L)), dim3(256), 0, ls, P);
        launch_local_nodes(P, ls);
    };
    auto launch_rank_moments = [&] {
        if (rank_moments_blocks(S) > 0)
            hipLaunchKernelGGL(k_rank_moments, dim3(rank_moments_blocks(S)), dim3(64 * kRankWaves), 0, ks, P);
    };
    auto launch_rank_rows = [&] {
        if (S.n_cpan == 0) return;
        hipLaunchKernelGGL(k_rank_weights, dim3(rank_weights_blocks(S)), dim3(256), 0, ks, P);
        if (S.n_tmulti > 0)
            hipLaunchKernelGGL(k_rank_translate, dim3(S.n_tmulti), dim3(kRankTransThreads), 0, ks, P);
    };
    auto launch_direct = [&] {
        if (P.n_d > 0) hipLaunchKernelGGL(k_direct_blocks, dim3(direct_workgroups(S)), dim3(kDirectThreads), 0, ls, P);
    };
    if (forked) {
        hipError_t e = hipEventRecord(fork->ev_fork, s);
        if (e == hipSuccess) e = hipStreamWaitEvent(ls, fork->ev_fork, 0);
        if (e != hipSuccess) return e;
    }
    // what the rows wait for ends on the side stream: with late, before the direct blocks
    auto join_rows = [&](bool here) { return here ? hipEventRecord(fork->ev_join, ls) : hipSuccess; };
    hipError_t e_join = hipSuccess;
    if (!rank_aside) {
        launch_local();
        e_join = join_rows(late);
        if (forked) launch_direct();
    }
    mark(marks, 2, s);
    if (!rank_aside) launch_rank_moments();
    dispatch_channels(P.nch, [&](auto k) { launch_spread<decltype(k)::value>(P, S, s); });
    mark(marks, 3, s);
    if (rank_aside) {
        launch_rank_moments();
        launch_local();
    }
    launch_rank_rows();
    if (rank_aside) {
        if (e_join == hipSuccess) e_join = join_rows(late);
        launch_direct();
    }
    if (e_join == hipSuccess) e_join = late ? hipEventRecord(fork->ev_fork, ls) : join_rows(forked);
    if (e_join != hipSuccess) return e_join;
    if (P.grid_cells > 0) {
        if (P.fp32)
            hipLaunchKernelGGL(k_spread_reduce<float2>, dim3(cdiv64(P.grid_units, 256)), dim3(256), 0, s, P);
        else
            hipLaunchKernelGGL(k_spread_reduce<double2>, dim3(cdiv64(P.grid_units, 256)), dim3(256), 0, s, P);
    }
    mark(marks, 4, s);
    if (P.small.n > 0 && P.small.wg0[P.small.n] > 0)
        hipLaunchKernelGGL(k_fft_small, dim3(P.small.wg0[P.small.n]), dim3(256),
                           sizeof(double2) << P.small.max_log2n, s, P);
    for (int q = 0; q < ncls; ++q)
        if (cls[q].log2n > 12) launch_fft_large(P, cls[q], s);
    if (S.n_fpan > 0) hipLaunchKernelGGL(k_fft_nodes, dim3(S.n_fpan), dim3(256), 0, s, P);
    mark(marks, 5, s);
    if (!forked) launch_direct();
    if (forked) {
        const hipError_t e = hipStreamWaitEvent(s, fork->ev_join, 0);
        if (e != hipSuccess) return e;
    }
    mark(marks, 6, s);                               // after the wait: the rows' interval holds them alone
    dispatch_rows(rows_channels(P), [&](auto k) {
        hipLaunchKernelGGL(k_rows<decltype(k)::value>, dim3(cdiv64(P.m, 256)), dim3(256), 0, s, P, io.g, io.g_slot,
                           late ? 0 : 1);
    });
    mark(marks, 7, s);
    if (late) {
        const hipError_t e = hipStreamWaitEvent(s, fork->ev_fork, 0);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_direct_rows, dim3(P.n_d), dim3(256), 0, s, P, io.g, io.g_slot);
    }
    mark(marks, 8, s);
    return hipGetLastError();
}

void small_fft_table(PlanDev& P, const FftClass* cls, int ncls)
{
    SmallFfts& F = P.small;
    F = SmallFfts{};
    int wg = 0;
    for (int q = 0; q < ncls; ++q) {
        const FftClass& C = cls[q];
        if (C.log2n > 12 || F.n == 8) continue;
        F.log2n[F.n] = C.log2n;
        F.first[F.n] = C.first;
        F.wg0[F.n] = wg;
        wg += C.count * P.nch;
        F.max_log2n = C.log2n > F.max_log2n ? C.log2n : F.max_log2n;
        ++F.n;
    }
    F.wg0[F.n] = wg;
}

// ---------------------------------------------------------------------------
// Batches: the launch list.  Kinds in execution order; a launch's variant is
// its channel count (spreading, grid rows) or local-row mode.
// ---------------------------------------------------------------------------
enum BatchKind : int32_t {
    kZeroOut, kGather, kLmom, kLmomReduce, kLocalNodes, kRankMoments, kRankWeights, kRankTranslate, kSpreadMfma, kSpreadMfmaMed, kSpreadVec, kSpreadReduce, kFftSmall,
    kFftPass0, kFftPass1, kFftPass2, kFftNodes, kDirect, kRows
};

void build_batch_schedule(const BatchTransform* tr, int count, const int* order, BatchSchedule& out)
{
    out = BatchSchedule{};
    std::vector<WorkSeg> segs;
    std::vector<FftSeg> fsegs;
    // one launch of `kind` over the transforms accepted by `take`, which gives
    // a transform's workgroups (0: none) and may raise the launch's LDS bytes
    auto add = [&](int32_t kind, int32_t variant, int32_t fp32, int32_t threads, auto&& take) {
        BatchLaunch L{};
        L.kind = kind; L.variant = variant; L.fp32 = fp32; L.threads = threads;
        L.seg0 = (int32_t)segs.size();
        int64_t g = 0;
        for (int q = 0; q < count; ++q) {
            const int t = order[q];
            size_t lds = 0;
            const int64_t wg = take(tr[t], lds);
            if (wg <= 0) continue;
            segs.push_back(WorkSeg{t, (int32_t)g});
            g += wg;
            if (lds > L.lds) L.lds = lds;
        }
        L.nseg = (int32_t)segs.size() - L.seg0;
        L.blocks = (int32_t)g;
        if (L.nseg > 0) out.launches.push_back(L);
    };
    auto live = [](const PlanDev& P) { return P.n > 0 && P.m > 0; };
    add(kZeroOut, 0, 0, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
        return (T.P->n == 0 && T.P->m > 0) ? cdiv64(T.P->m, 256) : 0;
    });
    add(kGather, 0, 0, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) ? cdiv64(T.P->n, 256) : 0;
    });
    for (const int width : {32, 64})
        add(kLmom, width, 0, 64, [&](const BatchTransform& T, size_t&) -> int64_t {
            return live(*T.P) && lmom_width(T.P->L) == width ? T.S->n_litems : 0;
        });
    add(kLmomReduce, 0, 0, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) && T.S->n_litems > T.S->n_l ? lmom_reduce_blocks(T.S->n_l, T.P->L) : 0;
    });
    for (int mode = 0; mode < 4; ++mode)
        add(kLocalNodes, mode, 0, 64, [&](const BatchTransform& T, size_t& lds) -> int64_t {
            if (!live(*T.P) || local_mode(*T.P) != mode) return 0;
            lds = local_nodes_lds(*T.P);
            return T.S->n_lwork;
        });
    add(kRankMoments, 0, 0, 64 * kRankWaves, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) ? rank_moments_blocks(*T.S) : 0;
    });
    add(kRankWeights, 0, 0, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) ? rank_weights_blocks(*T.S) : 0;
    });
    add(kRankTranslate, 0, 0, kRankTransThreads, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) ? T.S->n_tmulti : 0;
    });
    // the channel counts and precisions present
    std::vector<std::pair<int, int>> variants;
    for (int t = 0; t < count; ++t) {
        const std::pair<int, int> v{tr[t].P->nch, tr[t].P->fp32};
        if (live(*tr[t].P) && std::find(variants.begin(), variants.end(), v) == variants.end()) variants.push_back(v);
    }
    std::sort(variants.begin(), variants.end());
    for (const auto& v : variants) {
        const int nch = v.first, fp32 = v.second;
        auto same = [&](const PlanDev& P) { return live(P) && P.nch == nch && P.fp32 == fp32; };
        if (nch <= kMfmaMaxChannels)   // static LDS: no launch bytes
            add(kSpreadMfma, nch, fp32, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
                return same(*T.P) ? T.S->n_adense : 0;
            });
        if (nch <= kMfmaMedMaxChannels)
            add(kSpreadMfmaMed, nch, fp32, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
                return same(*T.P) ? T.S->n_amed : 0;
            });
        add(kSpreadVec, nch, fp32, 256, [&](const BatchTransform& T, size_t& lds) -> int64_t {
            if (!same(*T.P)) return 0;
            lds = fp32 ? spread_lds_bytes<float>(T.P->w) : spread_lds_bytes<double>(T.P->w);
            return (int64_t)(T.S->n_aspread - T.S->n_adense - T.S->n_amed) * T.P->spread_turns;
        });
    }
    for (int fp32 = 0; fp32 <= 1; ++fp32)
        add(kSpreadReduce, 0, fp32, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
            return live(*T.P) && T.P->fp32 == fp32 ? cdiv64(T.P->grid_units, 256) : 0;
        });
    add(kFftSmall, 0, 0, 256, [&](const BatchTransform& T, size_t& lds) -> int64_t {
        const SmallFfts& F = T.P->small;
        if (!live(*T.P) || F.n == 0) return 0;
        lds = sizeof(double2) << F.max_log2n;
        return F.wg0[F.n];
    });
    for (int pass = 0; pass < 3; ++pass) {
        BatchLaunch L{};
        L.kind = kFftPass0 + pass;
        L.threads = 256;
        L.seg0 = (int32_t)fsegs.size();
        int64_t g = 0;
        for (int q = 0; q < count; ++q) {
            const int t = order[q];
            if (!live(*tr[t].P)) continue;
            for (int c = 0; c < tr[t].ncls; ++c) {
                const FftClass& K = tr[t].cls[c];
                if (K.log2n <= 12) continue;
                FftSeg f{};
                int blocks = 0;
                size_t lds = 0;
                if (!fft_pass(K, tr[t].P->nch, pass, f.F, blocks, lds) || blocks <= 0) continue;
                f.t = t;
                f.g0 = (int32_t)g;
                fsegs.push_back(f);
                g += blocks;
                if (lds > L.lds) L.lds = lds;
            }
        }
        L.nseg = (int32_t)fsegs.size() - L.seg0;
        L.blocks = (int32_t)g;
        if (L.nseg > 0) out.launches.push_back(L);
    }
    add(kFftNodes, 0, 0, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) ? T.S->n_fpan : 0;
    });
    add(kDirect, 0, 0, kDirectThreads, [&](const BatchTransform& T, size_t&) -> int64_t {
        return live(*T.P) ? direct_workgroups(*T.S) : 0;
    });
    std::vector<int> chans;
    for (int t = 0; t < count; ++t) {
        const int c = rows_channels(*tr[t].P);
        if (live(*tr[t].P) && std::find(chans.begin(), chans.end(), c) == chans.end()) chans.push_back(c);
    }
    std::sort(chans.begin(), chans.end());
    for (int nch : chans)
        add(kRows, nch, 0, 256, [&](const BatchTransform& T, size_t&) -> int64_t {
            return live(*T.P) && rows_channels(*T.P) == nch ? cdiv64(T.P->m, 256) : 0;
        });
    // the device tables: PlanDev[count], WorkSeg[], FftSeg[] (each 256-byte aligned)
    auto align = [](size_t x) { return (x + 255) & ~(size_t)255; };
    out.segs_off = align(sizeof(PlanDev) * (size_t)count);
    out.fsegs_off = out.segs_off + align(sizeof(WorkSeg) * segs.size());
    out.table.assign(out.fsegs_off + sizeof(FftSeg) * fsegs.size(), 0);
    for (int t = 0; t < count; ++t) std::memcpy(out.table.data() + sizeof(PlanDev) * t, tr[t].P, sizeof(PlanDev));
    if (!segs.empty()) std::memcpy(out.table.data() + out.segs_off, segs.data(), sizeof(WorkSeg) * segs.size());
    if (!fsegs.empty()) std::memcpy(out.table.data() + out.fsegs_off, fsegs.data(), sizeof(FftSeg) * fsegs.size());
}

hipError_t launch_execute_many(const BatchSchedule& S, const void* table_dev, void* const* c_table,
                               void* const* g_table, hipStream_t s, const ExecFork* fork)
{
    const char* base = (const char*)table_dev;
    const PlanDev* plans = (const PlanDev*)base;
    const WorkSeg* segs = (const WorkSeg*)(base + S.segs_off);
    const FftSeg* fsegs = (const FftSeg*)(base + S.fsegs_off);
    const double* const* cin = (const double* const*)c_table;
    double* const* gout = (double* const*)g_table;
    // with `fork`: the local moments, the direct blocks and (where there are
    // grids) the rank blocks on its side stream, forked at the first of them (after the gather) and
    // joined before the row pass (or at the end)
    bool forked = false, joined = false, grids = false;
    for (const BatchLaunch& L : S.launches) grids |= L.kind == kSpreadReduce;
    auto join = [&]() -> hipError_t {
        hipError_t e = hipEventRecord(fork->ev_join, fork->side);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, fork->ev_join, 0);
        joined = true;
        return e;
    };
    for (const BatchLaunch& L : S.launches) {
        const dim3 grid(L.blocks), block(L.threads);
        const bool side_kind = L.kind == kLmom || L.kind == kLmomReduce || L.kind == kLocalNodes || L.kind == kDirect ||
                               (grids && (L.kind == kRankMoments || L.kind == kRankWeights || L.kind == kRankTranslate));
        hipStream_t st = s;
        if (fork && side_kind && !joined) {
            if (!forked) {
                hipError_t e = hipEventRecord(fork->ev_fork, s);
                if (e == hipSuccess) e = hipStreamWaitEvent(fork->side, fork->ev_fork, 0);
                if (e != hipSuccess) return e;
                forked = true;
            }
            st = fork->side;
        }
        if (forked && !joined && L.kind == kRows) {
            const hipError_t e = join();
            if (e != hipSuccess) return e;
        }
        const WorkSeg* sg = segs + L.seg0;
        const FftSeg* fs = fsegs + L.seg0;
        switch (L.kind) {
        case kZeroOut: hipLaunchKernelGGL(k_zero_output_many, grid, block, 0, s, plans, sg, L.nseg, gout); break;
        case kGather: hipLaunchKernelGGL(k_gather_many, grid, block, 0, s, plans, sg, L.nseg, cin); break;
        case kLmom:
            if (L.variant == 32) hipLaunchKernelGGL(k_lmom_many<32>, grid, block, 0, st, plans, sg, L.nseg);
            else hipLaunchKernelGGL(k_lmom_many<64>, grid, block, 0, st, plans, sg, L.nseg);
            break;
        case kLmomReduce: hipLaunchKernelGGL(k_lmom_reduce_many, grid, block, 0, st, plans, sg, L.nseg); break;
        case kLocalNodes:
            if (L.variant == 0) hipLaunchKernelGGL(k_local_nodes_many<0>, grid, block, L.lds, st, plans, sg, L.nseg);
            else if (L.variant == 1) hipLaunchKernelGGL(k_local_nodes_many<1>, grid, block, L.lds, st, plans, sg, L.nseg);
            else if (L.variant == 2) hipLaunchKernelGGL(k_local_nodes_many<2>, grid, block, L.lds, st, plans, sg, L.nseg);
            else hipLaunchKernelGGL(k_local_nodes_many<3>, grid, block, L.lds, st, plans, sg, L.nseg);
            break;
        case kRankMoments:
            hipLaunchKernelGGL(k_rank_moments_many, grid, block, 0, st, plans, sg, L.nseg);
            break;
        case kRankWeights: hipLaunchKernelGGL(k_rank_weights_many, grid, block, 0, st, plans, sg, L.nseg); break;
        case kRankTranslate: hipLaunchKernelGGL(k_rank_translate_many, grid, block, 0, st, plans, sg, L.nseg); break;
        case kSpreadMfma:
        case kSpreadMfmaMed:
            dispatch_channels(L.variant, [&](auto k) {
                constexpr int NCH = decltype(k)::value;
                if constexpr (NCH <= kMfmaMaxChannels) {
                    if (L.kind == kSpreadMfma)
                        hipLaunchKernelGGL((k_spread_mfma_many<NCH, kSpreadAnchors>), grid, block, 0, s, plans, sg,
                                           L.nseg);
                }
                if constexpr (NCH <= kMfmaMedMaxChannels) {
                    if (L.kind == kSpreadMfmaMed)
                        hipLaunchKernelGGL((k_spread_mfma_many<NCH, kSpreadAnchorsMed>), grid, block, 0, s, plans,
                                           sg, L.nseg);
                }
            });
            break;
        case kSpreadVec:
            dispatch_channels(L.variant, [&](auto k) {
                constexpr int NCH = decltype(k)::value;
                if (L.fp32) hipLaunchKernelGGL((k_spread_many<NCH, float>), grid, block, L.lds, s, plans, sg, L.nseg);
                else hipLaunchKernelGGL((k_spread_many<NCH, double>), grid, block, L.lds, s, plans, sg, L.nseg);
            });
            break;
        case kSpreadReduce:
            if (L.fp32) hipLaunchKernelGGL(k_spread_reduce_many<float2>, grid, block, 0, s, plans, sg, L.nseg);
            else hipLaunchKernelGGL(k_spread_reduce_many<double2>, grid, block, 0, s, plans, sg, L.nseg);
            break;
        case kFftSmall: hipLaunchKernelGGL(k_fft_small_many, grid, block, L.lds, s, plans, sg, L.nseg); break;
        case kFftPass0:
        case kFftPass1: hipLaunchKernelGGL(k_fft_col_many, grid, block, L.lds, s, plans, fs, L.nseg); break;
        case kFftPass2: hipLaunchKernelGGL(k_fft_row_many, grid, block, L.lds, s, plans, fs, L.nseg); break;
        case kFftNodes: hipLaunchKernelGGL(k_fft_nodes_many, grid, block, 0, s, plans, sg, L.nseg); break;
        case kDirect: hipLaunchKernelGGL(k_direct_blocks_many, grid, block, 0, st, plans, sg, L.nseg); break;
        case kRows:
            dispatch_rows(L.variant, [&](auto k) {
                hipLaunchKernelGGL((k_rows_many<decltype(k)::value>), grid, block, 0, s, plans, sg, L.nseg, gout);
            });
            break;
        default: return hipErrorInvalidValue;
        }
    }
    if (forked && !joined) {
        const hipError_t e = join();
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

hipError_t launch_half_difference(const double* w, const double* a, const double* b, double* out, int32_t n,
                                  hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_half_difference, dim3(cdiv64(n, 256)), dim3(256), 0, s, w, a, b, out, n);
    return hipGetLastError();
}

hipError_t launch_direct(const PlanDev& P, const double* r, const double* c, int32_t n, const double* w, int32_t m,
                         double* g, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_direct_all, dim3(cdiv64(m, 128)), dim3(128), 0, s, P, r, c, n, w, m, g);
    return hipGetLastError();
}

}  // namespace nuht
