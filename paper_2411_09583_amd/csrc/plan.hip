// plan.hip -- device-side planning: validation and sorting of the points and
// frequencies, the staircase of the local region, the block subdivision of
// Alg. 1 (Sec. 4.1), per-block parameters and the column work items.
#include "nuht_device.h"
#include "nuht_launch.h"

#include <type_traits>

namespace nuht {

// ---------------------------------------------------------------------------
// LSD radix sort, 8-bit digits, of two independent segments at once (the
// points and the frequencies).  Segment s owns tiles [tile0[s], tile0[s+1])
// and elements [off[s], off[s+1]).  Launches: the keys with the first pass's
// per-tile digit counts, then per pass the counts (from the second pass on),
// their scan and the scatter.
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortRounds = 8;
constexpr int kSortTile = kSortThreads * kSortRounds;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortWaveRounds = kSortTile / kSortThreads;   // 64-key rounds per wave (= kSortRounds)

// Orders one wave's LDS accesses around it (lanes read a counter that one
// lane of the same wave then updates).
__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct SortSegs {
    int32_t off[3];      // element offsets of segments 0, 1 and the end
    int32_t tile0[3];    // tile offsets
    int32_t hoff[3];     // histogram offsets (256 * tiles per segment)
};

__device__ __forceinline__ int tile_segment(const SortSegs& S, int tile)
{
    return tile >= S.tile0[1] ? 1 : 0;
}

// Lanes of the wave whose digit d equals the calling lane's (8 ballots, one
// per bit), among the lanes with `valid` set.
__device__ __forceinline__ uint64_t digit_peers(int d, bool valid)
{
    uint64_t peers = __ballot(valid);
    #pragma unroll
    for (int b = 0; b < 8; ++b) {
        uint64_t m = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? m : ~m;
    }
    return peers;
}

// Digit counts of a tile's keys held 64 per round by the waves of the block
// (digit -1: no key): in each round the lowest lane of each group of equal
// digits adds the group's size, so a digit shared by the whole round (the
// high bytes of clustered keys) costs one LDS atomic, not 64.
__device__ __forceinline__ void tile_digit_counts(const int (&dg)[kSortWaveRounds], int32_t* h)
{
    const int lane = threadIdx.x & 63;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    #pragma unroll
    for (int r = 0; r < kSortWaveRounds; ++r) {
        const bool valid = dg[r] >= 0;
        const uint64_t peers = digit_peers(dg[r], valid);
        if (valid && (peers & lt_mask) == 0) atomicAdd(&h[dg[r]], (int32_t)__popcll(peers));
    }
}

// Keys of both segments (the points, then the frequencies) in the sort's
// tiles: a nonnegative double's bit pattern, read as an unsigned integer, is
// monotone in its value, so sorting the bits sorts the values (-0.0 maps to
// 0).  Values are the caller indices within the segment.  Each tile also
// stores its digit counts for the first pass (tile-major, one row of 256 per
// tile) and errs[tile] = 1 if it holds a negative, NaN or infinite input
// (else 0).  Wave v of a tile takes its keys v * 512 .. v * 512 + 511.
__global__ __launch_bounds__(kSortThreads) void k_make_keys(const double* __restrict__ r,
                                                             const double* __restrict__ w, SortSegs S,
                                                             uint64_t* __restrict__ key, int32_t* __restrict__ val,
                                                             int32_t* __restrict__ hist, int32_t* __restrict__ errs)
{
    __shared__ int32_t h[256];
    const int tile = blockIdx.x;
    const int seg = tile_segment(S, tile);
    const int lt = tile - S.tile0[seg];
    const int base = S.off[seg], end = S.off[seg + 1];
    const double* __restrict__ x = seg ? w : r;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wbase = base + lt * kSortTile + wave * 64 * kSortWaveRounds;
    int dg[kSortWaveRounds];
    bool bad = false;
    #pragma unroll
    for (int q = 0; q < kSortWaveRounds; ++q) {
        const int i = wbase + q * 64 + lane;
        dg[q] = -1;
        if (i < end) {
            const double v = x[i - base];
            const bool ok = (v >= 0.0) && (v <= 1.7976931348623157e308);
            bad |= !ok;
            const uint64_t k = (v == 0.0 || !ok) ? 0ull : (uint64_t)__double_as_longlong(v);
            key[i] = k;
            val[i] = i - base;
            dg[q] = (int)(k & 255);
        }
    }
    h[threadIdx.x] = 0;
    __syncthreads();
    tile_digit_counts(dg, h);
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    hist[S.hoff[seg] + lt * 256 + threadIdx.x] = h[threadIdx.x];
    if (threadIdx.x == 0) errs[tile] = any_bad ? 1 : 0;
}

// Digit counts of one tile for a later pass (tile-major, one row of 256 per
// tile); wave v takes the tile's keys v * 512 .. v * 512 + 511, all loaded
// first.
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const uint64_t* __restrict__ key, SortSegs S,
                                                             int shift, int32_t* __restrict__ hist)
{
    __shared__ int32_t h[256];
    const int tile = blockIdx.x;
    const int seg = tile_segment(S, tile);
    const int lt = tile - S.tile0[seg];
    const int end = S.off[seg + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wbase = S.off[seg] + lt * kSortTile + wave * 64 * kSortWaveRounds;
    int dg[kSortWaveRounds];
    #pragma unroll
    for (int q = 0; q < kSortWaveRounds; ++q) {
        const int i = wbase + q * 64 + lane;
        dg[q] = i < end ? (int)((key[i] >> shift) & 255) : -1;
    }
    h[threadIdx.x] = 0;
    __syncthreads();
    tile_digit_counts(dg, h);
    __syncthreads();
    hist[S.hoff[seg] + lt * 256 + threadIdx.x] = h[threadIdx.x];
}

// 1 in *flag if any of the n tile flags is set, else 0 (one block).
__global__ __launch_bounds__(256) void k_reduce_errs(const int32_t* __restrict__ errs, int32_t n,
                                                     int32_t* __restrict__ flag)
{
    int any = 0;
    for (int32_t i = threadIdx.x; i < n; i += blockDim.x) any |= errs[i];
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) *flag = any ? 1 : 0;
}

// ---------------------------------------------------------------------------
// Block-wide scans (1024 threads = 16 waves): inclusive scans inside each wave
// with cross-lane shuffles, then a scan of the 16 wave totals.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ T wave_incl_scan(T v)
{
    const int lane = threadIdx.x & 63;
    #pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan of v[q] over the block of NW waves (at most 16); tot[q]
// receives the block total.
template <class T, int NV, int NW = 16>
__device__ void block_scan(T (&v)[NV], T (&tot)[NV], T (*wsum)[16])
{
    static_assert(NW >= 1 && NW <= 16, "one wave scans the wave totals");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T incl[NV];
    #pragma unroll
    for (int q = 0; q < NV; ++q) incl[q] = wave_incl_scan(v[q]);
    if (lane == 63) {
        #pragma unroll
        for (int q = 0; q < NV; ++q) wsum[q][wave] = incl[q];
    }
    __syncthreads();
    if (wave == 0) {
        #pragma unroll
        for (int q = 0; q < NV; ++q) {
            T x = lane < NW ? wsum[q][lane] : T(0);
            x = wave_incl_scan(x);
            if (lane < NW) wsum[q][lane] = x;
        }
    }
    __syncthreads();
    #pragma unroll
    for (int q = 0; q < NV; ++q) {
        T base = wave > 0 ? wsum[q][wave - 1] : T(0);
        tot[q] = wsum[q][NW - 1];
        v[q] = base + incl[q] - v[q];
    }
    __syncthreads();
}

// Exclusive scan over the block (NW waves) of VPT consecutive values per
// thread (NV independent sequences): each thread's own running sums, then a
// block scan of the thread totals.  tot receives the block totals.
template <int NV, int VPT, int NW = 16>
__device__ void block_scan_vpt(int64_t (&v)[VPT][NV], int64_t (&tot)[NV], int64_t (*wsum)[16])
{
    int64_t t[NV];
    #pragma unroll
    for (int q = 0; q < NV; ++q) t[q] = 0;
    #pragma unroll
    for (int k = 0; k < VPT; ++k)
        #pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int64_t x = v[k][q];
            v[k][q] = t[q];
            t[q] += x;
        }
    block_scan<int64_t, NV, NW>(t, tot, wsum);
    #pragma unroll
    for (int k = 0; k < VPT; ++k)
        #pragma unroll
        for (int q = 0; q < NV; ++q) v[k][q] += t[q];
}

// Per-digit scan of the tile counts (stored tile-major: each tile's 256
// counts are one contiguous row, written and read whole by the tile's own
// histogram and scatter workgroups): one wave per (segment, digit) turns the
// digit's column of tile counts into exclusive offsets within the digit and
// stores the digit's total; the scatter adds the digits' own offsets.  The
// column is read 64 tiles at a time, all chunks' loads issued first.
constexpr int kScanChunks = 16;   // rows up to 1024 tiles in registers; longer rows loop

__global__ __launch_bounds__(256) void k_sort_scan(int32_t* __restrict__ hist, int32_t* __restrict__ dtot,
                                                   SortSegs S)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);   // seg * 256 + digit
    const int seg = row >> 8, d = row & 255;
    const int ntiles = S.tile0[seg + 1] - S.tile0[seg];
    int32_t* h = hist + S.hoff[seg] + d;     // tile i's count at h[256 i]
    int32_t run = 0;
    for (int c0 = 0; c0 < ntiles; c0 += 64 * kScanChunks) {
        int32_t v[kScanChunks];
        #pragma unroll
        for (int q = 0; q < kScanChunks; ++q) {
            const int i = c0 + q * 64 + lane;
            v[q] = i < ntiles ? h[(int64_t)i * 256] : 0;
        }
        #pragma unroll
        for (int q = 0; q < kScanChunks; ++q) {
            const int i = c0 + q * 64 + lane;
            const int32_t incl = wave_incl_scan(v[q]);
            if (i < ntiles) h[(int64_t)i * 256] = run + incl - v[q];
            run += __shfl(incl, 63);
        }
    }
    if (lane == 0) dtot[row] = run;
}

// Stable scatter through LDS.  Wave v of the block owns the tile's keys
// v * 512 .. v * 512 + 511 (in order), taken 64 at a time: each key is
// ranked among the equal digits of its 64 with wave ballots, plus the count
// of that digit in the wave's earlier keys (a wave-private counter in LDS, so
// no block barrier per round).  One block step then turns the four waves'
// digit counts into the LDS start of each (wave, digit), after the digit's
// start in the tile (an exclusive scan of the tile's counts, which are the
// differences of consecutive tile offsets in the scanned histogram).  The
// finished tile is written out with consecutive threads on consecutive
// addresses of each digit's run.
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const uint64_t* __restrict__ kin,
                                                                const int32_t* __restrict__ vin,
                                                                uint64_t* __restrict__ kout,
                                                                int32_t* __restrict__ vout, SortSegs S,
                                                                int shift, const int32_t* __restrict__ hist,
                                                                const int32_t* __restrict__ dtot)
{
    __shared__ uint64_t skey[kSortTile];
    __shared__ int32_t sval[kSortTile];
    __shared__ int32_t gbase[256];     // global position of the tile's first key of each digit
    __shared__ int32_t lstart[256];    // LDS start of each digit's run
    __shared__ int32_t wcnt[kSortWaves][256];   // keys of each digit per wave (running, then final)
    __shared__ int32_t tsum[2][kSortWaves];
    int tile = blockIdx.x;
    int seg = tile_segment(S, tile);
    int lt = tile - S.tile0[seg];
    int ntiles = S.tile0[seg + 1] - S.tile0[seg];
    int start = S.off[seg] + lt * kSortTile;
    int end = S.off[seg + 1];
    int lane = threadIdx.x & 63;
    int wave = threadIdx.x >> 6;
    uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // the wave's keys and values, all loaded first (one memory round trip)
    const int wbase = start + wave * 64 * kSortWaveRounds;
    uint64_t kr[kSortWaveRounds];
    int32_t vr[kSortWaveRounds];
    #pragma unroll
    for (int r = 0; r < kSortWaveRounds; ++r) {
        const int i = wbase + r * 64 + lane;
        kr[r] = i < end ? kin[i] : 0ull;
        vr[r] = i < end ? vin[i] : 0;
    }
    {
        const int d = threadIdx.x;
        const int32_t* hd = hist + S.hoff[seg] + (int64_t)lt * 256 + d;
        const int32_t tot = dtot[seg * 256 + d];
        const int32_t mine = hd[0];
        const int32_t cnt = (lt + 1 < ntiles ? hd[256] : tot) - mine;
        // exclusive scans over the digits of the segment totals and of the
        // tile counts (256 threads = 4 waves)
        int32_t it = tot, ic = cnt;
        #pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            int32_t u = __shfl_up(it, o), v = __shfl_up(ic, o);
            if (lane >= o) { it += u; ic += v; }
        }
        if (lane == 63) { tsum[0][wave] = it; tsum[1][wave] = ic; }
        #pragma unroll
        for (int w2 = 0; w2 < kSortWaves; ++w2) wcnt[w2][d] = 0;
        __syncthreads();
        int32_t wt = 0, wc = 0;
        for (int w2 = 0; w2 < wave; ++w2) { wt += tsum[0][w2]; wc += tsum[1][w2]; }
        gbase[d] = S.off[seg] + wt + it - tot + mine;
        lstart[d] = wc + ic - cnt;
    }
    // ranks within the wave, in key order
    int32_t rk[kSortWaveRounds];
    int dg[kSortWaveRounds];
    int32_t* cw = wcnt[wave];
    #pragma unroll
    for (int r = 0; r < kSortWaveRounds; ++r) {
        const int i = wbase + r * 64 + lane;
        const bool valid = i < end;
        const int d = (int)((kr[r] >> shift) & 255);
        const uint64_t peers = digit_peers(d, valid);
        const int rank = __popcll(peers & lt_mask);
        const int32_t before = valid ? cw[d] : 0;
        wave_sync_lds();
        if (valid && rank == 0) cw[d] = before + __popcll(peers);
        wave_sync_lds();
        rk[r] = before + rank;
        dg[r] = valid ? d : -1;
    }
    __syncthreads();
    // LDS start of (wave, digit): the digit's start plus the earlier waves' counts
    {
        const int d = threadIdx.x;
        int32_t run = lstart[d];
        #pragma unroll
        for (int w2 = 0; w2 < kSortWaves; ++w2) {
            const int32_t c = wcnt[w2][d];
            wcnt[w2][d] = run;
            run += c;
        }
    }
    __syncthreads();
    #pragma unroll
    for (int r = 0; r < kSortWaveRounds; ++r) {
        if (dg[r] >= 0) {
            const int off = cw[dg[r]] + rk[r];
            skey[off] = kr[r];
            sval[off] = vr[r];
        }
    }
    __syncthreads();
    const int n_tile = (end - start) < kSortTile ? (end - start) : kSortTile;
    for (int q = threadIdx.x; q < n_tile; q += kSortThreads) {
        uint64_t k = skey[q];
        int d = (int)((k >> shift) & 255);
        int dst = gbase[d] + (q - lstart[d]);
        kout[dst] = k;
        vout[dst] = sval[q];
    }
}

// ---------------------------------------------------------------------------
// Sorts with fewer launches for short segments (same stable order as the LSD
// sort above, whose 25 launches dominate planning there):
// * both segments up to kSsCap keys: k_sort_small, one workgroup per segment
//   sorting it in LDS (bin_sort, or LSD on 8-bit digits over the bits that
//   vary where the keys crowd a few bins);
// * both up to 2^20 keys (kSsLargeMax): a splitter sort in five launches (64 bucket slots
//   per array up to 65536 keys, 1024 above) --
//   1. k_ss_sample (1024 slots: after k_ss_gather): one workgroup per segment sorts a stratified sample of the
//      keys in LDS (bin_sort; where that fails bitonic for 1024 keys, LSD
//      radix for 16384) and keeps its quantiles, without repeats, as the
//      splitters u_0 < ... < u_{U-1};
//   2. k_ss_count: each tile of kSsTile keys counts its keys per bucket (range
//      bucket 2p: the keys strictly between u_{p-1} and u_p; equality bucket
//      2p + 1: the keys equal to u_p, which never need sorting) and checks its
//      inputs;
//   3. k_ss_scan: per bucket, exclusive offsets over the tiles and the bucket
//      sizes;
//   4. k_ss_scatter: each tile scatters its keys, stably, into the buckets;
//   5. k_ss_local: one workgroup per bucket sorts it in LDS like k_sort_small;
//      a bucket beyond the LDS capacity (only when the sample misrepresents
//      the input) is sorted by the same workgroup through global memory.
// ---------------------------------------------------------------------------
constexpr int kSsBucketMean = 2048;      // target keys per range bucket
constexpr int kSsOversample = 32;        // sample keys per range bucket
constexpr int kSsThreads = 512;          // count and scatter workgroups: 8 waves
constexpr int kSsRounds = 16;            // 64-key rounds per wave
constexpr int kSsTile = kSsThreads * kSsRounds;
// LDS sort workgroups: 8 waves of 8 rounds (LDS holds two workgroups to a
// compute unit whatever their waves).
constexpr int kSsLocalThreads = 512;
constexpr int kSsLocalRounds = 8;
constexpr int kSsCap = kSsLocalThreads * kSsLocalRounds;   // longest run sorted in LDS

// The splitter sort with NB bucket slots per segment (2 U + 1 <= NB - 1
// used): 64 for segments up to 65536 keys, 1024 up to 2^20.
template <int NB>
struct SsCfg {
    static constexpr int kMaxSpl = NB / 2 - 1;                          // splitters per segment at most
    static constexpr int32_t kMaxLen = (kMaxSpl + 1) * kSsBucketMean;   // longest segment
    static constexpr int kSample = kSsOversample * (kMaxSpl + 1);       // sample keys per segment at most
    static constexpr int kBits = NB == 64 ? 6 : 10;                     // bits of a bucket id
    using Id = typename std::conditional<(NB <= 256), uint8_t, uint16_t>::type;
    // scratch layout in hist (int32 units): the splitters (2 x kMaxSpl
    // uint64), their counts, the bucket starts and sizes (2 x NB each), then
    // the tile-major bucket counts
    static constexpr int kNsplOff = (4 * kMaxSpl + 63) / 64 * 64;
    static constexpr int kStartOff = kNsplOff + 64;
    static constexpr int kTotOff = kStartOff + 2 * NB;
    static constexpr int kCntOff = kTotOff + 2 * NB;
};
static_assert(SsCfg<64>::kMaxLen == 65536 && SsCfg<64>::kSample == 1024, "small splitter sort");
static_assert(SsCfg<1024>::kMaxLen == (1 << 20) && SsCfg<1024>::kSample == 16384, "large splitter sort");

// Sort key of an input (see k_make_keys); ok is false for a negative, NaN or
// infinite value, whose key is 0.
__device__ __forceinline__ uint64_t sort_key(double v, bool& ok)
{
    ok = (v >= 0.0) && (v <= 1.7976931348623157e308);
    return (v == 0.0 || !ok) ? 0ull : (uint64_t)__double_as_longlong(v);
}

// Bucket of key k among the U sorted splitters su: 2p + (k == u_p), p the
// number of splitters below k.
template <int NB>
__device__ __forceinline__ int ss_bucket(const uint64_t* su, int U, uint64_t k)
{
    int p = 0;
    #pragma unroll
    for (int step = (SsCfg<NB>::kMaxSpl + 1) / 2; step > 0; step >>= 1)
        if (p + step <= U && su[p + step - 1] < k) p += step;
    return 2 * p + ((p < U && su[p] == k) ? 1 : 0);
}

// Lanes of the wave whose bucket b (BITS bits) equals the calling lane's,
// among the lanes with `valid` set.
template <int BITS>
__device__ __forceinline__ uint64_t bucket_peers(int b, bool valid)
{
    uint64_t peers = __ballot(valid);
    #pragma unroll
    for (int i = 0; i < BITS; ++i) {
        uint64_t m = __ballot((b >> i) & 1);
        peers &= ((b >> i) & 1) ? m : ~m;
    }
    return peers;
}

// Position of sample s of ns in a segment of n keys: one point drawn from each
// of ns equal strata (a fixed hash of s picks it), so that no period of the
// input lines up with the sample.
__device__ __forceinline__ int64_t ss_sample_pos(int s, int ns, int64_t n)
{
    uint32_t h = (uint32_t)s * 0x9E3779B9u;
    h ^= h >> 16; h *= 0x85EBCA6Bu; h ^= h >> 13; h *= 0xC2B2AE35u; h ^= h >> 16;
    // floor(s n / ns) in double, exactly: s n < 2^53, and a quotient that is
    // no integer is at least 1/ns away from one (a 64-bit integer division
    // takes ten times as long)
    const double dn = (double)n, dns = (double)ns;
    const int64_t lo = (int64_t)floor((double)s * dn / dns), hi = (int64_t)floor((double)(s + 1) * dn / dns);
    return lo + (int64_t)(((uint64_t)h * (uint64_t)(hi - lo)) >> 32);
}

// Stable ranks of the 8-bit digits (key >> shift) of a workgroup's keys, held
// R per lane in (wave, round, lane) order with `rounds` rounds per wave, n_valid of them: rk[q] receives the key's offset among the equal
// digits before it in its wave, wcnt[v][d] (zeroed by the caller) the count
// of digit d in wave v's keys.
template <int R>
__device__ __forceinline__ void ss_rank_digits(const uint64_t (&kr)[R], int shift, int rounds, int n_valid,
                                               int32_t (*wcnt)[256], int (&dg)[R], int (&rk)[R])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int32_t* cw = wcnt[wave];
    #pragma unroll
    for (int q = 0; q < R; ++q) {
        dg[q] = -1;
        if (q < rounds) {
            const int i = (wave * rounds + q) * 64 + lane;
            const bool valid = i < n_valid;
            const int d = (int)((kr[q] >> shift) & 255);
            const uint64_t peers = digit_peers(d, valid);
            const int rank = __popcll(peers & lt_mask);
            const int32_t before = valid ? cw[d] : 0;
            wave_sync_lds();
            if (valid && rank == 0) cw[d] = before + __popcll(peers);
            wave_sync_lds();
            rk[q] = before + rank;
            dg[q] = valid ? d : -1;
        }
    }
}

// Thread d < 256: the waves' starts of digit d in wcnt (counts in, starts
// out), after the digit's start among all the keys plus base.  Returns the
// digit's total (0 in the other threads).
__device__ __forceinline__ int32_t ss_digit_starts(int32_t (*wcnt)[256], int32_t base, int32_t* wtot)
{
    constexpr int kWaves = kSsLocalThreads / 64;
    const int d = threadIdx.x, lane = d & 63, wave = d >> 6;
    int32_t c = 0;
    if (d < 256)
        for (int v = 0; v < kWaves; ++v) c += wcnt[v][d];
    const int32_t incl = wave_incl_scan(c);
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    if (d < 256) {
        int32_t run = base + incl - c;
        for (int v = 0; v < wave; ++v) run += wtot[v];
        #pragma unroll
        for (int v = 0; v < kWaves; ++v) {
            const int32_t a = wcnt[v][d];
            wcnt[v][d] = run;
            run += a;
        }
    }
    return c;
}

// Smallest and largest of the valid keys kr[q] over the block.
__device__ __forceinline__ void ss_key_range(const uint64_t (&kr)[kSsLocalRounds], int rounds, int n_valid,
                                             uint64_t* red, uint64_t& kmin, uint64_t& kmax)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t lo = ~0ull, hi = 0ull;
    #pragma unroll
    for (int q = 0; q < kSsLocalRounds; ++q) {
        const int i = (wave * rounds + q) * 64 + lane;
        if (q < rounds && i < n_valid) { lo = kr[q] < lo ? kr[q] : lo; hi = kr[q] > hi ? kr[q] : hi; }
    }
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    if (lane == 0) { red[2 * wave] = lo; red[2 * wave + 1] = hi; }
    __syncthreads();
    kmin = ~0ull; kmax = 0ull;
    #pragma unroll
    for (int v = 0; v < kSsLocalThreads / 64; ++v) {
        kmin = red[2 * v] < kmin ? red[2 * v] : kmin;
        kmax = red[2 * v + 1] > kmax ? red[2 * v + 1] : kmax;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Sort of a workgroup's keys by bins: a key's place among kBins equal bins
// between the smallest and the largest key is nearly its rank where the keys
// are spread evenly, and the few keys that share a bin are compared with each
// other.  Keys go to the bins in any order (LDS counters); the comparison by
// (key, value) then makes the order the stable one.  One pass over LDS where
// a radix sort needs one per eight bits of the keys (up to eight).
//
// Bins divide the values (uniform, clustered at the ends) or, where a quarter
// or more of the keys lie in the lowest sixteenth of the range (points over
// several decades), the bit patterns, which grow like the logarithm.  Both are
// nondecreasing in the key.
// ---------------------------------------------------------------------------
constexpr int kBins = 4096;
// Fullest bin sorted by comparisons; fuller ones (clusters, many repeats)
// leave the keys to the radix sorts.
constexpr int32_t kBinMax = 96;

struct BinMap {
    uint64_t kmin;
    double vmin, scale;
    bool by_value;
};

__device__ __forceinline__ int bin_of(const BinMap& B, uint64_t k)
{
    const double d = B.by_value ? __longlong_as_double((long long)k) - B.vmin : (double)(k - B.kmin);
    const double t = d * B.scale;
    return t < kBins - 1 ? (int)t : kBins - 1;
}

// LDS words of bin_sort besides keys, values and bins.
template <int WAVES>
struct BinLds {
    uint64_t red[2 * WAVES];
    int32_t wtot[WAVES], wmax[WAVES];
    int32_t low;
};

// Sorts the block's n >= 1 keys kr[q] (with their values vr[q]; key i =
// (wave rounds + q) 64 + lane for q < rounds, i < n) and hands each to
// emit(rank, key, value).  key, val (n entries) and bin (kBins): LDS.  False,
// with nothing emitted, if a bin is too full.  val may be null: equal keys
// then rank in any order.
template <int WAVES, int R, class Emit>
__device__ bool bin_sort(const uint64_t (&kr)[R], const int32_t (&vr)[R], int rounds, int n, uint64_t* key,
                         int32_t* val, int32_t* bin, BinLds<WAVES>& L, Emit emit)
{
    constexpr int kThreads = 64 * WAVES, kPer = kBins / kThreads;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    auto valid = [&](int q) { return q < rounds && (wave * rounds + q) * 64 + lane < n; };
    uint64_t lo = ~0ull, hi = 0ull;
    #pragma unroll
    for (int q = 0; q < R; ++q)
        if (valid(q)) { lo = kr[q] < lo ? kr[q] : lo; hi = kr[q] > hi ? kr[q] : hi; }
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    if (lane == 0) { L.red[2 * wave] = lo; L.red[2 * wave + 1] = hi; }
    if (t == 0) L.low = 0;
    for (int i = t; i < kBins; i += kThreads) bin[i] = 0;
    __syncthreads();
    for (int v = 0; v < WAVES; ++v) {
        lo = L.red[2 * v] < lo ? L.red[2 * v] : lo;
        hi = L.red[2 * v + 1] > hi ? L.red[2 * v + 1] : hi;
    }
    BinMap B;
    B.kmin = lo;
    B.vmin = __longlong_as_double((long long)lo);
    const double vrange = __longlong_as_double((long long)hi) - B.vmin;
    const double cut = B.vmin + 0.0625 * vrange;
    int low = 0;
    #pragma unroll
    for (int q = 0; q < R; ++q)
        low += __popcll(__ballot(valid(q) && __longlong_as_double((long long)kr[q]) < cut));
    if (lane == 0) atomicAdd(&L.low, low);
    __syncthreads();
    const double vscale = kBins / vrange;
    B.by_value = 4 * L.low < n && vscale <= 1.7976931348623157e308;
    B.scale = B.by_value ? vscale : hi > lo ? kBins / (double)(hi - lo) : 0.0;
    int place[R];
    #pragma unroll
    for (int q = 0; q < R; ++q)
        if (valid(q)) place[q] = atomicAdd(&bin[bin_of(B, kr[q])], 1);
    __syncthreads();
    // the bins' starts (thread t: bins kPer t ..)
    {
        int32_t c[kPer], sum = 0, most = 0;
        #pragma unroll
        for (int j = 0; j < kPer; ++j) {
            c[j] = bin[kPer * t + j];
            sum += c[j];
            most = c[j] > most ? c[j] : most;
        }
        const int32_t incl = wave_incl_scan(sum);
        #pragma unroll
        for (int o = 32; o > 0; o >>= 1) { const int32_t u = __shfl_xor(most, o); most = u > most ? u : most; }
        if (lane == 63) { L.wtot[wave] = incl; L.wmax[wave] = most; }
        __syncthreads();
        int32_t run = incl - sum;
        for (int v = 0; v < WAVES; ++v) {
            if (v < wave) run += L.wtot[v];
            most = L.wmax[v] > most ? L.wmax[v] : most;
        }
        if (most > kBinMax) return false;          // the same in every thread
        #pragma unroll
        for (int j = 0; j < kPer; ++j) { bin[kPer * t + j] = run; run += c[j]; }
    }
    __syncthreads();
    #pragma unroll
    for (int q = 0; q < R; ++q)
        if (valid(q)) {
            const int at = bin[bin_of(B, kr[q])] + place[q];
            key[at] = kr[q];
            if (val) val[at] = vr[q];
        }
    __syncthreads();
    for (int i = t; i < n; i += kThreads) {
        const uint64_t k = key[i];
        const int32_t v = val ? val[i] : i;
        const int b = bin_of(B, k);
        const int first = bin[b], last = b + 1 < kBins ? bin[b + 1] : n;
        int rank = first;
        for (int j = first; j < last; ++j) {
            const uint64_t o = key[j];
            rank += o < k ? 1 : 0;
            if (o == k) rank += (val ? val[j] : j) < v ? 1 : 0;
        }
        emit(rank, k, v);
    }
    return true;
}

// LDS of a block sort of up to kSsCap keys.
struct SsBlockLds {
    uint64_t key[kSsCap];
    int32_t val[kSsCap];
    union {
        int32_t bin[kBins];
        int32_t wcnt[kSsLocalThreads / 64][256];
    };
    BinLds<kSsLocalThreads / 64> bl;
    int32_t wtot[kSsLocalThreads / 64];
    uint64_t red[2 * (kSsLocalThreads / 64)];
};

// Rounds per wave for n keys over the block's waves (wave-major order:
// key i sits in wave i / (64 rounds), round (i / 64) % rounds, lane i % 64).
__device__ __forceinline__ int ss_rounds(int n) { return (n + kSsLocalThreads - 1) / kSsLocalThreads; }

// Stable sort of the block's n <= kSsCap keys (with their values) held in
// registers as ss_rounds(n) rounds per wave: LSD passes of 8 bits over the
// bits in which the keys differ, each ranking the keys in registers and
// exchanging them through LDS.
__device__ void ss_block_sort(uint64_t (&kr)[kSsLocalRounds], int32_t (&vr)[kSsLocalRounds], int n, SsBlockLds& L)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rounds = ss_rounds(n);
    int dg[kSsLocalRounds], rk[kSsLocalRounds];
    uint64_t kmin, kmax;
    ss_key_range(kr, rounds, n, L.red, kmin, kmax);
    const uint64_t diff = kmin ^ kmax;
    const int passes = diff ? (64 - __clzll((long long)diff) + 7) / 8 : 0;
    for (int p = 0; p < passes; ++p) {
        for (int i = threadIdx.x; i < kSsLocalThreads / 64 * 256; i += kSsLocalThreads) (&L.wcnt[0][0])[i] = 0;
        __syncthreads();
        ss_rank_digits(kr, 8 * p, rounds, n, L.wcnt, dg, rk);
        __syncthreads();
        ss_digit_starts(L.wcnt, 0, L.wtot);
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < kSsLocalRounds; ++q) {
            if (dg[q] >= 0) {
                const int off = L.wcnt[wave][dg[q]] + rk[q];
                L.key[off] = kr[q];
                L.val[off] = vr[q];
            }
        }
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < kSsLocalRounds; ++q) {
            const int i = (wave * rounds + q) * 64 + lane;
            if (q < rounds && i < n) { kr[q] = L.key[i]; vr[q] = L.val[i]; }
        }
    }
}

// Both segments at most kSsCap keys: one workgroup per segment makes the keys
// and values, sorts them in LDS into (k0, v0), and sets errs[segment] (1 if
// the segment holds a negative, NaN or infinite input).
__global__ __launch_bounds__(kSsLocalThreads) void k_sort_small(const double* __restrict__ r,
                                                                const double* __restrict__ w, SortSegs S,
                                                                uint64_t* __restrict__ k0, int32_t* __restrict__ v0,
                                                                int32_t* __restrict__ errs)
{
    __shared__ SsBlockLds L;
    const int seg = blockIdx.x;
    const int base = S.off[seg];
    const int n = S.off[seg + 1] - base;
    const double* __restrict__ x = seg ? w : r;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rounds = ss_rounds(n);
    uint64_t kr[kSsLocalRounds];
    int32_t vr[kSsLocalRounds];
    bool bad = false;
    #pragma unroll
    for (int q = 0; q < kSsLocalRounds; ++q) {
        const int i = (wave * rounds + q) * 64 + lane;
        kr[q] = 0ull; vr[q] = 0;
        if (q < rounds && i < n) {
            bool ok;
            kr[q] = sort_key(x[i], ok);
            bad |= !ok;
            vr[q] = i;
        }
    }
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    if (threadIdx.x == 0) errs[seg] = any_bad ? 1 : 0;
    if (n == 0) return;
    if (bin_sort<kSsLocalThreads / 64>(kr, vr, rounds, n, L.key, L.val, L.bin, L.bl,
                                       [&](int i, uint64_t k, int32_t v) { k0[base + i] = k; v0[base + i] = v; }))
        return;
    __syncthreads();
    ss_block_sort(kr, vr, n, L);
    #pragma unroll
    for (int q = 0; q < kSsLocalRounds; ++q) {
        const int i = (wave * rounds + q) * 64 + lane;
        if (q < rounds && i < n) { k0[base + i] = kr[q]; v0[base + i] = vr[q]; }
    }
}

// The B - 1 quantiles sk[step], sk[2 step], .. of the sorted sample, each kept
// if it differs from the one before, as the segment's splitters (threads
// t < B - 1 of a 1024-thread block; every thread calls it).
__device__ __forceinline__ void ss_pick_splitters(const uint64_t* sk, int step, int B, uint64_t* spl_seg,
                                                  int32_t* nspl_seg, int32_t* wtot)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint64_t c = 0;
    bool keep = false;
    if (t < B - 1) {
        c = sk[(t + 1) * step];
        keep = t == 0 || c != sk[t * step];
    }
    const uint64_t kb = __ballot(keep);
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (lane == 0) wtot[wave] = __popcll(kb);
    __syncthreads();
    int pos = __popcll(kb & lt_mask);
    for (int v = 0; v < wave; ++v) pos += wtot[v];
    if (keep) spl_seg[pos] = c;
    if (t == 0) {
        int tot = 0;
        for (int v = 0; v < 1024 / 64; ++v) tot += wtot[v];
        *nspl_seg = tot;
    }
}

// The sample's keys of NB = 1024 into samp, from the segment's offset on: a
// thread a key, so that the loads, a cache line each, come from many compute
// units (16384 of them by the one workgroup that sorts them: 30 us).
__global__ __launch_bounds__(256) void k_ss_gather(const double* __restrict__ r, const double* __restrict__ w,
                                                   SortSegs S, uint64_t* __restrict__ samp)
{
    const int seg = blockIdx.y;
    const int64_t n = S.off[seg + 1] - S.off[seg];
    const int ns = kSsOversample * (int)((n + kSsBucketMean - 1) / kSsBucketMean);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (n <= kSsBucketMean || i >= ns) return;
    bool ok;
    samp[S.off[seg] + i] = sort_key((seg ? w : r)[ss_sample_pos(i, ns, n)], ok);
}

// One workgroup of 1024 threads per segment: a stratified sample of the keys
// sorted in LDS (by bins; where those are too full, bitonic for the 1024-key
// samples of NB = 64 and LSD on 8-bit digits over the bits that vary, 16 waves
// of up to 16 rounds, for the 16384-key samples of NB = 1024), then its
// quantiles as splitters.
template <int NB>
__global__ __launch_bounds__(1024) void k_ss_sample(const double* __restrict__ r, const double* __restrict__ w,
                                                    const uint64_t* __restrict__ samp, SortSegs S,
                                                    uint64_t* __restrict__ spl,
                                                    int32_t* __restrict__ nspl)
{
    using C = SsCfg<NB>;
    constexpr int kRounds = (C::kSample + 1023) / 1024;
    __shared__ uint64_t sk[C::kSample];
    __shared__ uint64_t quant[C::kMaxSpl + 1];
    __shared__ int32_t bin[kBins];             // also the radix sort's digit counts
    __shared__ BinLds<16> bl;
    int32_t* const wtot = bl.wtot;
    const int seg = blockIdx.x;
    const int64_t n = S.off[seg + 1] - S.off[seg];
    const double* __restrict__ x = seg ? w : r;
    const int B = (int)((n + kSsBucketMean - 1) / kSsBucketMean);   // range buckets wanted
    if (B <= 1) {
        if (threadIdx.x == 0) nspl[seg] = 0;
        return;
    }
    const int ns = kSsOversample * B;          // below n: a bucket has kSsBucketMean keys
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int rounds = (ns + 1024 - 1) / 1024;
    uint64_t kr[kRounds];
    int32_t none[kRounds];
    #pragma unroll
    for (int q = 0; q < kRounds; ++q) {
        const int i = (wave * rounds + q) * 64 + lane;
        kr[q] = 0ull;
        none[q] = 0;
        if (q < rounds && i < ns) {
            if constexpr (NB == 64) {
                bool ok;
                kr[q] = sort_key(x[ss_sample_pos(i, ns, n)], ok);
            } else {
                kr[q] = samp[S.off[seg] + i];
            }
        }
    }
    if (bin_sort<16>(kr, none, rounds, ns, sk, (int32_t*)nullptr, bin, bl, [&](int i, uint64_t k, int32_t) {
            if (i % kSsOversample == 0) quant[i / kSsOversample] = k;
        })) {
        __syncthreads();
        ss_pick_splitters(quant, 1, B, spl + seg * C::kMaxSpl, nspl + seg, wtot);
        return;
    }
    __syncthreads();
    if constexpr (NB == 64) {
        int np2 = 1;
        while (np2 < ns) np2 <<= 1;
        sk[t] = t < ns ? kr[0] : ~0ull;        // one round: lane and wave in order
        __syncthreads();
        for (int k = 2; k <= np2; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                const int l = t ^ j;
                if (t < np2 && l > t) {
                    const uint64_t a = sk[t], b = sk[l];
                    if ((a > b) == ((t & k) == 0)) { sk[t] = b; sk[l] = a; }
                }
                __syncthreads();
            }
    } else {
        int32_t (*wcnt)[256] = reinterpret_cast<int32_t (*)[256]>(bin);
        static_assert(kBins == 16 * 256, "digit counts of 16 waves");
        #pragma unroll
        for (int q = 0; q < kSsRounds; ++q) {
            const int i = (wave * rounds + q) * 64 + lane;
            if (q < rounds && i < ns) sk[i] = kr[q];
        }
        // the bits in which the sample's keys differ
        uint64_t kmin = ~0ull, kmax = 0ull;
        for (int v = 0; v < 16; ++v) {
            kmin = bl.red[2 * v] < kmin ? bl.red[2 * v] : kmin;
            kmax = bl.red[2 * v + 1] > kmax ? bl.red[2 * v + 1] : kmax;
        }
        const uint64_t diff = kmin ^ kmax;
        const int passes = diff ? (64 - __clzll((long long)diff) + 7) / 8 : 0;
        int dg[kSsRounds], rk[kSsRounds];
        for (int p = 0; p < passes; ++p) {
            for (int i = t; i < 16 * 256; i += 1024) (&wcnt[0][0])[i] = 0;
            __syncthreads();
            ss_rank_digits(kr, 8 * p, rounds, ns, wcnt, dg, rk);
            __syncthreads();
            // thread d < 256: the digit's start, then the waves' starts
            int32_t c = 0, incl = 0;
            if (t < 256) {
                for (int v = 0; v < 16; ++v) c += wcnt[v][t];
                incl = wave_incl_scan(c);
                if (lane == 63) wtot[wave] = incl;
            }
            __syncthreads();
            if (t < 256) {
                int32_t run = incl - c;
                for (int v = 0; v < wave; ++v) run += wtot[v];
                for (int v = 0; v < 16; ++v) {
                    const int32_t a = wcnt[v][t];
                    wcnt[v][t] = run;
                    run += a;
                }
            }
            __syncthreads();
            #pragma unroll
            for (int q = 0; q < kSsRounds; ++q)
                if (dg[q] >= 0) sk[wcnt[wave][dg[q]] + rk[q]] = kr[q];
            __syncthreads();
            #pragma unroll
            for (int q = 0; q < kSsRounds; ++q) {
                const int i = (wave * rounds + q) * 64 + lane;
                if (q < rounds && i < ns) kr[q] = sk[i];
            }
        }
        __syncthreads();
    }
    ss_pick_splitters(sk, kSsOversample, B, spl + seg * C::kMaxSpl, nspl + seg, wtot);
}

// Per tile: the bucket counts (tile-major, NB per tile) and errs[tile] (1 if
// the tile holds a negative, NaN or infinite input).
template <int NB>
__global__ __launch_bounds__(kSsThreads) void k_ss_count(const double* __restrict__ r,
                                                         const double* __restrict__ w, SortSegs S,
                                                         const uint64_t* __restrict__ spl,
                                                         const int32_t* __restrict__ nspl,
                                                         int32_t* __restrict__ cnt, int32_t* __restrict__ errs)
{
    using C = SsCfg<NB>;
    __shared__ uint64_t su[C::kMaxSpl];
    __shared__ int32_t h[NB];
    const int tile = blockIdx.x;
    const int seg = tile_segment(S, tile);
    const int lt = tile - S.tile0[seg];
    const int base = S.off[seg], end = S.off[seg + 1];
    const int U = nspl[seg];
    const double* __restrict__ x = seg ? w : r;
    for (int i = threadIdx.x; i < U; i += kSsThreads) su[i] = spl[seg * C::kMaxSpl + i];
    for (int i = threadIdx.x; i < NB; i += kSsThreads) h[i] = 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wbase = base + lt * kSsTile + wave * 64 * kSsRounds;
    double v[kSsRounds];
    #pragma unroll
    for (int q = 0; q < kSsRounds; ++q) {
        const int i = wbase + q * 64 + lane;
        v[q] = i < end ? x[i - base] : 0.0;
    }
    __syncthreads();
    bool bad = false;
    #pragma unroll
    for (int q = 0; q < kSsRounds; ++q) {
        const int i = wbase + q * 64 + lane;
        int b = -1;
        if (i < end) {
            bool ok;
            const uint64_t k = sort_key(v[q], ok);
            bad |= !ok;
            b = ss_bucket<NB>(su, U, k);
        }
        // a bucket shared by the whole round (sorted or clustered input) costs one add
        const int b0 = __shfl(b, 0);
        const uint64_t valid = __ballot(b >= 0);
        const uint64_t same = __ballot(b >= 0 && b == b0);
        if (b0 >= 0 && same == valid) {
            if (lane == 0) atomicAdd(&h[b0], (int32_t)__popcll(valid));
        } else if (b >= 0) {
            atomicAdd(&h[b], 1);
        }
    }
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    for (int i = threadIdx.x; i < NB; i += kSsThreads) cnt[(int64_t)tile * NB + i] = h[i];
    if (threadIdx.x == 0) errs[tile] = any_bad ? 1 : 0;
}

// A workgroup takes 64 buckets of one segment: their counts over the segment's
// tiles become exclusive offsets, and btot receives the bucket sizes.  Its
// waves split the tiles, all of a wave's loads in flight at once (a bucket's
// counts one after the other are a chain of latencies: 17 us at 123 tiles).
constexpr int kSsScanWaves = 8;

template <int NB>
__global__ __launch_bounds__(64 * kSsScanWaves) void k_ss_scan(SortSegs S, int32_t* __restrict__ cnt,
                                                               int32_t* __restrict__ btot)
{
    constexpr int kTiles = (SsCfg<NB>::kMaxLen + kSsTile - 1) / kSsTile;    // of a segment, at most
    constexpr int kPer = (kTiles + kSsScanWaves - 1) / kSsScanWaves;
    __shared__ int32_t part[kSsScanWaves][64];
    const int seg = blockIdx.x / (NB / 64), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = (blockIdx.x % (NB / 64)) * 64 + lane;
    const int nt = S.tile0[seg + 1] - S.tile0[seg];
    int32_t* c = cnt + (int64_t)S.tile0[seg] * NB + b;
    int32_t v[kPer], sum = 0;
    #pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int t = wave * kPer + q;
        v[q] = t < nt ? c[(int64_t)t * NB] : 0;
    }
    #pragma unroll
    for (int q = 0; q < kPer; ++q) sum += v[q];
    part[wave][lane] = sum;
    __syncthreads();
    int32_t run = 0;
    for (int u = 0; u < wave; ++u) run += part[u][lane];
    #pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int t = wave * kPer + q;
        if (t < nt) c[(int64_t)t * NB] = run;
        run += v[q];
    }
    if (wave == kSsScanWaves - 1) btot[seg * NB + b] = run;
}

// Stable scatter of a tile into the buckets, through LDS: wave v owns the
// tile's keys v * 1024 .. v * 1024 + 1023 (in order), ranked 64 at a time
// among the equal buckets of their round plus the wave's earlier keys of that
// bucket; one block step turns the waves' counts into LDS starts; the staged
// tile is written out with consecutive threads on consecutive addresses of
// each bucket's run.  Every tile adds up the buckets' starts from their sizes;
// a segment's first tile stores them.
template <int NB>
__global__ __launch_bounds__(kSsThreads) void k_ss_scatter(const double* __restrict__ r,
                                                           const double* __restrict__ w, SortSegs S,
                                                           const uint64_t* __restrict__ spl,
                                                           const int32_t* __restrict__ nspl,
                                                           const int32_t* __restrict__ cnt,
                                                           const int32_t* __restrict__ btot,
                                                           int32_t* __restrict__ bstart,
                                                           uint64_t* __restrict__ kout, int32_t* __restrict__ vout)
{
    using C = SsCfg<NB>;
    using Id = typename C::Id;
    constexpr int kWaves = kSsThreads / 64;
    __shared__ uint64_t skey[kSsTile];
    __shared__ int32_t sval[kSsTile];
    __shared__ Id sbk[kSsTile];
    __shared__ uint64_t su[C::kMaxSpl];
    __shared__ int32_t wcnt[kWaves][NB];
    __shared__ int32_t gbase[NB];
    __shared__ int32_t lstart[NB];
    __shared__ int32_t wtot[kWaves], btsum[kWaves];
    const int tile = blockIdx.x;
    const int seg = tile_segment(S, tile);
    const int lt = tile - S.tile0[seg];
    const int base = S.off[seg], end = S.off[seg + 1];
    const int start = base + lt * kSsTile;
    const int U = nspl[seg];
    const double* __restrict__ x = seg ? w : r;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int wbase = start + wave * 64 * kSsRounds;
    uint64_t kr[kSsRounds];
    #pragma unroll
    for (int q = 0; q < kSsRounds; ++q) {
        const int i = wbase + q * 64 + lane;
        bool ok;
        kr[q] = i < end ? sort_key(x[i - base], ok) : 0ull;
    }
    for (int i = threadIdx.x; i < U; i += kSsThreads) su[i] = spl[seg * C::kMaxSpl + i];
    for (int i = threadIdx.x; i < kWaves * NB; i += kSsThreads) (&wcnt[0][0])[i] = 0;
    __syncthreads();
    int bk[kSsRounds], rk[kSsRounds];
    int32_t* cw = wcnt[wave];
    #pragma unroll
    for (int q = 0; q < kSsRounds; ++q) {
        const int i = wbase + q * 64 + lane;
        const bool valid = i < end;
        const int b = valid ? ss_bucket<NB>(su, U, kr[q]) : 0;
        const uint64_t peers = bucket_peers<C::kBits>(b, valid);
        const int rank = __popcll(peers & lt_mask);
        const int32_t before = valid ? cw[b] : 0;
        wave_sync_lds();
        if (valid && rank == 0) cw[b] = before + __popcll(peers);
        wave_sync_lds();
        rk[q] = before + rank;
        bk[q] = valid ? b : -1;
    }
    __syncthreads();
    // per bucket: the tile's count, its LDS start (exclusive scan over the
    // buckets), the waves' starts and the global base
    if constexpr (NB == 64) {
        if (wave == 0) {
            const int b = lane;
            int32_t c = 0;
            #pragma unroll
            for (int v = 0; v < kWaves; ++v) c += wcnt[v][b];
            const int32_t ls = wave_incl_scan(c) - c;
            lstart[b] = ls;
            int32_t run = ls;
            #pragma unroll
            for (int v = 0; v < kWaves; ++v) {
                const int32_t a = wcnt[v][b];
                wcnt[v][b] = run;
                run += a;
            }
            const int32_t size = btot[seg * NB + b], at = wave_incl_scan(size) - size;
            if (lt == 0) bstart[seg * NB + b] = at;
            gbase[b] = base + at + cnt[(int64_t)tile * NB + b];
        }
    } else {
        // thread t: buckets BPT t .. BPT t + BPT - 1
        constexpr int BPT = NB / kSsThreads;
        const int b0 = BPT * threadIdx.x;
        int32_t c[BPT], size[BPT], sum = 0, bsum = 0;
        #pragma unroll
        for (int j = 0; j < BPT; ++j) {
            c[j] = 0;
            #pragma unroll
            for (int v = 0; v < kWaves; ++v) c[j] += wcnt[v][b0 + j];
            sum += c[j];
            size[j] = btot[seg * NB + b0 + j];
            bsum += size[j];
        }
        const int32_t incl = wave_incl_scan(sum), bincl = wave_incl_scan(bsum);
        if (lane == 63) { wtot[wave] = incl; btsum[wave] = bincl; }
        __syncthreads();
        int32_t ex = incl - sum, at = bincl - bsum;
        for (int v = 0; v < wave; ++v) { ex += wtot[v]; at += btsum[v]; }
        #pragma unroll
        for (int j = 0; j < BPT; ++j) {
            const int b = b0 + j;
            lstart[b] = ex;
            int32_t run = ex;
            #pragma unroll
            for (int v = 0; v < kWaves; ++v) {
                const int32_t a = wcnt[v][b];
                wcnt[v][b] = run;
                run += a;
            }
            if (lt == 0) bstart[seg * NB + b] = at;
            gbase[b] = base + at + cnt[(int64_t)tile * NB + b];
            at += size[j];
            ex += c[j];
        }
    }
    __syncthreads();
    #pragma unroll
    for (int q = 0; q < kSsRounds; ++q) {
        if (bk[q] >= 0) {
            const int off = cw[bk[q]] + rk[q];
            skey[off] = kr[q];
            sval[off] = wbase + q * 64 + lane - base;
            sbk[off] = (Id)bk[q];
        }
    }
    __syncthreads();
    const int n_tile = (end - start) < kSsTile ? (end - start) : kSsTile;
    for (int q = threadIdx.x; q < n_tile; q += kSsThreads) {
        const int b = sbk[q];
        const int dst = gbase[b] + (q - lstart[b]);
        kout[dst] = skey[q];
        vout[dst] = sval[q];
    }
}

__device__ __forceinline__ uint64_t load_coherent(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t load_coherent(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One workgroup per (segment, bucket slot): the bucketed keys (kin, vin) of
// the bucket, sorted stably, into (kout, vout) at the same offsets.
template <int NB>
__global__ __launch_bounds__(kSsLocalThreads) void k_ss_local(SortSegs S, const int32_t* __restrict__ nspl,
                                                              const int32_t* __restrict__ bstart,
                                                              const int32_t* __restrict__ btot,
                                                              uint64_t* __restrict__ kin, int32_t* __restrict__ vin,
                                                              uint64_t* __restrict__ kout,
                                                              int32_t* __restrict__ vout)
{
    constexpr int kWaves = kSsLocalThreads / 64;
    __shared__ SsBlockLds L;
    __shared__ int32_t gb[256];
    const int seg = blockIdx.x / NB, b = blockIdx.x % NB;
    if (b > 2 * nspl[seg]) return;
    const int32_t size = btot[seg * NB + b];
    if (size == 0) return;
    const int64_t start = S.off[seg] + bstart[seg * NB + b];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((b & 1) || size == 1) {   // equal keys: already in order
        for (int32_t i = threadIdx.x; i < size; i += kSsLocalThreads) {
            kout[start + i] = kin[start + i];
            vout[start + i] = vin[start + i];
        }
        return;
    }
    uint64_t kr[kSsLocalRounds];
    int32_t vr[kSsLocalRounds];
    if (size <= kSsCap) {
        const int rounds = ss_rounds(size);
        #pragma unroll
        for (int q = 0; q < kSsLocalRounds; ++q) {
            const int i = (wave * rounds + q) * 64 + lane;
            const bool in = q < rounds && i < size;
            kr[q] = in ? kin[start + i] : 0ull;
            vr[q] = in ? vin[start + i] : 0;
        }
        if (bin_sort<kWaves>(kr, vr, rounds, size, L.key, L.val, L.bin, L.bl,
                             [&](int i, uint64_t k, int32_t v) { kout[start + i] = k; vout[start + i] = v; }))
            return;
        __syncthreads();
        ss_block_sort(kr, vr, size, L);
        #pragma unroll
        for (int q = 0; q < kSsLocalRounds; ++q) {
            const int i = (wave * rounds + q) * 64 + lane;
            if (q < rounds && i < size) { kout[start + i] = kr[q]; vout[start + i] = vr[q]; }
        }
        return;
    }
    // A bucket beyond the LDS: LSD passes through global memory, chunk by
    // chunk (kSsCap keys, kSsLocalRounds rounds per wave) in order, between
    // (kin, vin) and (kout, vout); a chunk's keys are written straight to
    // their places.  Data written by an earlier pass is read with
    // cache-coherent loads.
    int dg[kSsLocalRounds], rk[kSsLocalRounds];
    uint64_t kmin = ~0ull, kmax = 0ull;
    for (int32_t c0 = 0; c0 < size; c0 += kSsCap) {
        const int nv = size - c0 < kSsCap ? size - c0 : kSsCap;
        #pragma unroll
        for (int q = 0; q < kSsLocalRounds; ++q) {
            const int i = (wave * kSsLocalRounds + q) * 64 + lane;
            kr[q] = i < nv ? kin[start + c0 + i] : 0ull;
        }
        uint64_t lo, hi;
        ss_key_range(kr, kSsLocalRounds, nv, L.red, lo, hi);
        kmin = lo < kmin ? lo : kmin;
        kmax = hi > kmax ? hi : kmax;
    }
    const uint64_t diff = kmin ^ kmax;
    const int passes = diff ? (64 - __clzll((long long)diff) + 7) / 8 : 0;
    uint64_t* ks = kin; int32_t* vs = vin; uint64_t* kd = kout; int32_t* vd = vout;
    for (int p = 0; p < passes; ++p) {
        // digit totals over the bucket
        for (int i = threadIdx.x; i < kWaves * 256; i += kSsLocalThreads) (&L.wcnt[0][0])[i] = 0;
        __syncthreads();
        for (int32_t c0 = 0; c0 < size; c0 += kSsCap) {
            const int nv = size - c0 < kSsCap ? size - c0 : kSsCap;
            #pragma unroll
            for (int q = 0; q < kSsLocalRounds; ++q) {
                const int i = (wave * kSsLocalRounds + q) * 64 + lane;
                kr[q] = i < nv ? load_coherent(ks + start + c0 + i) : 0ull;
            }
            ss_rank_digits(kr, 8 * p, kSsLocalRounds, nv, L.wcnt, dg, rk);   // wcnt accumulates over the chunks
        }
        __syncthreads();
        {
            int32_t c = 0;
            if (threadIdx.x < 256)
                for (int v = 0; v < kWaves; ++v) c += L.wcnt[v][threadIdx.x];
            const int32_t incl = wave_incl_scan(c);
            if (lane == 63) L.wtot[wave] = incl;
            __syncthreads();
            int32_t ex = incl - c;
            for (int v = 0; v < wave; ++v) ex += L.wtot[v];
            if (threadIdx.x < 256) gb[threadIdx.x] = ex;   // the digit's next free place in the bucket
        }
        __syncthreads();
        for (int32_t c0 = 0; c0 < size; c0 += kSsCap) {
            const int nv = size - c0 < kSsCap ? size - c0 : kSsCap;
            #pragma unroll
            for (int q = 0; q < kSsLocalRounds; ++q) {
                const int i = (wave * kSsLocalRounds + q) * 64 + lane;
                kr[q] = i < nv ? load_coherent(ks + start + c0 + i) : 0ull;
                vr[q] = i < nv ? load_coherent(vs + start + c0 + i) : 0;
            }
            for (int i = threadIdx.x; i < kWaves * 256; i += kSsLocalThreads) (&L.wcnt[0][0])[i] = 0;
            __syncthreads();
            ss_rank_digits(kr, 8 * p, kSsLocalRounds, nv, L.wcnt, dg, rk);
            __syncthreads();
            const int32_t c = ss_digit_starts(L.wcnt, 0, L.wtot);   // chunk-local starts
            __syncthreads();
            #pragma unroll
            for (int q = 0; q < kSsLocalRounds; ++q) {
                if (dg[q] >= 0) {
                    // the digit's next free place + the key's offset among the chunk's keys of that digit
                    const int32_t dst = gb[dg[q]] + (L.wcnt[wave][dg[q]] + rk[q]) - L.wcnt[0][dg[q]];
                    kd[start + dst] = kr[q];
                    vd[start + dst] = vr[q];
                }
            }
            __syncthreads();
            if (threadIdx.x < 256) gb[threadIdx.x] += c;
            __syncthreads();
        }
        uint64_t* tk = ks; ks = kd; kd = tk;
        int32_t* tv = vs; vs = vd; vd = tv;
    }
    if (ks != kout) {   // an even number of passes: the result is still in (kin, vin)
        for (int32_t i = threadIdx.x; i < size; i += kSsLocalThreads) {
            kout[start + i] = load_coherent(kin + start + i);
            vout[start + i] = load_coherent(vin + start + i);
        }
    }
}

// ---------------------------------------------------------------------------
// Staircases of the local region (the product decided exactly):
//   K[j]  = #{k : omega_j r_k <= z}   (rows; K is nonincreasing in j)
//   Jc[k] = #{j : omega_j r_k <= z}   (columns; Jc is nonincreasing in k)
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool exact_le(double a, double b, double z)
{
    dd p = two_prod(a, b);
    if (p.hi < z) return true;
    if (p.hi > z) return false;
    return p.lo <= 0.0;
}

// One wave per 64 consecutive queries.  The queries are sorted, so the counts
// are nonincreasing along the wave: the counts of the wave's first and last
// queries come first, each from a 32-ary search by one half of the wave (32
// probes per step split the range into 33 parts), then every lane finishes
// with a binary search inside that bracket (a few steps where the sorted
// points are spread evenly).
__device__ __forceinline__ void staircase_body(const double* __restrict__ sorted, int32_t len,
                                               const double* __restrict__ q, int32_t nq, double z,
                                               int32_t* __restrict__ out, int32_t bid)
{
    const int lane = threadIdx.x & 63;
    const int32_t j0 = (int32_t)((bid * blockDim.x + threadIdx.x) & ~63u);
    if (j0 >= nq) return;                              // the whole wave
    const int32_t jl = j0 + 63 < nq ? j0 + 63 : nq - 1;
    const int half = lane >> 5, hl = lane & 31;
    const double wt = q[half ? jl : j0];
    // the count (first index whose product exceeds z) lies in [lo, hi]
    int32_t lo = 0, hi = len;
    while (hi - lo > 32) {
        const int64_t span = hi - lo;
        const int32_t pos = lo + (int32_t)(((int64_t)(hl + 1) * span) / 33);   // lo < pos < hi
        const uint64_t b = __ballot(exact_le(wt, sorted[pos], z));
        const int c = __popc(half ? (uint32_t)(b >> 32) : (uint32_t)b);        // probes at or below z
        const int32_t nlo = c > 0 ? lo + (int32_t)(((int64_t)c * span) / 33) + 1 : lo;
        const int32_t nhi = c < 32 ? lo + (int32_t)(((int64_t)(c + 1) * span) / 33) : hi;
        lo = nlo;
        hi = nhi;
    }
    {
        const int32_t pos = lo + hl;
        const uint64_t b = __ballot(pos < hi && exact_le(wt, sorted[pos], z));
        lo += __popc(half ? (uint32_t)(b >> 32) : (uint32_t)b);
    }
    const int32_t top = __shfl(lo, 0), bottom = __shfl(lo, 32);
    const int32_t j = j0 + lane;
    if (j > jl) return;
    const double w = q[j];
    lo = bottom;
    hi = top;
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (exact_le(w, sorted[mid], z)) lo = mid + 1; else hi = mid;
    }
    out[j] = lo;
}

// Both staircases of a geometry in one launch (they are independent): the
// first nba workgroups count, for each sorted frequency, the sorted points
// whose product with it is at most z (K); the rest count, for each sorted
// point, the sorted frequencies (Jc).  One launch fewer on the plan's path.
__device__ __forceinline__ void staircases(const PlanArgs& a)
{
    const PlanDev& P = a.P;
    const int32_t nba = (P.m + 255) / 256;
    if ((int32_t)blockIdx.x < nba) staircase_body(P.rs, P.n, P.ws, P.m, P.z, a.K, blockIdx.x);
    else staircase_body(P.ws, P.m, P.rs, P.n, P.z, a.Jc, blockIdx.x - nba);
}

// ---------------------------------------------------------------------------
// Alg. 1 (Subdivide), level by level in one 256-thread block.  Every mixed
// block of a level becomes a Node; its split follows the quasi-optimal
// SplitIndices of Sec. 4.1 (candidate rows equispaced over the rows that hold
// a local entry, minimal mixed area, ties to the smaller row).  Numbering is
// deterministic: nodes in level order, children in (parent, position) order.
//
// A level is a chain of latencies (its nodes' headers, their candidates, the
// scans, the stores: 5 us and more per 256 nodes), so for large transforms the
// first workgroup stops at a level of kSubFront nodes or more, a workgroup
// each subdivides the subtrees below (k_subtrees), and a third kernel numbers
// them one after the other and writes their blocks (k_subtree_blocks).
// ---------------------------------------------------------------------------
// The split of one mixed node (Alg. 1) and the classes of its children.
struct NodeSplit {
    int32_t js, ks;
    bool cl, ca, ur_m, ur_d, ll_m, ll_d;
};

// Candidate counts up to this are evaluated with all their loads in flight.
constexpr int32_t kSplitUnroll = 16;

// kj1 = K[R.j1], kj0 = K[R.j0], jc = Jc[R.k0], loaded by the caller.  G
// consecutive lanes (a power of two up to kSplitUnroll) share a node.
template <int G>
__device__ __forceinline__ NodeSplit split_node(const Rect& R, int32_t kj1, int32_t kj0, int32_t jc,
                                                const int32_t* __restrict__ K, int64_t min_size, int32_t ncand)
{
    NodeSplit o;
    int32_t js = 0, ks = 0;
    if (kj1 >= R.k1 + 1) {              // wholly local
        js = R.j1; ks = R.k1;
    } else if (kj0 <= R.k0) {           // wholly asymptotic
        js = R.j0 - 1; ks = R.k0 - 1;
    } else {
        // the last row holding a local entry: K[j] > k0 <=> j < Jc[k0]
        int32_t jl = jc - 1;
        if (jl > R.j1) jl = R.j1;
        int64_t best = INT64_MAX;
        int32_t span = jl - R.j0;
        // more candidates than rows is every row (the exact optimum)
        int32_t nc = span > 0 ? (ncand <= span ? ncand : span + 1) : 1;
        // candidate c is row j0 + floor(c span / (nc - 1)): the product with the
        // divisor's reciprocal is within one of the quotient, and the remainder
        // (exact: c span < 2^53) sets it right.  (A division per candidate
        // made a level 7 us, of which this function 4.7.)
        const double dspan = (double)span, div = (double)(nc > 1 ? nc - 1 : 1), rdiv = 1.0 / div;
        const bool every = nc == span + 1;                  // every row
        auto row_of = [&](int32_t c) {
            const double x = (double)c * dspan;
            double q = floor(x * rdiv);
            const double rem = __builtin_fma(-q, div, x);
            q += rem < 0.0 ? -1.0 : rem >= div ? 1.0 : 0.0;
            return R.j0 + (every ? c : (int32_t)q);
        };
        auto consider = [&](int32_t j, int32_t kraw) {
            int32_t k = kraw - 1;
            if (k > R.k1) k = R.k1;
            if (k < R.k0) k = R.k0 - 1;
            int64_t mixed = (int64_t)(j - R.j0 + 1) * (R.k1 - k) + (int64_t)(R.j1 - j) * (k - R.k0 + 1);
            if (mixed < best) { best = mixed; js = j; ks = k; }
        };
        if (nc <= kSplitUnroll) {
            // all candidate loads in flight together, then taken in order
            constexpr int32_t kPer = kSplitUnroll / G;
            const int32_t sub = threadIdx.x % G;
            int32_t jv[kPer], kv[kPer];
            #pragma unroll
            for (int32_t q = 0; q < kPer; ++q) {
                const int32_t c = sub + G * q;
                jv[q] = row_of(c < nc ? c : 0);
                kv[q] = K[jv[q]];
            }
            #pragma unroll
            for (int32_t q = 0; q < kPer; ++q)
                if (sub + G * q < nc) consider(jv[q], kv[q]);
            // the lanes' minima: rows increase with the candidate, so ties go
            // to the smaller row
            #pragma unroll
            for (int32_t g = 1; g < G; g <<= 1) {
                const int64_t om = __shfl_xor(best, g);
                const int32_t oj = __shfl_xor(js, g), ok = __shfl_xor(ks, g);
                if (om < best || (om == best && oj < js)) { best = om; js = oj; ks = ok; }
            }
        } else {
            // batches of kSplitUnroll candidates with their loads in flight
            for (int32_t c0 = 0; c0 < nc; c0 += kSplitUnroll) {
                int32_t jv[kSplitUnroll], kv[kSplitUnroll];
                #pragma unroll
                for (int32_t c = 0; c < kSplitUnroll; ++c) {
                    jv[c] = row_of(c0 + c < nc ? c0 + c : c0);
                    kv[c] = K[jv[c]];
                }
                #pragma unroll
                for (int32_t c = 0; c < kSplitUnroll; ++c)
                    if (c0 + c < nc) consider(jv[c], kv[c]);
            }
        }
    }
    o.js = js; o.ks = ks;
    o.cl = ks >= R.k0 && js >= R.j0;
    o.ca = js < R.j1 && ks < R.k1;
    o.ur_m = o.ur_d = o.ll_m = o.ll_d = false;
    if (ks < R.k1 && js >= R.j0) {
        if ((int64_t)(js - R.j0 + 1) * (R.k1 - ks) > min_size) o.ur_m = true; else o.ur_d = true;
    }
    if (js < R.j1 && ks >= R.k0) {
        if ((int64_t)(R.j1 - js) * (ks - R.k0 + 1) > min_size) o.ll_m = true; else o.ll_d = true;
    }
    return o;
}

// Workgroups of the subdivision, a node a thread (several a thread would
// serialise their candidate loads).  256 threads rather than 1024:
// a 1024-thread workgroup needs a compute unit with sixteen free wave slots,
// which the execution running beside the plan rarely leaves.
constexpr int kSubThreads = 256;
// The first entries of each level's queue live in LDS (the queue of the next
// level is written while the current one is read, so two buffers); entries
// past them go to the global queues at the same index.
constexpr int kSubLds = 1920;

__device__ __forceinline__ DBlock direct_block(int32_t j0, int32_t j1, int32_t k0, int32_t k1)
{
    return DBlock{j0, j1, k0, k1, 0, 0, 0.0, 0.0, 0.0, 0.0};
}

// Counts of a subdivision: nodes, blocks of each kind, levels, and what
// overflowed (kOver*).
struct SubCounts {
    int32_t nodes, l, a, d, level, overflow;
};

__device__ __forceinline__ LBlock local_block(int32_t j0, int32_t j1, int32_t k0, int32_t k1, int32_t level)
{
    LBlock b;
    b.j0 = j0; b.j1 = j1; b.k0 = k0; b.k1 = k1;
    b.R = 0.0; b.item0 = 0; b.nitems = 0; b.level = level;
    b.K = 0; b.pr = 0; b.slot0 = 0; b.D = 0.0; b.rw = 0.0;
    return b;
}

__device__ __forceinline__ ABlock asymptotic_block(int32_t j0, int32_t j1, int32_t k0, int32_t k1, int32_t level)
{
    ABlock b = {};
    b.j0 = j0; b.j1 = j1; b.k0 = k0; b.k1 = k1; b.level = level;
    return b;
}

// The levels from the n_cur = 1 block in lq[0][0] on, counted on from c.
// SUB: nodes alone, into nodes[0 .. node_cap), with the subtree's own numbers;
// else nodes and blocks into A's tables, up to a level of `stop` nodes (whose
// blocks are then in lq[*buf], *left of them).  q0, q1 (q_cap entries): queue
// entries past the LDS.
template <bool SUB>
__device__ __forceinline__ void subdivide_levels(const PlanArgs& a, Rect (*lq)[kSubLds], int32_t (*wsum)[16],
                                                 Node* __restrict__ nodes, int32_t node_cap, Rect* q0, Rect* q1,
                                                 int32_t q_cap, int32_t stop, SubCounts& c, int32_t* left, int* buf)
{
    const int32_t* __restrict__ K = a.K;
    const int32_t* __restrict__ Jc = a.Jc;
    const Arena& A = a.A;
    const int32_t ncand = a.ncand;
    const int64_t min_size = a.min_size;
    const int tid = threadIdx.x;
    Rect* cur = q0;
    Rect* nxt = q1;
    int cb = 0;                                      // LDS buffer of the current level
    int32_t n_cur = 1;
    int32_t n_nodes = c.nodes, n_l = c.l, n_a = c.a, n_d = c.d, level = c.level, overflow = 0;
    while (n_cur > 0 && n_cur < stop) {
        ++level;
        int32_t n_next = 0;
        for (int32_t c0 = 0; c0 < n_cur; c0 += kSubThreads) {
            // a short level: sixteen lanes a node (a level 7 us with one, 3.5 so)
            const bool wide = n_cur <= kSubThreads / kSplitUnroll;
            const int32_t i = wide ? tid / kSplitUnroll : c0 + tid;
            bool act = i < n_cur;
            const Rect R = act ? (i < kSubLds ? lq[cb][i] : cur[i - kSubLds]) : Rect{0, 0, 0, 0};
            const int32_t kj1 = K[R.j1], kj0 = K[R.j0], jc = Jc[R.k0];   // all header loads in flight together
            NodeSplit o;
            int32_t v[4] = {0, 0, 0, 0};
            if (act) {
                if (wide) o = split_node<kSplitUnroll>(R, kj1, kj0, jc, K, min_size, ncand);
                else o = split_node<1>(R, kj1, kj0, jc, K, min_size, ncand);
            }
            act = act && (!wide || tid % kSplitUnroll == 0);
            if (act) {
                v[0] = o.cl;
                v[1] = o.ca;
                v[2] = (int)o.ur_d + (int)o.ll_d;
                v[3] = (int)o.ur_m + (int)o.ll_m;
            }
            int32_t tot[4];
            block_scan<int32_t, 4, kSubThreads / 64>(v, tot, wsum);
            int32_t l_slot = n_l + v[0], a_slot = n_a + v[1], d_slot = n_d + v[2], m_slot = n_next + v[3];
            const int32_t next_base = n_nodes + n_cur;   // first node index of the next level
            if (act) {
                const int32_t node = n_nodes + i;
                Node nd;
                nd.j0 = R.j0; nd.j1 = R.j1; nd.k0 = R.k0; nd.k1 = R.k1;
                nd.js = o.js; nd.ks = o.ks;
                nd.lblk = o.cl ? l_slot : -1;
                nd.ablk = o.ca ? a_slot : -1;
                nd.level = level; nd.pad = 0;
                nd.ur = -1; nd.ll = -1;
                auto queue = [&](const Rect& child) {
                    if (m_slot < kSubLds) lq[cb ^ 1][m_slot] = child;
                    else if (m_slot - kSubLds < q_cap) nxt[m_slot - kSubLds] = child;
                    return next_base + m_slot++;
                };
                auto direct = [&](int32_t j0, int32_t j1, int32_t k0, int32_t k1) {
                    if constexpr (!SUB)
                        if (d_slot < A.d_cap) A.db[d_slot] = direct_block(j0, j1, k0, k1);
                    return encode_direct(d_slot++);
                };
                if (o.ur_m) nd.ur = queue(Rect{R.j0, o.js, o.ks + 1, R.k1});
                if (o.ur_d) nd.ur = direct(R.j0, o.js, o.ks + 1, R.k1);
                if (o.ll_m) nd.ll = queue(Rect{o.js + 1, R.j1, R.k0, o.ks});
                if (o.ll_d) nd.ll = direct(o.js + 1, R.j1, R.k0, o.ks);
                if (node < node_cap) nodes[node] = nd;
                if constexpr (!SUB) {
                    if (o.cl && l_slot < A.l_cap) A.lb[l_slot] = local_block(R.j0, o.js, R.k0, o.ks, level);
                    if (o.ca && a_slot < A.a_cap)
                        A.ab[a_slot] = asymptotic_block(o.js + 1, R.j1, o.ks + 1, R.k1, level);
                }
            }
            n_l += tot[0];
            n_a += tot[1];
            n_d += tot[2];
            n_next += tot[3];
        }
        n_nodes += n_cur;
        if (n_next - kSubLds > q_cap) overflow = kOverQueue;
        if (level >= kMaxLevels) overflow = kOverLevels;
        Rect* t = cur; cur = nxt; nxt = t;
        cb ^= 1;
        n_cur = overflow ? 0 : n_next;
        __syncthreads();
    }
    if (!overflow && n_nodes > node_cap) overflow = kOverTables;
    c = SubCounts{n_nodes, n_l, n_a, n_d, level, overflow};
    *left = n_cur;
    *buf = cb;
}

__device__ __forceinline__ void store_counts(Summary* __restrict__ sum, const Arena& A, const SubCounts& c)
{
    sum->n_nodes = c.nodes; sum->n_l = c.l; sum->n_a = c.a; sum->n_d = c.d;
    sum->levels = c.level;
    const bool stopped = c.overflow == kOverLevels || c.overflow == kOverQueue;
    sum->overflow = !stopped && (c.nodes > A.node_cap || c.l > A.l_cap || c.a > A.a_cap || c.d > A.d_cap)
                        ? kOverTables : c.overflow;
}

__device__ __forceinline__ void subdivide(const PlanArgs& a)
{
    Summary* __restrict__ sum = a.sum;
    const Arena& A = a.A;
    const int32_t m = a.P.m, n = a.P.n, n_errs = a.n_errs;
    __shared__ int32_t wsum[4][16];
    __shared__ Rect lq[2][kSubLds];
    const int tid = threadIdx.x;
    // the summary starts clear (this is the first planning kernel to use it),
    // with the input check's verdict
    int bad = 0;
    for (int32_t i = tid; i < n_errs; i += kSubThreads) bad |= a.errs[i];
    bad = __syncthreads_or(bad);
    if (tid == 0) {
        *sum = Summary{};
        sum->domain_error = bad ? 1 : 0;
        lq[0][0] = Rect{0, m - 1, 0, n - 1};
    }
    __syncthreads();
    SubCounts c{0, 0, 0, 0, 0, 0};
    int32_t left = 0;
    int buf = 0;
    if (m > 0 && n > 0)
        subdivide_levels<false>(a, lq, wsum, A.nodes, A.node_cap, A.q0, A.q1, A.q_cap, A.sub ? kSubFront : INT32_MAX,
                                c, &left, &buf);
    if (A.sub) {
        // the subtrees' roots are numbered after the nodes above them
        if (tid < left) {
            const Rect R = lq[buf][tid];
            int32_t* q = A.sub + kSubRoots + 4 * tid;
            q[0] = R.j0; q[1] = R.j1; q[2] = R.k0; q[3] = R.k1;
        }
        if (tid == 0) {
            A.sub[0] = left;
            A.sub[1] = c.nodes; A.sub[2] = c.l; A.sub[3] = c.a; A.sub[4] = c.d; A.sub[5] = c.level;
        }
    }
    if (tid == 0) store_counts(sum, A, c);
}

// Subtree blockIdx.x: its nodes, numbered on their own, into its share of the
// staging table, its counts into A.sub.
__global__ __launch_bounds__(kSubThreads) void k_subtrees(PlanArgs a)
{
    const Arena& A = a.A;
    __shared__ int32_t wsum[4][16];
    __shared__ Rect lq[2][kSubLds];
    const int t = blockIdx.x;
    const int32_t trees = A.sub[0];
    if (t >= trees) return;
    const int32_t* q = A.sub + kSubRoots + 4 * t;
    if (threadIdx.x == 0) lq[0][0] = Rect{q[0], q[1], q[2], q[3]};
    __syncthreads();
    const int32_t cap = A.node_cap / trees, qcap = A.q_cap / trees;
    SubCounts c{0, 0, 0, 0, A.sub[5], 0};
    int32_t left;
    int buf;
    subdivide_levels<true>(a, lq, wsum, A.stage + (int64_t)t * cap, cap, A.q0 + (int64_t)t * qcap,
                           A.q1 + (int64_t)t * qcap, qcap, INT32_MAX, c, &left, &buf);
    if (threadIdx.x == 0) {
        int32_t* o = A.sub + kSubCounts + 8 * t;
        o[0] = c.nodes; o[1] = c.l; o[2] = c.a; o[3] = c.d; o[4] = c.level; o[5] = c.overflow;
    }
}

// Numbers subtree blockIdx.x after the subtrees before it and writes its nodes
// and blocks.
__global__ __launch_bounds__(kSubThreads) void k_subtree_blocks(PlanArgs a)
{
    static_assert(kSubThreads == kSubTrees, "a thread a subtree");
    const Arena& A = a.A;
    __shared__ int32_t wsum[4][16];
    __shared__ int32_t first[4], top[2];
    const int t = blockIdx.x, tid = threadIdx.x;
    const int32_t trees = A.sub[0];
    if (t >= trees) return;
    const int32_t* o = A.sub + kSubCounts + 8 * tid;
    const bool on = tid < trees;
    int32_t v[4] = {on ? o[0] - 1 : 0, on ? o[1] : 0, on ? o[2] : 0, on ? o[3] : 0};   // nodes below the root
    int32_t tot[4];
    if (tid == 0) top[0] = top[1] = 0;
    __syncthreads();
    if (on) { atomicMax(&top[0], o[4]); atomicMax(&top[1], o[5]); }
    block_scan<int32_t, 4, kSubThreads / 64>(v, tot, wsum);
    if (tid == t)
        for (int q = 0; q < 4; ++q) first[q] = v[q];
    __syncthreads();
    const int32_t roots = A.sub[1];
    if (t == 0 && tid == 0)
        store_counts(a.sum, A, SubCounts{roots + trees + tot[0], A.sub[2] + tot[1], A.sub[3] + tot[2],
                                         A.sub[4] + tot[3], top[0], top[1] == kOverTables ? kOverShare : top[1]});
    if (top[1]) return;
    const int32_t node0 = roots + trees + first[0] - 1;   // node i > 0 of the subtree is node0 + i
    const int32_t l0 = A.sub[2] + first[1], a0 = A.sub[3] + first[2], d0 = A.sub[4] + first[3];
    const int32_t nodes = A.sub[kSubCounts + 8 * t];
    const Node* __restrict__ stage = A.stage + (int64_t)t * (A.node_cap / trees);
    for (int32_t i = tid; i < nodes; i += kSubThreads) {
        Node nd = stage[i];
        if (nd.lblk >= 0) {
            nd.lblk += l0;
            if (nd.lblk < A.l_cap) A.lb[nd.lblk] = local_block(nd.j0, nd.js, nd.k0, nd.ks, nd.level);
        }
        if (nd.ablk >= 0) {
            nd.ablk += a0;
            if (nd.ablk < A.a_cap) A.ab[nd.ablk] = asymptotic_block(nd.js + 1, nd.j1, nd.ks + 1, nd.k1, nd.level);
        }
        if (nd.ur >= 0) nd.ur += node0;
        else if (nd.ur <= -2) {
            const int32_t d = decode_direct(nd.ur) + d0;
            if (d < A.d_cap) A.db[d] = direct_block(nd.j0, nd.js, nd.ks + 1, nd.k1);
            nd.ur = encode_direct(d);
        }
        if (nd.ll >= 0) nd.ll += node0;
        else if (nd.ll <= -2) {
            const int32_t d = decode_direct(nd.ll) + d0;
            if (d < A.d_cap) A.db[d] = direct_block(nd.js + 1, nd.j1, nd.k0, nd.ks);
            nd.ll = encode_direct(d);
        }
        const int32_t node = i == 0 ? roots + t : node0 + i;
        if (node < A.node_cap) A.nodes[node] = nd;
    }
}

// ---------------------------------------------------------------------------
// Per-block parameters: 16 lanes per asymptotic block, a lane per local block
// (grid-stride over the blocks the subdivision made).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int32_t iceil(double x) { return (int32_t)ceil(x); }

// Terms of a Chebyshev expansion of  H(omega r) e^{i (omega - D)(r - C)}  (H:
// Hankel's terms) over an interval of one of the two variables, centre `cen`
// and half-width `half` > 0, the other at least `other` and off its centre by
// at most xi / half.  On the ellipse with foci at the interval's ends and
// semi-axes summing to rho the exponential is at most e^{xi (rho - 1/rho)/2}
// and H at most its terms' sum at the smallest omega r there, so the
// interpolant of K terms is off by at most 4 max / ((rho - 1) rho^(K-1))
// (Trefethen, Approximation Theory and Approximation Practice, Thm. 8.2).
// Sixteen lanes take a rho each; the result is the smallest K over them.
__device__ __forceinline__ double rank_terms(const PlanDev& P, double cen, double half, double other, double xi)
{
    if (!(half > 0.0)) return 1.0;
    const double lr = kRankLr0 + kRankLrStep * (threadIdx.x & 15);
    const double rho = exp(lr), inv = 1.0 / rho;
    double H = fabs(P.chan[0]);
    bool ok = true;
    if (!P.rank_const) {
        const double x = (cen - 0.5 * half * (rho + inv)) * other;
        ok = x > 0.0;
        const double ix = ok ? 1.0 / x : 0.0;
        double v = 0.0;
        for (int p = 2 * P.M - 1; p >= 0; --p) v = v * ix + fabs(P.chan[p]);
        H = v;
    }
    double k = (log(4.0 * H) + 0.5 * xi * (rho - inv) - log(rho - 1.0) - P.rank_ltol) / lr + 1.0;
    if (!ok || !(k < 1e9)) k = 1e9;
    if (k < 1.0) k = 1.0;
    for (int o = 8; o >= 1; o >>= 1) k = fmin(k, __shfl_xor(k, o));
    return k;
}

// Panels of one variable: the fewest equal panels (from xi on) whose
// expansions need at most kRankK terms -- the panel at the smallest values is
// the worst, as H varies fastest there.  Returns the panels (0: more than
// `most`), their terms in *terms.
__device__ __forceinline__ int rank_panels(const PlanDev& P, double lo, double span_half, double other, double xi,
                                           int32_t most, double* terms)
{
    int pc = (int)ceil(fmin(xi / P.rank_xi, 1e6));
    if (pc < 1) pc = 1;
    while (pc <= most) {
        const double half = span_half / pc;
        const double k = rank_terms(P, lo + half, half, other, xi / pc);
        if (k <= (double)kRankK) { *terms = k; return pc; }
        pc += pc < 64 ? (pc + 1) / 2 : pc / 8;
    }
    return 0;
}

// Rows a node of an FFT-path block's expansions has to replace.  At 1e6 rows
// (order 0, 8 channels) a node takes 0.21 ns, and a row 0.054 ns less through
// an expansion than from the grid: even at 4, with a launch more.
constexpr int kRowsPerNode = 5;
constexpr int32_t kRankRowPanels = 1 << 17;

// Half-width of each of `panels` panels over a half-range: rounded up to 40
// bits, so that the panels' middles (small integers times it) are exact and
// evenly spaced.
__device__ __forceinline__ double rank_half_width(double half_range, int panels)
{
    const double h = half_range / panels;
    if (panels == 1 || h == 0.0) return h;
    return __longlong_as_double((__double_as_longlong(h) + ((1ll << 12) - 1)) & ~((1ll << 12) - 1));
}

__device__ __forceinline__ void block_params(const PlanArgs& a)
{
    const PlanDev& P = a.P;
    const Arena& A = a.A;
    Summary* __restrict__ sum = a.sum;
    const int32_t dft_max = a.dft_max;
    const double sigma = a.sigma;
    if (sum->overflow) return;
    const int32_t n_l = sum->n_l, n_a = sum->n_a, n_d = sum->n_d;
    const int w = P.w;
    const int lane = threadIdx.x & 15;
    const int32_t group = (int32_t)((blockIdx.x * blockDim.x + threadIdx.x) >> 4), groups = (int32_t)((gridDim.x * blockDim.x) >> 4);
    for (int32_t b = group; b < n_a; b += groups) {
        ABlock B = A.ab[b];
        double rlo = P.rs[B.k0], rhi = P.rs[B.k1];
        double wlo = P.ws[B.j0], whi = P.ws[B.j1];
        double C = 0.5 * (rlo + rhi);
        double X = fmax(rhi - C, C - rlo);
        double D = 0.5 * (wlo + whi);
        double S = fmax(whi - D, D - wlo);
        B.K = 0; B.pc = 0; B.pr = 0; B.cw = 0.0; B.rw = 0.0;
        // (half-widths too small for their reciprocals stay on the ES path)
        if (P.rank && (X == 0.0 || X > 1e-290) && (S == 0.0 || S > 1e-290)) {
            const double xi = X * S;
            double kc = 1.0, kr = 1.0;
            const int pc = rank_panels(P, rlo, X, wlo, xi, kRankPanels, &kc);
            const int pr = pc > 0 ? rank_panels(P, wlo, S, rlo, xi, 64, &kr) : 0;
            if (pc > 0 && pr > 0) {
                int K = ((int)ceil(fmax(kc, kr)) + 3) & ~3;
                B.K = K < 4 ? 4 : K;
                B.pc = pc; B.pr = pr;
                B.cw = rank_half_width(X, pc); B.rw = rank_half_width(S, pr);
            }
        }
        const double S_rows = S;
        if (!(S > 1e-280)) S = 1e-280;
        // grid spacing: the largest power of two with S h <= pi / sigma
        double h = exp2(floor(log2(kPi / (sigma * S))));
        if (S * h > kPi / sigma) h *= 0.5;
        double span = X / h;
        if (!(span < (double)(1 << (kMaxFftLog2 - 3)))) {   // grid too large for the FFT sizes
            if (lane == 0) atomicOr(&sum->grid_error, 1);
            span = 0.0;
        }
        int32_t llo = iceil(-span - 0.5 * w) - 1;
        int32_t lhi = iceil(span - 0.5 * w) + w;
        int32_t N1 = lhi - llo + 1;
        B.C = C; B.D = D; B.h = h; B.r0 = rlo; B.alpha = 0.5 * w * h;
        B.llo = llo; B.N1 = N1;
        int32_t fft = (B.K > 0 || (dft_max >= 0 && N1 <= dft_max)) ? 0 : 1;
        int32_t N2 = 0;
        if (fft) {
            int32_t maxl = llo < 0 ? -llo : llo;
            if (lhi > maxl) maxl = lhi;
            N2 = 64;
            while (N2 < 4 * maxl + 4) N2 <<= 1;
            // h N2 / (2 pi): exact scaling of the double-double 1/(2 pi)
            B.Khi = h * (double)N2 * kInvTwoPi;
            B.Klo = h * (double)N2 * kInvTwoPiLo;
        }
        B.fft = fft; B.N2 = N2;
        // rows of an FFT-path block through expansions on panels of
        // frequencies, where they outnumber the nodes by kRowsPerNode
        B.rK = B.K;
        if (P.rank && fft && X > 1e-290 && S_rows > 1e-290) {
            double kr = 1.0;
            const int pr = rank_panels(P, wlo, S_rows, rlo, X * S_rows, kRankRowPanels, &kr);
            const int K = ((int)ceil(kr) + 3) & ~3;
            if (pr > 0 && (int64_t)kRowsPerNode * K * pr <= B.j1 - B.j0 + 1) {
                B.rK = K;
                B.pr = pr;
                B.rw = rank_half_width(S_rows, pr);
            }
        }
        int32_t ncol = B.k1 - B.k0 + 1;
        B.nitems = (ncol + P.spread_chunk - 1) / P.spread_chunk;
        if (lane == 0) {
            A.ab[b] = B;
            A.ascan[b] = AScan{B.nitems, B.K > 0 ? 0 : fft ? N2 : N1, B.pc, B.pr, B.j1 - B.j0 + 1, ncol,
                               B.K > 0 ? -1 : fft ? 31 - __clz(N2) : 0, B.rK == 0 ? 1 : 0,
                               B.K > 0 ? 0 : (int64_t)(fft ? N2 : N1) * (grid_crowded(N1, B.nitems, w) ? P.nch : 1), 0};
        }
    }
    long long entries = 0;
    for (int32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < n_d; b += gridDim.x * blockDim.x) {
        DBlock E = A.db[b];
        entries += (long long)(E.j1 - E.j0 + 1) * (E.k1 - E.k0 + 1);
        const double rlo = P.rs[E.k0], rhi = P.rs[E.k1], wlo = P.ws[E.j0], whi = P.ws[E.j1];
        E.C = 0.5 * (rlo + rhi);
        E.D = 0.5 * (wlo + whi);
        E.cw = fmax(rhi - E.C, E.C - rlo);
        E.rw = fmax(whi - E.D, E.D - wlo);
        // J_nu(omega r) is entire in either variable and at most e^{|Im|}, so
        // the width of an expansion is its half-range times the largest value
        // of the other variable.  Taken when its work -- a point 2 K + 20
        // operations, a node pair about 60, a row 2 K -- is less than half of
        // the entries' 45 each.
        const double xi = fmax(E.cw * whi, E.rw * rhi);
        const bool ok = (E.cw == 0.0 || E.cw > 1e-290) && (E.rw == 0.0 || E.rw > 1e-290);
        if (ok && xi <= P.direct_xi[kRankK / 4 - 1]) {
            int i = 0;
            while (i < kRankK / 4 - 1 && xi > P.direct_xi[i]) ++i;
            const double K = 4.0 * (i + 1), mb = E.j1 - E.j0 + 1, nb = E.k1 - E.k0 + 1;
            if (2.0 * (nb * (2.0 * K + 20.0) + 60.0 * K * K + 2.0 * K * mb) < 45.0 * mb * nb) E.K = (int32_t)K;
        }
        A.db[b] = E;
        if (E.K == 0 && (P.jtab_np == 0 || wlo * rlo < P.jtab_x0)) {
            const int64_t area = (int64_t)(E.j1 - E.j0 + 1) * (E.k1 - E.k0 + 1);
            atomicMax(&sum->d_area, area < INT32_MAX ? (int32_t)area : INT32_MAX);
        }
    }
    if (__ballot(entries != 0)) {
        for (int o = 32; o >= 1; o >>= 1) entries += __shfl_xor(entries, o);
        if ((threadIdx.x & 63) == 0) atomicAdd((unsigned long long*)&sum->d_ent, (unsigned long long)entries);
    }
    for (int32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < n_l; b += gridDim.x * blockDim.x) {
        LBlock L = A.lb[b];
        double R = P.rs[L.k1];
        if (R == 0.0) {
            double wm = P.ws[L.j1];
            R = wm > 0.0 ? P.z / wm : 1.0;
        }
        L.R = R;
        int32_t ncol = L.k1 - L.k0 + 1;
        L.nitems = (ncol + local_chunk(P.n) - 1) / local_chunk(P.n);
        // rows: panels of as many terms as their share of xi = S R needs,
        // unless they have more nodes than the block has rows
        const double wlo = P.ws[L.j0], whi = P.ws[L.j1];
        const double D = 0.5 * (wlo + whi), S = fmax(whi - D, D - wlo), xi = S * R;
        const double pr = ceil(xi / P.local_xi[kRankK / 4 - 1]);
        L.D = D;
        L.K = 0; L.pr = 0; L.rw = 0.0;
        if (pr < 1e6 && (S == 0.0 || S > 1e-290)) {
            L.pr = pr < 1.0 ? 1 : (int32_t)pr;
            int i = 0;
            while (i < kRankK / 4 - 1 && xi / L.pr > P.local_xi[i]) ++i;
            L.K = 4 * (i + 1);
            L.rw = rank_half_width(S, L.pr);
            if ((int64_t)L.K * L.pr > L.j1 - L.j0 + 1) L.K = 0;
        }
        A.lb[b] = L;
        A.lscan[b] = LScan{L.nitems, local_slots(L), L.j1 - L.j0 + 1, ncol};
    }
}

// ---------------------------------------------------------------------------
// Offsets and totals: exclusive scans over the blocks of item counts and grid
// slots, the FFT size classes, membership statistics.  A workgroup takes a run
// of blocks: it first adds up all blocks (and those before its run), then
// scans its own, so that none waits for another (one workgroup over 12000
// blocks of each kind took 117 us).  The workgroups, as that of the scan over
// the items, are of kPlanScanThreads (at most 128 VGPRs per wave): a workgroup
// this small fits on a compute unit as soon as one workgroup of a running
// transform's kernels retires there, where a 1024-thread one waits for a whole
// compute unit to drain.
// ---------------------------------------------------------------------------
constexpr int kPlanScanThreads = 256;
constexpr int kPlanScanBlocks = 16;                  // workgroups of the scan over the blocks

__device__ __forceinline__ void plan_scan(const PlanArgs& a)
{
    const PlanDev& P = a.P;
    const Arena& A = a.A;
    Summary* __restrict__ sum = a.sum;
    constexpr int kVpt = 4;                          // blocks of a kind per thread per pass (1024 per pass)
    constexpr int kWaves = kPlanScanThreads / 64;
    __shared__ int64_t wsum[5][16];
    __shared__ int32_t cls_all[kMaxFftLog2 + 1], cls_next[kMaxFftLog2 + 1];
    constexpr int kSums = 8 + 8;                     // all blocks: seven sums, grid rows, then statistics
    __shared__ int64_t red[kSums + 7][kWaves];
    if (sum->overflow) return;
    const int32_t n_l = sum->n_l, n_a = sum->n_a;
    const int32_t n_la = n_l > n_a ? n_l : n_a;
    constexpr int32_t kPass = kPlanScanThreads * kVpt;
    const int32_t run = ((n_la + kPlanScanBlocks - 1) / kPlanScanBlocks + kPass - 1) / kPass * kPass;
    const int32_t first = (int32_t)blockIdx.x * run;
    if (first >= n_la && first > 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nch = P.nch;
    if (tid <= kMaxFftLog2) cls_all[tid] = cls_next[tid] = 0;
    __syncthreads();
    // all[]: items and slots of the local blocks; items, grid slots, panels of
    // points and of frequencies and assembly units of the asymptotic ones;
    // blocks whose rows read the grids; then rows and columns of either kind, direct-sum cells, FFT
    // points, direct-sum row cells, FFT rows.  before[]: the first seven over the
    // blocks before the run.
    int64_t all[kSums], before[7];
    #pragma unroll
    for (int q = 0; q < kSums; ++q) all[q] = 0;
    #pragma unroll
    for (int q = 0; q < 7; ++q) before[q] = 0;
    #pragma unroll 2
    for (int32_t i = tid; i < n_l; i += kPlanScanThreads) {
        const LScan L = A.lscan[i];
        all[0] += L.items; all[1] += L.slots; all[8] += L.rows; all[9] += L.cols;
        if (i < first) { before[0] += L.items; before[1] += L.slots; }
    }
    #pragma unroll 2
    for (int32_t i = tid; i < n_a; i += kPlanScanThreads) {
        const AScan B = A.ascan[i];
        all[2] += B.items; all[3] += B.slots; all[4] += B.pc; all[5] += B.pr; all[6] += B.units; all[7] += B.gridrows;
        all[10] += B.rows; all[11] += B.cols;
        if (B.fft > 0) { all[13] += B.slots; all[15] += B.rows; }
        else if (B.fft == 0) { all[12] += B.slots; all[14] += (int64_t)B.rows * B.slots; }
        if (i < first) { before[2] += B.items; before[3] += B.slots; before[4] += B.pc; before[5] += B.pr; before[6] += B.units; }
        if (B.fft > 0) {
            atomicAdd(&cls_all[B.fft], 1);
            if (i < first) atomicAdd(&cls_next[B.fft], 1);
        }
    }
    #pragma unroll
    for (int q = 0; q < kSums; ++q) {
        int64_t x = all[q];
        for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
        if (lane == 0) red[q][wave] = x;
    }
    if (first > 0) {
        #pragma unroll
        for (int q = 0; q < 7; ++q) {
            int64_t x = before[q];
            for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
            if (lane == 0) red[kSums + q][wave] = x;
        }
    }
    __syncthreads();
    auto total = [&](int q) {
        int64_t x = 0;
        for (int v = 0; v < kWaves; ++v) x += red[q][v];
        return x;
    };
    if (blockIdx.x == 0) {
        if (tid <= kMaxFftLog2) {
            int32_t f = 0;
            for (int c = 0; c < tid; ++c) f += cls_all[c];
            sum->fft_first[tid] = f;
            sum->fft_count[tid] = cls_all[tid];
            if (tid == kMaxFftLog2) sum->n_fft = f + cls_all[tid];
        }
        if (tid == 64) {
            const int64_t l_items = total(0), l_slots = total(1), a_items = total(2), grid = total(3), n_cp = total(4),
                          n_rp = total(5);
            A.gslot[n_a] = grid;
            A.gunit[n_a] = sum->grid_units = total(6);
            sum->l_row = total(8); sum->l_col = total(9); sum->a_row = total(10); sum->a_col = total(11);
            sum->dft_cells = total(12); sum->fft_points = total(13);
            sum->dft_row_cells = total(14); sum->fft_rows = total(15);
            sum->n_litems = (int32_t)l_items; sum->n_aitems = (int32_t)a_items;
            sum->max_nch = nch;
            sum->n_gridrows = (int32_t)total(7);
            sum->grid_cells = grid;
            sum->n_cpan = (int32_t)n_cp; sum->n_rpan = (int32_t)n_rp; sum->n_lslots = (int32_t)l_slots;
            // (read by the kernels that follow, not by the other workgroups of this one)
            if (l_items > A.litem_cap || a_items > A.aitem_cap || n_cp > A.pan_cap || n_rp > A.pan_cap ||
                l_slots > A.lslot_cap)
                sum->scan_overflow = 1;
        }
    }
    int64_t l_items = 0, l_slots = 0, a_items = 0, grid = 0, cpan = 0, rpan = 0, unit = 0;
    if (first > 0) {
        l_items = total(kSums); l_slots = total(kSums + 1); a_items = total(kSums + 2);
        grid = total(kSums + 3); cpan = total(kSums + 4); rpan = total(kSums + 5);
        unit = total(kSums + 6);
    }
    const int32_t end = first + run < n_la ? first + run : n_la;
    for (int32_t c0 = first; c0 < end; c0 += kPass) {
        const int32_t i0 = c0 + tid * kVpt;
        int64_t v[kVpt][5];                          // items and slots; items; grid slots; panels (2^32 apart); units
        int32_t fft[kVpt];
        #pragma unroll
        for (int k = 0; k < kVpt; ++k) {
            v[k][0] = v[k][1] = v[k][2] = v[k][3] = v[k][4] = 0;
            fft[k] = 0;
            if (i0 + k < n_l) {
                const LScan L = A.lscan[i0 + k];
                v[k][0] = L.items + ((int64_t)L.slots << 32);
            }
            if (i0 + k < n_a) {
                const AScan B = A.ascan[i0 + k];
                v[k][1] = B.items;
                v[k][2] = B.slots;
                v[k][3] = B.pc + ((int64_t)B.pr << 32);
                v[k][4] = B.units;
                fft[k] = B.fft;
            }
        }
        int64_t tot[5];
        block_scan_vpt<5, kVpt, kWaves>(v, tot, wsum);
        #pragma unroll
        for (int k = 0; k < kVpt; ++k) {
            const int32_t i = i0 + k;
            if (i < n_l) {
                A.lb[i].item0 = (int32_t)(l_items + (v[k][0] & 0xffffffff));
                A.lb[i].slot0 = (int32_t)(l_slots + (v[k][0] >> 32));
            }
            if (i < n_a) {
                A.ab[i].item0 = (int32_t)(a_items + v[k][1]);
                A.ab[i].grid_off = (grid + v[k][2]) * nch;
                A.gslot[i] = grid + v[k][2];
                A.gunit[i] = unit + v[k][4];
                A.ab[i].cpan0 = (int32_t)(cpan + (v[k][3] & 0xffffffff));
                A.ab[i].rpan0 = (int32_t)(rpan + (v[k][3] >> 32));
                if (fft[k] > 0) {
                    // FFT-path blocks grouped by size class (order inside a
                    // class is immaterial)
                    int32_t slot = atomicAdd(&cls_next[fft[k]], 1);
                    for (int c = 0; c < fft[k]; ++c) slot += cls_all[c];
                    A.fft_list[slot] = i;
                    A.ab[i].fft_slot = slot;
                }
            }
        }
        l_items += tot[0] & 0xffffffff;
        l_slots += tot[0] >> 32;
        a_items += tot[1];
        grid += tot[2];
        cpan += tot[3] & 0xffffffff;
        rpan += tot[3] >> 32;
        unit += tot[4];
    }
}

// ---------------------------------------------------------------------------
// Work items (grid-stride over all items: local, asymptotic, the rank blocks'
// panels of points and of frequencies, the slots of the local blocks' rows,
// the direct blocks).
// An item is a chunk of one block's columns; a spread item also carries the
// subgrid of cells its points can reach (one cell of margin each side), an
// item of a rank block the panels its points lie in.
// ---------------------------------------------------------------------------
// Last block b with first_of(b) <= i (first_of nondecreasing, first_of(0) <= i),
// for the 64 consecutive values i0 .. i0 + 63 of a wave (lane l: i = i0 + l;
// every lane calls it).  The wave finds the block of i0 by 64-ary steps; when
// the next 63 blocks reach past the wave's last value each lane then searches
// their first values, loaded once, through lane reads.
template <class F>
__device__ __forceinline__ int32_t block_of(int32_t n, int32_t i0, F&& first_of)
{
    const int lane = threadIdx.x & 63;
    const int32_t i = i0 + lane;
    int32_t lo = 0, hi = n;                          // the block of i0 lies in [lo, hi)
    while (hi - lo > 1) {
        const int32_t step = (hi - lo + 63) / 64;
        const int32_t p = lo + (lane + 1) * step;    // first_of(p) <= i0 for the first c lanes
        const int c = __popcll(__ballot(p < hi && first_of(p) <= i0));
        lo += c * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    const int32_t b = lo + 1 + lane;
    const int32_t f = b < n ? first_of(b) : INT32_MAX;
    if (__shfl(f, 63) > i0 + 63) {
        int c = 0;                                   // blocks after lo that start at or before i
        #pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            if (__shfl(f, c + o - 1) <= i) c += o;
        return lo + c;
    }
    int32_t a = lo, e = n - 1;
    while (a < e) {
        const int32_t mid = (a + e + 1) >> 1;
        if (first_of(mid) <= i) a = mid; else e = mid - 1;
    }
    return a;
}

// Panel of the rank block's point r: the one with edge(q) <= r - C < edge(q + 1),
// the outer panels open-ended.
__device__ __forceinline__ int32_t rank_panel_of(const ABlock& B, double r)
{
    if (B.pc == 1) return 0;
    const double b = r - B.C;
    int32_t q = (int32_t)((b - rank_edge(B, 0)) / (2.0 * B.cw));
    q = q < 0 ? 0 : q >= B.pc ? B.pc - 1 : q;
    while (q > 0 && b < rank_edge(B, q)) --q;
    while (q + 1 < B.pc && b >= rank_edge(B, q + 1)) ++q;
    return q;
}

// First column of panel q of a rank block (q = pc: one past its last).
__device__ __forceinline__ int32_t rank_panel_col(const ABlock& B, const double* __restrict__ rs, int32_t q)
{
    if (q <= 0) return B.k0;
    if (q >= B.pc) return B.k1 + 1;
    const double e = rank_edge(B, q);
    int32_t lo = B.k0, hi = B.k1 + 1;
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (rs[mid] - B.C < e) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Appends the calling lanes with `take` set to a list whose length is *count:
// one atomic per wave.  The order of a list depends on timing; nothing that is
// computed from it does.
__device__ __forceinline__ int32_t wave_append(bool take, int32_t* count)
{
    const uint64_t m = __ballot(take);
    if (m == 0) return 0;
    const int lane = threadIdx.x & 63;
    const int lead = __builtin_ctzll(m);
    int32_t base = 0;
    if (lane == lead) base = atomicAdd(count, (int32_t)__popcll(m));
    base = __shfl(base, lead);
    return base + (int32_t)__popcll(m & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
}

__device__ __forceinline__ void items(const PlanArgs& a)
{
    const PlanDev& P = a.P;
    const Arena& A = a.A;
    Summary* __restrict__ sum = a.sum;
    int32_t* __restrict__ a_cells = a.a_cells;
    if (sum->overflow || sum->scan_overflow) return;
    const int32_t n_l = sum->n_l, n_a = sum->n_a, n_d = sum->n_d;
    const int32_t n_li = sum->n_litems, n_ai = sum->n_aitems, n_cp = sum->n_cpan, n_rp = sum->n_rpan, n_ls = sum->n_lslots;
    const int w = P.w;
    // the six kinds of work, each rounded up to whole waves
    const int32_t w_li = (n_li + 63) & ~63, w_ai = (n_ai + 63) & ~63, w_cp = (n_cp + 63) & ~63, w_rp = (n_rp + 63) & ~63;
    const int32_t w_ls = (n_ls + 63) & ~63, w_d = (n_d + 63) & ~63;
    const int32_t total = w_li + w_ai + w_cp + w_rp + w_ls + w_d;
    for (int32_t j0 = blockIdx.x * blockDim.x + (threadIdx.x & ~63); j0 < total; j0 += gridDim.x * blockDim.x) {
        const int lane = threadIdx.x & 63;
        bool ritem = false;                           // an item of a rank block
        bool tone = false, tmany = false;             // a panel of frequencies of a block of one wave / of another
        bool wmany = false;                           // a panel of points of another
        bool fpan = false;                            // the first of a group of panels of an FFT-path block
        bool lwork = false;                           // the first slot of a wave of local rows
        bool drank = false, dentry = false;           // a direct block through expansions / entry by entry
        int32_t id = 0;
        LocalWork W{};
        RankItem R{};
        Panel T{};
        if (j0 < w_li) {
            const int32_t i = j0 + lane;
            const int32_t lo = block_of(n_l, j0, [&](int32_t b) { return A.lb[b].item0; });
            if (i < n_li) {
                const LBlock L = A.lb[lo];
                int32_t it = i - L.item0;
                int32_t ka = L.k0 + it * local_chunk(P.n);
                int32_t kb = ka + local_chunk(P.n);
                if (kb > L.k1 + 1) kb = L.k1 + 1;
                Item I;
                I.blk = lo; I.ka = ka; I.kb = kb; I.sub_lo = 0; I.sub_n = 0; I.dense = 0; I.off = 0;
                A.litems[i] = I;
            }
        } else if (j0 < w_li + w_ai) {
            const int32_t i0 = j0 - w_li, ia = i0 + lane;
            const int32_t lo = block_of(n_a, i0, [&](int32_t b) { return A.ab[b].item0; });
            if (ia < n_ai) {
                const ABlock B = A.ab[lo];
                int32_t it = ia - B.item0;
                int32_t ka = B.k0 + it * P.spread_chunk;
                int32_t kb = ka + P.spread_chunk - 1;
                if (kb > B.k1) kb = B.k1;
                int32_t lhi = B.llo + B.N1 - 1;
                const double ra = P.rs[ka], rb = P.rs[kb];
                double u0 = (ra - B.C) / B.h, u1 = (rb - B.C) / B.h;
                int32_t s0 = iceil(u0 - 0.5 * w) - 1;
                int32_t s1 = iceil(u1 - 0.5 * w) + w;
                if (s0 < B.llo) s0 = B.llo;
                if (s1 > lhi) s1 = lhi;
                Item I;
                I.blk = lo; I.ka = ka; I.kb = kb + 1; I.sub_lo = s0; I.sub_n = s1 - s0 + 1; I.off = 0;
                // first cells of the points lie in s0 .. s1 - w + 1 (one cell of
                // margin each side for rounding): dense if at most kSpreadAnchors,
                // medium if at most kSpreadAnchorsMed
                const int32_t anchors = I.sub_n - w + 1;
                I.dense = !P.mfma ? 0
                        : anchors <= kSpreadAnchors ? 1
                        : (anchors <= kSpreadAnchorsMed && P.nch <= kMfmaMedMaxChannels) ? 2 : 0;
                int32_t cells = I.sub_n;
                if (B.K > 0) {
                    ritem = true;
                    R.blk = lo; R.slot = ia + B.cpan0; R.ka = ka; R.kb = kb + 1;
                    R.q0 = rank_panel_of(B, ra);
                    R.nq = rank_panel_of(B, rb) - R.q0 + 1;
                    cells = 0;
                }
                A.aitems[ia] = I;
                // cells, the item's kind and whether its block is a rank block
                a_cells[ia] = cells | (I.dense << 28) | (B.K > 0 ? (1 << 30) : 0);
            }
        } else if (j0 < w_li + w_ai + w_cp) {
            const int32_t i0 = j0 - w_li - w_ai, ip = i0 + lane;
            const int32_t lo = block_of(n_a, i0, [&](int32_t b) { return A.ab[b].cpan0; });
            if (ip < n_cp) {
                const ABlock B = A.ab[lo];
                T.blk = lo; T.q = ip - B.cpan0;
                T.ka = rank_panel_col(B, P.rs, T.q);
                T.kb = rank_panel_col(B, P.rs, T.q + 1);
                A.cpans[ip] = T;
                wmany = !rank_one_wave(B);
            }
        } else if (j0 >= total - w_d) {
            id = j0 - (total - w_d) + lane;
            if (id < n_d) {
                drank = A.db[id].K > 0;
                dentry = !drank;
            }
        } else if (j0 >= w_li + w_ai + w_cp + w_rp) {
            const int32_t i0 = j0 - w_li - w_ai - w_cp - w_rp, is = i0 + lane;
            const int32_t lo = block_of(n_l, i0, [&](int32_t b) { return A.lb[b].slot0; });
            if (is < n_ls) {
                W.blk = lo;
                W.q = is - A.lb[lo].slot0;
                lwork = W.q % local_wave_slots(A.lb[lo].K) == 0;
            }
        } else {
            const int32_t i0 = j0 - w_li - w_ai - w_cp, ip = i0 + lane;
            const int32_t lo = block_of(n_a, i0, [&](int32_t b) { return A.ab[b].rpan0; });
            if (ip < n_rp) {
                const ABlock B = A.ab[lo];
                T.blk = lo; T.q = ip - B.rpan0;
                fpan = B.K == 0 && T.q % kFftPanels == 0;
                tone = B.K > 0 && rank_one_wave(B);
                tmany = B.K > 0 && !tone;
            }
        }
        const bool small = ritem && R.kb - R.ka <= kRankWaveCols && R.nq <= kRankWavePanels;
        const int32_t p0 = wave_append(ritem && !small, &sum->n_ritems), p4 = wave_append(small, &sum->n_rsmall);
        if (ritem) A.rlist[small ? A.aitem_cap - 1 - p4 : p0] = R;
        const int32_t p3 = wave_append(wmany, &sum->n_wmulti);
        if (wmany) A.wlist[p3] = T;
        const int32_t p6 = wave_append(dentry, &sum->n_dentry), p7 = wave_append(drank, &sum->n_drank);
        if (dentry) A.dlist[p6] = id;
        if (drank) A.dlist[n_d - 1 - p7] = id;
        const int32_t p5 = wave_append(lwork, &sum->n_lwork);
        if (lwork) A.lwork[p5] = W;
        const int32_t p8 = wave_append(fpan, &sum->n_fpan);
        if (fpan) A.flist[p8] = T;
        const int32_t p1 = wave_append(tone, &sum->n_tsingle);
        if (tone) A.tlist[p1] = T;
        const int32_t p2 = wave_append(tmany, &sum->n_tmulti);
        if (tmany) A.tlist[A.pan_cap - 1 - p2] = T;
    }
}

// Partial-subgrid offsets of the asymptotic items, and the spreading order:
// dense items at alist[0 ..), medium ones after them, and the others at
// alist[n_ai - 1], alist[n_ai - 2], ..., each list in item order (one
// workgroup).  Items of rank blocks are not spread and in none of them.
__device__ __forceinline__ void item_scan(const PlanArgs& a)
{
    const PlanDev& P = a.P;
    const Arena& A = a.A;
    Summary* __restrict__ sum = a.sum;
    const int32_t* __restrict__ a_cells = a.a_cells;
    __shared__ int64_t wsum[2][16];
    __shared__ int32_t n_dense_total, n_dense_all;
    if (sum->overflow || sum->scan_overflow) return;
    const int32_t n_ai = sum->n_aitems;
    const int nch = P.nch;
    constexpr int kVpt = 8;                          // items per thread per pass (2048 per pass)
    // the dense items' total first: the medium ones follow them in the list
    {
        int32_t nd = 0, all = 0;
        #pragma unroll 8
        for (int32_t i = threadIdx.x; i < n_ai; i += kPlanScanThreads) {
            const int32_t c = a_cells[i];
            const int kind = (c >> 28) & 3;
            all += kind != 0 ? 1 : 0;
            nd += (kind == 1 && !(c >> 30)) ? 1 : 0;
        }
        for (int o = 32; o >= 1; o >>= 1) { nd += __shfl_xor(nd, o); all += __shfl_xor(all, o); }
        if (threadIdx.x == 0) { n_dense_total = 0; n_dense_all = 0; }
        __syncthreads();
        if ((threadIdx.x & 63) == 0) { atomicAdd(&n_dense_total, nd); atomicAdd(&n_dense_all, all); }
        __syncthreads();
    }
    const int64_t nd_total = n_dense_total;
    int64_t run = 0, run_dense = 0, run_med = 0, run_rank = 0;
    for (int32_t c0 = 0; c0 < n_ai; c0 += kPlanScanThreads * kVpt) {
        const int32_t i0 = c0 + threadIdx.x * kVpt;
        int64_t v[kVpt][2];                          // cells; a pass's dense, medium and rank items, 16 bits each
        int cls[kVpt];                               // 1 dense, 2 medium, 0 vector, 3 an item of a rank block
        static_assert(kPlanScanThreads * kVpt < (1 << 16), "counts of a pass");
        #pragma unroll
        for (int k = 0; k < kVpt; ++k) {
            const int32_t c = i0 + k < n_ai ? a_cells[i0 + k] : (1 << 30);
            v[k][0] = c & ((1 << 28) - 1);
            cls[k] = (c >> 30) ? 3 : (c >> 28) & 3;
            v[k][1] = cls[k] ? int64_t(1) << (16 * (cls[k] - 1)) : 0;
        }
        int64_t tot[2];
        block_scan_vpt<2, kVpt, kPlanScanThreads / 64>(v, tot, wsum);
        #pragma unroll
        for (int k = 0; k < kVpt; ++k) {
            const int32_t i = i0 + k;
            if (i < n_ai && cls[k] != 3) {
                A.aitems[i].off = (run + v[k][0]) * nch;
                // dense from the front, then medium, the others from the back
                const int64_t nd_before = run_dense + (v[k][1] & 0xffff), nm_before = run_med + (v[k][1] >> 16 & 0xffff);
                const int64_t pos = cls[k] == 1 ? nd_before
                                  : cls[k] == 2 ? nd_total + nm_before
                                                : n_ai - 1 - (i - nd_before - nm_before - (run_rank + (v[k][1] >> 32)));
                A.alist[pos] = i;
            }
        }
        run += tot[0];
        run_dense += tot[1] & 0xffff;
        run_med += tot[1] >> 16 & 0xffff;
        run_rank += tot[1] >> 32;
    }
    if (threadIdx.x == 0) {
        // the last pass counted its unused places as items of rank blocks
        const int64_t pass = kPlanScanThreads * kVpt, unused = (n_ai + pass - 1) / pass * pass - n_ai;
        sum->part_cells = run;
        sum->n_adense = (int32_t)run_dense;
        sum->n_amed = (int32_t)run_med;
        sum->n_aspread = (int32_t)(n_ai - (run_rank - unused));
        sum->n_dense_info = n_dense_all;
    }
}

// ---------------------------------------------------------------------------
// The planning kernels: for one partition, its arguments passed by value; for
// several (k_*_many), read from device memory through the constant address
// space, partition blockIdx.y.
// ---------------------------------------------------------------------------
typedef const __attribute__((address_space(4))) PlanArgs ConstPlanArgs;
__device__ __forceinline__ const PlanArgs& args_of(const PlanArgs* args)
{
    return *(const PlanArgs*)((ConstPlanArgs*)args + blockIdx.y);
}

#define NUHT_PLANNING_KERNEL(name, ...)                                                      \
    __global__ __VA_ARGS__ void k_##name(PlanArgs a) { name(a); }                            \
    __global__ __VA_ARGS__ void k_##name##_many(const PlanArgs* args) { name(args_of(args)); }

NUHT_PLANNING_KERNEL(staircases, __launch_bounds__(256))
NUHT_PLANNING_KERNEL(subdivide, __launch_bounds__(kSubThreads))
NUHT_PLANNING_KERNEL(block_params, __launch_bounds__(128))
NUHT_PLANNING_KERNEL(plan_scan, __launch_bounds__(kPlanScanThreads) __attribute__((amdgpu_waves_per_eu(4))))
NUHT_PLANNING_KERNEL(items, __launch_bounds__(128))
NUHT_PLANNING_KERNEL(item_scan, __launch_bounds__(kPlanScanThreads) __attribute__((amdgpu_waves_per_eu(4))))

#undef NUHT_PLANNING_KERNEL

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

static SortSegs sort_segs(int32_t na, int32_t nb)
{
    SortSegs S;
    S.off[0] = 0; S.off[1] = na; S.off[2] = na + nb;
    const int ta = cdiv(na, kSortTile), tb = cdiv(nb, kSortTile);
    S.tile0[0] = 0; S.tile0[1] = ta; S.tile0[2] = ta + tb;
    S.hoff[0] = 0; S.hoff[1] = 256 * ta; S.hoff[2] = 256 * (ta + tb);
    return S;
}

// The 1024-slot splitter sort is taken as far as its slots go: its launches
// take 112 us for 2 x 1e6 keys, 128 with the gaps between them; the LSD sort's
// 24 take 276 and 397.  Beyond 2^20 keys a bucket would outgrow the LDS.
constexpr int32_t kSsLargeMax = 1 << 20;
static_assert(kSsLargeMax <= SsCfg<1024>::kMaxLen, "splitter sort capacity");

enum class SortPath { small, splitter64, splitter1024, lsd };

static SortPath sort_path(int32_t na, int32_t nb)
{
    const int32_t mx = na > nb ? na : nb;
    if (mx <= kSsCap) return SortPath::small;
    if (mx <= SsCfg<64>::kMaxLen) return SortPath::splitter64;
    if (mx <= kSsLargeMax) return SortPath::splitter1024;
    return SortPath::lsd;
}

static SortSegs ss_segs(int32_t na, int32_t nb)
{
    SortSegs S;
    S.off[0] = 0; S.off[1] = na; S.off[2] = na + nb;
    const int ta = cdiv(na, kSsTile), tb = cdiv(nb, kSsTile);
    S.tile0[0] = 0; S.tile0[1] = ta; S.tile0[2] = ta + tb;
    S.hoff[0] = S.hoff[1] = S.hoff[2] = 0;
    return S;
}

template <int NB>
static hipError_t launch_splitter_sort(const double* r, int32_t na, const double* w, int32_t nb, uint64_t* k0,
                                       int32_t* v0, uint64_t* k1, int32_t* v1, int32_t* hist, int32_t* errs,
                                       hipStream_t s)
{
    using C = SsCfg<NB>;
    const SortSegs S = ss_segs(na, nb);
    const int tiles = S.tile0[2];
    uint64_t* spl = (uint64_t*)hist;
    int32_t* nspl = hist + C::kNsplOff;
    int32_t* bstart = hist + C::kStartOff;
    int32_t* btot = hist + C::kTotOff;
    int32_t* cnt = hist + C::kCntOff;
    // k0 holds the sample's keys until the last kernel writes it
    if (NB > 64) hipLaunchKernelGGL(k_ss_gather, dim3(C::kSample / 256, 2), dim3(256), 0, s, r, w, S, k0);
    hipLaunchKernelGGL(k_ss_sample<NB>, dim3(2), dim3(1024), 0, s, r, w, k0, S, spl, nspl);
    hipLaunchKernelGGL(k_ss_count<NB>, dim3(tiles), dim3(kSsThreads), 0, s, r, w, S, spl, nspl, cnt, errs);
    hipLaunchKernelGGL(k_ss_scan<NB>, dim3(2 * NB / 64), dim3(64 * kSsScanWaves), 0, s, S, cnt, btot);
    hipLaunchKernelGGL(k_ss_scatter<NB>, dim3(tiles), dim3(kSsThreads), 0, s, r, w, S, spl, nspl, cnt, btot, bstart,
                       k1, v1);
    hipLaunchKernelGGL(k_ss_local<NB>, dim3(2 * NB), dim3(kSsLocalThreads), 0, s, S, nspl, bstart, btot, k1, v1,
                       k0, v0);
    return hipGetLastError();
}

hipError_t launch_keys_and_sort(const double* r, int32_t na, const double* w, int32_t nb, uint64_t* k0, int32_t* v0,
                                uint64_t* k1, int32_t* v1, int32_t* hist, int32_t* errs, hipStream_t s)
{
    const SortPath path = sort_path(na, nb);
    if (path == SortPath::small) {
        if (na + nb == 0) return hipSuccess;
        const SortSegs S = ss_segs(na, nb);
        hipLaunchKernelGGL(k_sort_small, dim3(2), dim3(kSsLocalThreads), 0, s, r, w, S, k0, v0, errs);
        return hipGetLastError();
    }
    if (path == SortPath::splitter64) return launch_splitter_sort<64>(r, na, w, nb, k0, v0, k1, v1, hist, errs, s);
    if (path == SortPath::splitter1024)
        return launch_splitter_sort<1024>(r, na, w, nb, k0, v0, k1, v1, hist, errs, s);
    const SortSegs S = sort_segs(na, nb);
    const int tiles = S.tile0[2];
    if (tiles == 0) return hipSuccess;
    // the per-tile counts, then the 2 x 256 digit totals
    int32_t* dtot = hist + S.hoff[2];
    hipLaunchKernelGGL(k_make_keys, dim3(tiles), dim3(kSortThreads), 0, s, r, w, S, k0, v0, hist, errs);
    uint64_t* kin = k0; int32_t* vin = v0; uint64_t* kout = k1; int32_t* vout = v1;
    for (int pass = 0; pass < 8; ++pass) {
        if (pass > 0)   // the first pass's counts come with the keys
            hipLaunchKernelGGL(k_sort_hist, dim3(tiles), dim3(kSortThreads), 0, s, kin, S, 8 * pass, hist);
        hipLaunchKernelGGL(k_sort_scan, dim3(2 * 256 / 4), dim3(256), 0, s, hist, dtot, S);
        hipLaunchKernelGGL(k_sort_scatter, dim3(tiles), dim3(kSortThreads), 0, s, kin, vin, kout, vout, S, 8 * pass,
                           hist, dtot);
        uint64_t* tk = kin; kin = kout; kout = tk;
        int32_t* tv = vin; vin = vout; vout = tv;
    }
    return hipGetLastError();   // eight passes: the result is back in (k0, v0)
}

hipError_t launch_reduce_errs(const int32_t* errs, int32_t n, int32_t* flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_reduce_errs, dim3(1), dim3(256), 0, s, errs, n, flag);
    return hipGetLastError();
}

int sort_tiles(int32_t na, int32_t nb)
{
    switch (sort_path(na, nb)) {
        case SortPath::small: return 2;
        case SortPath::splitter64:
        case SortPath::splitter1024: return cdiv(na, kSsTile) + cdiv(nb, kSsTile);
        default: return cdiv(na, kSortTile) + cdiv(nb, kSortTile);
    }
}

int sort_hist_len(int32_t na, int32_t nb)
{
    switch (sort_path(na, nb)) {
        case SortPath::small: return 1;
        case SortPath::splitter64: return SsCfg<64>::kCntOff + 64 * sort_tiles(na, nb);
        case SortPath::splitter1024: return SsCfg<1024>::kCntOff + 1024 * sort_tiles(na, nb);
        default: return 256 * sort_tiles(na, nb) + 2 * 256;
    }
}

constexpr int kParamBlocks = 1536, kItemBlocks = 512;

hipError_t launch_planning(const PlanArgs& a, hipStream_t s)
{
    const int32_t n = a.P.n, m = a.P.m;
    hipLaunchKernelGGL(k_staircases, dim3(cdiv(m, 256) + cdiv(n, 256)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_subdivide, dim3(1), dim3(kSubThreads), 0, s, a);
    if (a.A.sub) {
        hipLaunchKernelGGL(k_subtrees, dim3(kSubTrees), dim3(kSubThreads), 0, s, a);
        hipLaunchKernelGGL(k_subtree_blocks, dim3(kSubTrees), dim3(kSubThreads), 0, s, a);
    }
    hipLaunchKernelGGL(k_block_params, dim3(kParamBlocks), dim3(128), 0, s, a);
    hipLaunchKernelGGL(k_plan_scan, dim3(kPlanScanBlocks), dim3(kPlanScanThreads), 0, s, a);
    hipLaunchKernelGGL(k_items, dim3(kItemBlocks), dim3(128), 0, s, a);
    hipLaunchKernelGGL(k_item_scan, dim3(1), dim3(kPlanScanThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_planning_many(const PlanArgs* args_dev, int count, int64_t nm, hipStream_t s)
{
    // cdiv(m) + cdiv(n) workgroups of staircases, at most cdiv(n + m) + 1;
    // their kernel ignores workgroups past a partition's queries
    hipLaunchKernelGGL(k_staircases_many, dim3(cdiv(nm, 256) + 1, count), dim3(256), 0, s, args_dev);
    hipLaunchKernelGGL(k_subdivide_many, dim3(1, count), dim3(kSubThreads), 0, s, args_dev);
    hipLaunchKernelGGL(k_block_params_many, dim3(kParamBlocks, count), dim3(128), 0, s, args_dev);
    hipLaunchKernelGGL(k_plan_scan_many, dim3(kPlanScanBlocks, count), dim3(kPlanScanThreads), 0, s, args_dev);
    hipLaunchKernelGGL(k_items_many, dim3(kItemBlocks, count), dim3(128), 0, s, args_dev);
    hipLaunchKernelGGL(k_item_scan_many, dim3(1, count), dim3(kPlanScanThreads), 0, s, args_dev);
    return hipGetLastError();
}

}  // namespace nuht
