// nuht_internal.h -- data structures shared by the host code and the HIP kernels.
//
// Index conventions follow the paper (Sec. 4.1): rows j index the frequencies
// omega (sorted ascending), columns k index the points r (sorted ascending).
// A block is the inclusive index rectangle rows j0..j1, columns k0..k1.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nuht {

constexpr int kMaxChannels = 40;       // 2M with M <= 20 (eq. num-asy-terms caps M at 20)
constexpr int kMaxFftLog2 = 24;        // largest FFT of an asymptotic block: 2^24 = 4096^2 points (two passes)
// Columns per local-moment work item (one wave) of a transform of n points.
// A wave's points are a serial chain, so items are short enough for the waves
// to cover the chip at every n, and long enough that adding up the items of
// the largest block stays cheap.  Against items of 4096 columns: k_lmom at n =
// 5229, order 18: 10 us (93); at 1e6, order 0, 31 (48); 40 transforms of 1e3
// to 1e5 points in one batch 113 (343); the sums 4 to 9 us (5 to 8) through
// the split of lmom_reduce_body.
inline __host__ __device__ int32_t local_chunk(int32_t n) { return n <= (1 << 17) ? 256 : n <= (1 << 19) ? 512 : 1024; }
constexpr int kSpreadChunk = 1024;     // default points per spreading work item (a plan option)
// Default direct-block threshold of Alg. 1 for an n x m transform.  The
// paper leaves min_size to numerical experiments (its example: 1024).  The rule
// takes the power of two at or below n m / 256, within [1024, 8192]; it was
// found when every direct block was applied entry by entry, and most are
// applied through expansions now.  An execution's time over that of the best of
// 256 .. 131072 (geometric mean over orders 0, 10, 40 and 3/2, tolerances 1e-6
// to 1e-12 and three layouts), with the rule's threshold and the best fixed one:
// 500 x 500 1.07 and 1.04 (256), 1000 x 1000 1.02, 2000 x 2000 1.11 and 1.02
// (2048), 5000 x 5000 1.04 and 1.02 (16384), 1e5 x 1e5 1.09, 3e5 x 3e5 1.13 and
// 1.11 (4096), 1e6 x 1e6 1.12 and 1.10 (16384); far off only where points
// outnumber frequencies many times, 30000 x 500 1.24 and 1.03 (256).
constexpr int64_t kMinSizeLo = 1024;
constexpr int64_t kMinSizeHi = 8192;
inline int64_t default_min_size(int64_t n, int64_t m) {
    const double a = (double)n * (double)m / 256.0;
    int64_t s = kMinSizeLo;
    while (s < kMinSizeHi && (double)(2 * s) <= a) s *= 2;
    return s;
}
// Workgroups per vector spreading item, of n items: an item is a chain of
// sub-chunks and of turns of its cells, so few items are shared to fill the
// chip.
inline int32_t spread_turns(int32_t n) { int32_t t = 1; while (t < 8 && 2 * t * (int64_t)n <= 1024) t *= 2; return t; }
constexpr int kMaxEsWidth = 18;        // largest ES kernel width
constexpr int kEshatTerms = 16;        // terms of the polynomial for the ES kernel's Fourier transform
constexpr int kEsDeg = 13;             // degree of the per-cell polynomial pieces of the ES kernel
constexpr int kSpreadAnchors = 6;      // first cells (anchors) of a dense matrix-core spreading item
constexpr int kSpreadAnchorsMed = 40;  // first cells of a medium one (its own launch, larger LDS cell sums)
constexpr int kMfmaMaxChannels = 32;   // channel counts whose dense items go to the matrix cores
constexpr int kMfmaMedMaxChannels = 16; // ... and whose medium items (their LDS cell sums grow with the channels)
constexpr int kMaxLevels = 4096;       // subdivision depth limit
constexpr int kHalfDeg = 20;           // degree of the half-integer local coefficients on a panel
constexpr double kHalfWidth = 4.0;     // panel width (in omega R) of those coefficients
constexpr int kJtabCoef = 16;          // coefficients per panel of the direct-block J_nu table (degree 15)
constexpr double kJtabWidth = 2.0;     // panel width (in x = omega r) of that table

// Asymptotic blocks applied through Chebyshev expansions in r and omega
// instead of type-3 transforms (rank blocks; see exec.hip).  An expansion has
// K terms, a multiple of 4 up to kRankK; the points and the frequencies of a
// block are cut into equal-width panels, at most kRankPanels of points.
constexpr int kRankK = 24;
constexpr int kRankPanels = 40;
// Neighbouring panels of an FFT-path block's frequencies expanded by one
// workgroup.
constexpr int kFftPanels = 2;
// The narrowest ES kernel at which plans have rank blocks (eps up to about
// 1e-8).  The expansions are good to max(eps / 1000, 2e-16) and the ES transforms
// to about 10^(1-w), so the two forms of a block agree to 1e-9 or better from
// this width on.  That is no limit of the expansions, which are the more exact
// form everywhere: looser plans keep the grids that they had, and so their
// results.
constexpr int kRankMinWidth = 11;
// Items of at most this many columns over at most this many panels take one
// wave, larger ones four.
constexpr int kRankWaveCols = 256;
constexpr int kRankWavePanels = 4;
// Blocks with one panel of points and at most this many items are translated
// by the wave that adds up their moments.
constexpr int kRankSingleItems = 16;
// log rho of the ellipses the expansions' length is bounded on (16 of them).
constexpr double kRankLr0 = 0.1, kRankLrStep = 0.28;
// Cosine tables of the expansion lengths K = 4, 8, .., kRankK, one after the
// other: cos(pi m (2 s + 1) / (2 K)) as [m][s], then as [s][m].
__host__ __device__ inline int rank_tab_off(int K) { const int i = K / 4 - 1; return 2 * 16 * (i * (i + 1) * (2 * i + 1) / 6); }

// A mixed block of Alg. 1 and the split chosen for it.  Rows j0..js and
// columns k0..ks are the local (upper-left) side.  A wholly local block is
// stored with (js, ks) = (j1, k1), a wholly asymptotic one with
// (js, ks) = (j0-1, k0-1).
struct Node {
    int32_t j0, j1, k0, k1;
    int32_t js, ks;
    int32_t lblk, ablk;   // local / asymptotic child block index, -1 if empty
    int32_t ur, ll;       // upper-right / lower-left child: >= 0 mixed node,
                          // <= -2 direct block (-2 - index), -1 empty
    int32_t level, pad;
};

__host__ __device__ inline int32_t encode_direct(int32_t d) { return -2 - d; }
__host__ __device__ inline int32_t decode_direct(int32_t c) { return -2 - c; }

struct LBlock {
    int32_t j0, j1, k0, k1;
    double R;             // expansion radius: r_{k1}, or z / omega_{j1} when r_{k1} = 0
    int32_t item0, nitems;
    int32_t level;
    // its rows: a Chebyshev expansion of K terms on each of pr panels of
    // frequencies (middles about D, half-width rw), or (K = 0) one value per
    // row; both from slot slot0 on, kRankK values a slot
    int32_t K, pr, slot0;
    double D, rw;
};

// Whether a grid of N1 cells is assembled by a thread a cell and channel: the
// items, w + 2 cells wider than their points, cover a cell more than three
// times on average.  (Else a thread a cell: see k_spread_reduce.)
__host__ __device__ inline bool grid_crowded(int32_t N1, int32_t nitems, int32_t w) { return (int64_t)nitems * (w + 2) > 2 * (int64_t)N1; }

// Slots of a local block's rows, and those evaluated by one wave.
__host__ __device__ inline int32_t local_slots(const LBlock& B) { return B.K > 0 ? B.pr : (B.j1 - B.j0 + kRankK) / kRankK; }
__host__ __device__ inline int32_t local_wave_slots(int32_t K) { return K > 0 ? 64 / K : 64 / kRankK; }

// A wave's slots q .. of local block blk.
struct LocalWork {
    int32_t blk, q;
};

struct ABlock {
    int32_t j0, j1, k0, k1;
    double C, D;          // centres of the point and frequency ranges
    double h;             // spread-grid spacing (a power of two)
    double r0;            // smallest point of the block (weights are normalised by it)
    double alpha;         // ES kernel half-width w h / 2
    double Khi, Klo;      // h N2 / (2 pi) as a double-double (FFT path)
    int32_t llo, N1;      // spread-grid cells llo .. llo + N1 - 1
    int32_t N2, fft;      // FFT size and 1 for the FFT path; 0 for the direct-sum path
    int64_t grid_off;     // offset of the block's grid (complex elements)
    int32_t item0, nitems;
    int64_t part_off;     // first partial-subgrid element of its items (complex)
    int32_t level, fft_slot;  // fft_slot: position in the FFT size-class list
    // rank blocks (K > 0): expansion length, panels of points and frequencies
    // with their half-widths and first panel numbers
    // (rK: terms of the rows' expansions, K in a rank block; an FFT-path block
    // (K = 0) may have them too, its transform then read at their nodes alone)
    int32_t K, pc, pr, cpan0, rpan0, rK;
    double cw, rw;
};

// A panel of a rank block's points (columns ka .. kb - 1) or frequencies
// (ka, kb unused), panel q of its block.
struct Panel {
    int32_t blk, q, ka, kb;
};

// A rank block's item: columns ka .. kb - 1 of block blk, in panels q0 .. q0 +
// nq - 1; its moments of panel q are number `slot` + q.
struct RankItem {
    int32_t blk, slot, ka, kb, q0, nq;
};

// Panels are laid out about the block's centres: left edge (q = pc: the right
// end) and middle of panel q of the points, as offsets from C, and middle of
// panel q of the frequencies, as an offset from D.  (Offsets keep the panels'
// places exact to their own size, whatever the size of r and omega.)
__host__ __device__ inline double rank_edge(const ABlock& B, int q) { return (2 * q - B.pc) * B.cw; }
__host__ __device__ inline double rank_mid(int q, int panels, double half) { return (2 * q + 1 - panels) * half; }

struct DBlock {
    int32_t j0, j1, k0, k1;
    // K > 0: applied through K-term expansions about (C, D), half-widths cw of
    // its points and rw of its frequencies; 0: entry by entry
    int32_t K, pad;
    double C, cw, D, rw;
};

// Whether one wave adds up a rank block's moments and translates them.
__host__ __device__ inline bool rank_one_wave(const ABlock& B) { return B.pc == 1 && B.nitems <= kRankSingleItems; }

// Work item of the column-side kernels: a chunk of one block's columns.
struct Item {
    int32_t blk;
    int32_t ka, kb;       // columns ka .. kb-1
    int32_t sub_lo, sub_n;  // spread items: subgrid cells sub_lo .. sub_lo + sub_n - 1
    int32_t dense;        // spread items on the matrix cores: 1 (dense) if its points' first cells
                          // lie in sub_lo .. sub_lo + kSpreadAnchors - 1, 2 (medium) if within
                          // kSpreadAnchorsMed of sub_lo; else 0 (vector spreading)
    int64_t off;          // spread items: partial-subgrid offset (complex elements)
};

// What a subdivision overflowed: a table (the counting goes on), the levels, a
// subtree's share of tables that hold the whole, or the queue of a level (the
// counts are those so far).
constexpr int32_t kOverTables = 1, kOverLevels = 2, kOverShare = 3, kOverQueue = 4;

// Written by the planning kernels, read once by the host.
struct Summary {
    int32_t n_nodes, n_l, n_a, n_d;
    int32_t levels, overflow;  // overflow: kOver*
    int32_t scan_overflow;     // of the tables of items, panels and slots
    int32_t n_litems, n_aitems;
    int32_t n_fft, max_nch;
    int32_t n_adense, n_amed;  // dense and medium spread items (the first n_adense, then n_amed, of the item list)
    int32_t n_aspread;         // spread items (the items of blocks that are not rank blocks)
    int32_t n_dense_info;      // items of all asymptotic blocks that are dense or medium by their cells
    int32_t n_ritems, n_rsmall;    // items of rank blocks: of four waves (kRankWaveCols, kRankWavePanels), of one
    int32_t n_cpan, n_rpan;    // panels of the rank blocks
    int32_t n_tsingle, n_tmulti;   // their panels of frequencies: of blocks translated by one wave, of others
    int32_t n_wmulti;              // panels of points of those others
    int32_t n_fpan;                // groups of kFftPanels panels of frequencies of FFT-path blocks
    int32_t n_gridrows;            // asymptotic blocks whose rows read the grids
    int32_t n_lslots, n_lwork;     // slots of the local blocks' rows; waves that fill them
    int32_t n_dentry, n_drank;     // direct blocks applied entry by entry, through expansions
    int32_t d_area, pad;           // largest of the former that reaches below the J_nu table
    int64_t l_row, l_col, a_row, a_col, d_ent;
    int64_t grid_cells;     // sum N1 (all asymptotic blocks)
    int64_t grid_units;     // threads that assemble the grids
    int64_t dft_cells;      // sum N1 over direct-sum-path blocks
    int64_t fft_points;     // sum N2 over FFT-path blocks
    int64_t part_cells;     // sum of item subgrid sizes
    int64_t dft_row_cells;  // sum of rows x N1 over direct-sum-path blocks
    int64_t fft_rows;       // sum of rows over FFT-path blocks
    int32_t fft_count[kMaxFftLog2 + 1];   // FFT-path blocks per log2(N2)
    int32_t fft_first[kMaxFftLog2 + 1];   // start of each size class in the FFT list
    int32_t domain_error;
    int32_t grid_error;     // an asymptotic block needs an FFT larger than 2^kMaxFftLog2
};

// FFT-path grids of at most 4096 points, every size class in one launch:
// workgroup g belongs to class c when wg0[c] <= g < wg0[c + 1], and within it
// to the FFT-list slot (g - wg0[c]) / nch of the class and channel
// (g - wg0[c]) % nch.
struct SmallFfts {
    int32_t n;                 // classes
    int32_t log2n[8], first[8];
    int32_t wg0[9];            // wg0[n]: workgroups of the launch
    int32_t max_log2n;         // largest class (its transform sets the launch's LDS)
};

// Everything the execution kernels need for one transform (passed by value to
// the kernels of a single transform; kept in a device array for a batch).
struct PlanDev {
    int32_t n, m, nu, M, L, w;       // sizes, |order| (its integer part when half), terms, local rank, ES width
    int32_t half, half_np;           // half = 1: the order is nu + 1/2; panels of the local coefficient table
    int32_t half_ns, pad0;           // leading panels holding the coefficients divided by x^nu
    int32_t nch, sign;               // channels (2M padded to a kernel instance); (-1)^nu for negative orders, else 1
    int32_t fp32;                    // FP32 spreading (weights, kernel values and channel sums in float)
    int32_t rank, rank_const;        // plan has rank blocks; the Hankel terms beyond the first vanish
    double local_xi[kRankK / 4];     // largest (half omega range) x R that 4, 8, .. terms of a local panel cover
    double direct_xi[kRankK / 4];    // the same for the two expansions of a direct block, to full precision
    double rank_ltol, rank_xi;       // log of the expansions' tolerance; largest (half r range) x (half
                                     // omega range) that kRankK terms cover
    const double* rank_tab;          // cosine tables (rank_tab_off)
    int32_t mfma;                    // dense spreading items go to the matrix cores (FP64, w <= 16, nch <= 32)
    double z, beta, eps;
    double phi_hi, phi_lo;           // -(2nu+1) pi/4 reduced to [0, 2pi), double-double
    double hank[2 * 20 + 2];         // a_p(nu), p = 0 .. 2M+1 (Hankel coefficients)
    double chan[kMaxChannels];       // channel factors (-1)^(p/2) a_p(nu) for p < 2M (odd p carry a factor i), 0 above
    double eshat[kEshatTerms];       // ES^ on [0, kappa_max]: monomial coefficients in s = 2 (kappa / kappa_max)^2 - 1
    int32_t spread_chunk;            // points per spreading work item
    int32_t spread_turns;            // workgroups that share a vector item's cells (spread_turns)
    double kappa_max, eshat_s;       // eshat_s = 2 / kappa_max^2
    const double* rs;                // sorted points (n)
    const double* ws;                // sorted frequencies (m)
    const int32_t* perm_r;           // sorted position -> caller index (points)
    const int32_t* perm_w;           // sorted position -> caller index (frequencies)
    const Node* nodes;
    const LBlock* lb;
    const ABlock* ab;
    const DBlock* db;
    const Item* litems;
    const Item* aitems;
    const int32_t* alist;            // spreading order: dense items from the front, the others from the back
    const int32_t* fft_list;         // FFT-path blocks grouped by size class
    const int64_t* gslot;            // first grid slot of each asymptotic block; gslot[n_a] = all slots
    const int64_t* gunit;            // first unit of its grid's assembly; gunit[n_a] = grid_units
    int64_t grid_units;
    const double* es_poly;           // ES kernel pieces, w x (kEsDeg + 1) monomial coefficients
    const double* half_tab;          // half-integer orders: [panel][l][degree] local coefficients
    double half_inv_h;               // 1 / panel width
    const double* jtab;              // J_nu on [jtab_x0, jtab_x0 + jtab_np kJtabWidth): per panel the
                                     // monomial coefficients in u in [-1, 1] of its Chebyshev interpolant
    double jtab_x0;
    int32_t jtab_np, pad2;
    int32_t n_nodes, n_l, n_a, n_d, n_litems, n_aitems, n_adense, n_amed;
    int32_t n_tsingle, n_tmulti, n_wmulti, n_ritems, n_rsmall, n_lwork, n_fpan, n_gridrows;
    const Panel* flist;              // panels of frequencies of FFT-path blocks, the first of each group
    const LocalWork* lwork;          // the local blocks' rows by waves
    const int32_t* dlist;            // direct blocks: entry by entry from the front, expansions from the back
    int32_t n_dentry, n_drank;
    const Panel* cpans;              // panels of the rank blocks' points
    const RankItem* rlist;           // items of rank blocks: large ones from the front, small ones from the back
    const Panel* tlist;              // panels of frequencies: blocks of one wave from the front, others from the back
    const Panel* wlist;              // panels of points of the latter blocks
    int32_t tlist_cap, rlist_cap;
    // execution buffers of the partition
    double* cs;                      // weights gathered into sorted point order (n)
    double* lpart;                   // local-moment partial sums (items x (L + 1))
    double* lmom;                    // local moments (local blocks x (L + 1))
    double* lcoef;                   // expansions or values of the local blocks' rows, by slot
    double* dcoef;                   // expansions of the direct blocks' rows, kRankK a block
    double2* rmom;                   // rank blocks: moments of (item i, panel q) at (i + q) kRankK
    double2* rwts;                   // their nodal weights per panel of points
    double2* rcoef;                  // their expansion coefficients per panel of frequencies
    double2* part;                   // spread partial subgrids
    double2* grids;                  // spread grids (direct-sum path) and FFT buffers (FFT path)
    double2* scratch;                // second buffer of the multi-pass FFTs
    double* gd;                      // per-row direct-block sums (m)
    const double2* fft_tw;           // FFT twiddles (8192 entries)
    int64_t grid_cells;              // grid slots (without the channel factor)
    SmallFfts small;                 // the FFT size classes up to 4096 points
};

// One transform's share of a batched launch: workgroups g0 .. (next g0) - 1
// of the launch work on transform t, as its workgroups 0, 1, ...
struct WorkSeg {
    int32_t t, g0;
};

}  // namespace nuht
