// Host-side launch plan for the signature-kernel sweeps: pure arithmetic, no HIP calls, so that the
// workspace query and the launches agree by construction.
//
// Geometry (paper Section 3.1/3.2): the refined grid has m = (L1-1) << lam1 by n = (L2-1) << lam2 cells.
// The sweep works on square blocks of 2^BL x 2^BL refined cells that share one entry of the increment
// Gram matrix (BL = min(lam1, lam2, 2)); the block grid has mb = (L1-1) << rs1 rows and
// nb = (L2-1) << rs2 columns, rs = lam - BL.  A strip is 64 consecutive block rows, one per lane.
#pragma once
#include <cstddef>
#include <cstdint>

namespace sk {

constexpr int kWave = 64;
constexpr int kWavesPerWG = 4;            // waves (independent pairs) per workgroup
constexpr size_t kLdsPerCU = 160 * 1024;  // gfx950: 160 KB of LDS per compute unit / workgroup
constexpr size_t kLdsPerWave = kLdsPerCU / kWavesPerWG - 1024;
constexpr int kNumCU = 256;
constexpr int kMaxBL = 2;

// Channel counts with a dedicated kernel instantiation (increments kept in registers).  (More: the wide kernels, or, where
// their scratch is too much, the sweep kernels with a run-time loop over the channels, template argument 0.)
constexpr int kTemplD[] = {2, 3, 4, 5, 6, 8, 16};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Plan {
    bool valid = false;
    bool backward = false;
    bool symmetric = false;     // Gram with Y == X: one increment buffer, one gradient accumulator
    int elem = 8;               // bytes per element of every internal buffer (sweeps run in double)
    int io_elem = 8;            // bytes per element of the caller's arrays
    int64_t nx = 0, ny = 0;     // number of x paths and y paths
    int64_t npairs = 0;         // pairs the sweep launch works through
    int64_t kcount = 0;         // entries of k / K (differs from npairs only for tri)
    int tri = 0;                // symmetric Gram matrix in solo / tile mode: only the pairs n <= m are solved
    int64_t gramM = 0;          // > 0: pair id -> (id / gramM, id % gramM); 0: pair id -> (id, id)
    int L1 = 0, L2 = 0, d = 0;
    int BL = 0, rs1 = 0, rs2 = 0;
    int r = 0, q = 0;           // coarse cells per side
    int rpad = 0, qpad = 0;
    int mb = 0, nb = 0;         // block rows / columns
    int ns = 0;                 // strips per pair
    int rowlen = 0;             // elements of one boundary row (node columns, padded)
    int DT = 0;                 // kernel template channel count (0 = runtime loop over d)
    int DP = 0;                 // channels stored per increment row (d padded to the kernel's count)
    int S = 0, nseg = 0;        // backward: macro-steps per replay segment, segments per strip
    int y_lds = 0;              // y increments (and their gradient accumulators) staged in LDS
    size_t lds_wave = 0, lds_bytes = 0, ring_off = 0;
    int grid = 0;
    int64_t nslots = 0;
    int64_t xstride = 0, ystride = 0, rows_slot = 0, ckpt_slot = 0, adj_slot = 0;
    size_t off_dxT = 0, off_dyT = 0, off_gdxT = 0, off_gdyT = 0, off_rows = 0, off_adj = 0, off_ckpt = 0;
    size_t off_kio = 0, off_gkio = 0;   // float callers: double staging of k and grad_k
    size_t off_keep_tag = 0;
    int keep_solo = 0;                  // solo backward plan with per-pair checkpoints and bottom rows
    int64_t keep_len = 0;               // doubles per kept bottom row (solo)
    size_t off_keep = 0;                // backward: what a kept forward sweep leaves besides rows and checkpoints
                                        // (lock-step: the hand-over rows; band: the kernel values)
    size_t off_err = 0;                 // one int: a bounded wait between cooperating waves ran out
    size_t total = 0;
    // cooperative mode: one workgroup per pair, its strips pipelined over nw waves
    int coop = 0, nw = 0, RB = 0, CH = 0;
    int uncompute = 0;   // backward: reverse sweep recovers forward values by inverting Eq. (1) (no replay ring)
    size_t coop_off_gdy = 0, coop_off_flags = 0, coop_off_obox = 0, coop_off_ring = 0, coop_ring_stride = 0;
    // lock-step mode: one workgroup per pair, per strip one stencil wave and one coefficient wave
    int band = 0, bd_nbands = 0;   // bands of kBandStrips strips on different compute units (sk_band.hip)
    size_t bd_off_y = 0, bd_off_gy = 0, bd_off_rings = 0, off_flags = 0;
    int nflags = 0;
    // Pairs whose inverse recurrence drifted are listed here by the reverse sweep and solved once more by the replay
    // kernel (sk_api.hip): a counter (the int behind the progress counters, cleared with them) and the pair ids.
    size_t off_badcnt = 0, off_badlist = 0;
    int ll = 0;     // lead-lag form of the sweep: 0 none, 1 the level lies inside a block, 2 above the blocks
    int tile = 0;   // one wave per pair, at most 64 x 64 cells, contractions on the matrix cores (sk_tile.hip)
    int quad = 0;   // four pairs per wave, forward Gram calls on the tile kernels' shapes (sk_quad.hip)
    int64_t nquads = 0;   // groups of four pairs of one Gram row the quad launch works through
    int64_t qd_even = 0;  // quads of a four-pair launch that are handed out in equal shares (the rest by a counter)
    int four = 0;         // four pairs per wave, backward Gram calls (sk_four.hip); lk_M: 1 = one band, 2 = several
    bool four_over_kept = false;   // faster than a one-pair reverse sweep that takes over the forward call's sweep, too
    int fv_bands = 0;     // bands of 16 lanes per pair
    int64_t fv_gx_slot = 0;
    size_t off_fvgx = 0;  // x-side sums of the strips of the pairs in work (several strips only)
    // split mode: the forward and the adjoint sweep side by side, then independent tasks (sk_split_*.hip); lock or band says how
    // the first of the two launches is laid out
    int split = 0, sp_chunks = 0, sp_tasks = 0, sp_win = 0;
    size_t sp_lds = 0, sp_off_gy = 0, sp_off_feed = 0, off_sp_arows = 0, off_sp_ackpt = 0;
    int64_t sp_ackpt_slot = 0;
    int wide = 0;         // p of every block in scratch, any channel count and any number of strips (sk_wide.hip)
    int64_t wd_slot = 0;  // doubles of that scratch per workgroup
    size_t off_wd = 0;
    int solo = 0;   // one wave per pair, a single strip of 64 * lk_M block rows (many pairs of short paths)
    int lock = 0, lk_M = 0, lk_ns = 0, lk_NT = 0, lk_padb = 0, lk_rowlen = 0;
    size_t lk_off_y = 0, lk_off_gy = 0, lk_off_cring = 0, lk_off_gp = 0, lk_off_krows = 0, lk_off_arows = 0,
           lk_off_dump = 0, lk_cring_stride = 0, lk_gp_stride = 0, lk_off_ck = 0, lk_ck_stride = 0, lk_off_gyp = 0;
};

// Lock-step mode constants: chunk lengths (macro-steps between workgroup barriers) of the forward and the
// reverse sweep, checkpoint spacing, and the lag between consecutive strips.  A value written to a hand-over
// row in one chunk is read by the neighbouring strip in a later chunk if lag >= 63 + chunk.
constexpr int kLockCH1 = 8, kLockCH2 = 4, kLockS = 8;
constexpr int kLockLag1 = 72, kLockLag2 = 68;
constexpr int kLockMaxStrips = 4;      // forward: a stencil and a coefficient wave per strip
constexpr int kLockMaxStripsBwd = 2;   // backward: plus a gradient wave per strip

// Block rows per lane the lock-step kernels are built for: two, unless the lane state would not fit the
// register file (largest blocks or most channels in the backward kernel; both together in the forward one);
// zero: no lock-step kernel for this combination.
constexpr int lock_max_rows(bool backward, int BL, int DT)
{
    if (DT == 0) return 0;
    if (backward) return (BL >= 2 && DT >= 16) ? 0 : ((BL >= 2 || DT >= 16) ? 1 : 2);
    return (BL >= 2 && DT >= 16) ? 1 : 2;
}

// Block rows per lane of the solo kernels (one wave does the stencil, the coefficients and the gradients).
constexpr int solo_max_rows(bool backward, int BL, int DT)
{
    if (DT == 0) return 0;
    if (backward) return ((BL <= 1 && DT <= 8) || DT <= 4) ? 2 : 1;
    return (BL >= 2 && DT >= 16) ? 1 : 2;
}

// Wavefronts per SIMD the solo backward kernel is built for: two, or one where the lane state of two block rows of
// 4 x 4 cells, or the sums and increments of sixteen channels, need the whole register file (accumulation registers
// included: with 256 registers the sixteen-channel kernels spill a kilobyte per lane and run four times slower).
constexpr int solo_bwd_waves_per_simd(int BL, int M, int DT)
{
    return ((BL >= 2 && M >= 2) || DT >= 16 || (DT >= 8 && (M >= 2 || BL >= 2))) ? 1 : 2;
}
// Whether a launch of the solo backward kernel puts two workgroups on a compute unit (lds: bytes per workgroup); if
// not, the kernel's one-wave build is launched, which has the whole register file.
constexpr bool solo_bwd_shares_simd(int BL, int M, int DT, size_t lds)
{
    return solo_bwd_waves_per_simd(BL, M, DT) >= 2 && 2 * lds <= kLdsPerCU;
}

// Tile mode: the increment Gram matrix of a pair as a 64 x 64 array of doubles in LDS, column stride
// kTileStride (even, not a multiple of 4: row-contiguous, skewed and transposed accesses all stay at most
// two-way bank conflicted), kTileCols columns (-1 .. 64: a zero guard column on either side).
constexpr int kTileStride = 66, kTileCols = 66;
// Quad mode: a wavefront works on four pairs that share the y path, 16 lanes with four to eight block rows each.
constexpr int kQuadPairs = 4;
// Block rows per lane the quad kernel is built for (0: none): blocks of at most 2 x 2 cells, and the increments of a
// lane's rows in at most 128 registers (eight channels: Gram 500 x 123, 99 x 76 cells, 702 us in the solo kernel, 378
// with seven rows per lane; Gram 256 x 256, 127 rows, order 1, where the kernel keeps 104 bytes per lane in scratch, 1461
// against 998 us).
constexpr int kQuadMinRows = 4;
constexpr int quad_max_rows(int BL, int DT)
{
    if (BL > 1 || DT == 0) return 0;
    if (DT == 16) return BL == 0 ? 4 : 0;
    return 8;
}
// Whether the quad kernel with eight channels and M = 5 to 8 rows per lane is faster than the solo kernel it replaces, in
// rounds of block rows as in four_gain; a wavefront alone on its SIMD goes through them in 0.5 (quad) and 0.8 (solo) of the
// time it takes where it shares it.  Solo and quad, us per call: L = 128, order 0, d = 8: 32 x 32 / 24 x 100 / 1 x 2000 /
// 2 x 1000 / 128 x 128: 35 / 62 / 55 / 51 / 266 and 50 / 50 / 91 / 56 / 164; L = 70: 25 / 44 / 41 / 37 / 178 and 25 / 25 / 45 /
// 29 / 67.  (Up to four rows, and up to six channels, the kernel is always taken.)
inline bool quad_pays(int64_t pairs, int64_t slots1, double steps1, int64_t quads, int64_t slots4, double steps4)
{
    constexpr int64_t kSimds = 4 * kNumCU;
    if (slots1 > 2 * kSimds) slots1 = 2 * kSimds;
    const double r1 = (double)((pairs + slots1 - 1) / slots1), r4 = (double)((quads + slots4 - 1) / slots4);
    return r4 * steps4 * (quads <= kSimds ? 0.5 : 0.85) < r1 * steps1 * (pairs <= kSimds ? 0.8 : 1.0);
}
// Row stride of the y copy in LDS (doubles): for an even channel count a multiple of 16 bytes that spreads the
// 16-byte reads of lanes at consecutive rows over the banks; an odd count does that by itself.
constexpr int quad_y_stride(int DT) { return DT % 2 ? DT : (DT == 6 ? 10 : DT + 2); }
// Four-pair mode (backward Gram calls, sk_four.hip): block rows per lane, doubles per lane of a checkpoint, doubles
// between the groups' rings of finished y-side sums, wavefronts per SIMD the kernel is built for (0: no such kernel).
constexpr int four_rows(int BL, int DT) { return (BL == 2 || DT >= 8) ? 2 : 4; }
constexpr int four_ckpt_values(int BL, int DT) { return (four_rows(BL, DT) << BL) + 1 + (1 << BL); }
constexpr int four_gring_stride(int DT) { return 16 * DT + 2; }
constexpr int four_occupancy(int BL, int DT)
{
    return DT < 2 || DT > 16 ? 0 : (DT >= 16 || (BL == 2 && DT >= 12)) ? 1 : 2;
}
// Channel count of the four-pair kernel for d channels (16 is far from most counts above 8).
constexpr int four_channels(int DT, int d) { return DT == 16 && d <= 12 ? 12 : DT; }
// Quads of a four-pair launch that are handed out in equal shares: all of them unless every wavefront has work for about
// 0.5 ms (`instr`: vector instructions per quad, at ten clocks each), and then half.
inline int64_t four_even_share(int64_t nquads, int64_t nwaves, int64_t instr)
{
    return nquads < 3 * nwaves || nquads / nwaves * instr < 100000 ? nquads : nquads / 2 / nwaves * nwaves;
}
// Macro-steps between its checkpoints: kFourCkpt, or twice or four times as many in a band whose largest increment product
// of a block, |dx| |dy|, is at most kFourSteady or kFourCalm (sk_four.hip has the pairs that drift; the first ones do with 8 at
// products of 0.55 and with 16 at 0.2.  Gradient errors up to either bound are those of half the spacing to a tenth).
constexpr int kFourCkpt = 4;
constexpr double kFourSteady = 0.5, kFourCalm = 0.16;
// Both are for four block rows per lane and for two of 4 x 4 cells; with two of fewer cells an error goes half as far per
// macro-step.  96 x 48 paths, gradient errors (mean, largest) and us, one-pair / bounds as above / twice those: L = 60, order 1,
// d = 8, squared length 20: 1.3e-14, 3.9e-14, 379 / 1.4e-14, 4.2e-14, 306 / 1.4e-14, 4.0e-14, 296; L = 30, order 0, d = 16,
// squared length 6: 3.6e-15, 2.2e-14, 510 / 3.3e-15, 6.1e-15, 212 / 3.2e-15, 6.2e-15, 185.
constexpr double four_calm_scale(int BL, int DT) { return BL < 2 && four_rows(BL, DT) == 2 ? 2.0 : 1.0; }
// Its drift guard (kDriftTol elsewhere).  With its short spacing and its 1 / B recovered values stay closer, so the guard can:
// L = 60, order 0, d = 5, squared length 20, largest gradient error of the pairs that pass 2.8e-12 (1.1e-11 with 1e-11).
constexpr double kFourDriftTol = 3e-12;
// Scratch that mode may take where the one-pair kernels need less: its checkpoints are many for long paths of high order
// (722 x 43 paths of 890 and 415 points, order 3: 101 GiB against 16 in the wave-per-pair kernel).
constexpr size_t kFourScratch = (size_t)4 << 30;
// Groups of four pairs of one row of the Gram matrix in a launch's sequence (tri: rows of the pairs n <= m).
inline int64_t gram_quads(bool tri, int64_t nx, int64_t ny)
{
    if (!tri) return ny * ((nx + kQuadPairs - 1) / kQuadPairs);
    const int64_t J = nx / kQuadPairs, e = nx % kQuadPairs;
    return 2 * J * (J + 1) + e * (J + 1);
}
// One side of the choice between one pair and four per wavefront: what its launch has to do, and how many wavefronts of
// it the chip holds.
struct SweepLoad {
    int64_t items;    // pairs or quads
    int64_t slots;    // wavefronts resident at once
    double steps;     // block rows a lane goes through per item
    int64_t even;     // items handed out in equal shares
};
// How much faster the four-pair kernel is.  Either launch takes rounds of `slots` items, a nearly empty round as long
// as a full one (unless the last items are handed out one by one), and a round about as long as its steps.  step: a step of
// the four-pair kernel next to one of the other; lone: where few quads leave its wavefronts alone on their SIMDs, next to
// where they share them.
// One-pair and four-pair, us per call (n x n; (n): K(X, X)):
//   L = 128, order 1, d = 3: 64 / 80 / 96 / 128: 377 / 613 / 819 / 1393 and 406 / 527 / 944 / 1156
//                            (72) / (84) / (112) / (128): 342 / 347 / 613 / 784 and 351 / 369 / 523 / 942
//   L = 64, order 0, d = 4:  (60) / (72) / (112), 64, 128: 80 / 133 / 233, 141, 490 and 86 / 96 / 146, 118, 361
//   L = 120, order 1, d = 8 (alone): 64 / 80 / 160 / 256: 711 / 1082 / 3641 / 8982 and 766 / 1343 / 3307 / 7420
//   L = 128, order 2, d = 3 (alone): 64 / 80 / 96 / 128: 929 / 1580 / 2110 / 3931 and 878 / 1298 / 2569 / 2857
//   L = 200, order 0, d = 4 (chained): 40 / 48 / 64 / 128: 597 / 967 / 1173 / 4584 and 677 / 722 / 860 / 2267
inline double four_gain(const SweepLoad& one, const SweepLoad& four, double step, double lone)
{
    auto rounds = [](const SweepLoad& l) {
        return l.even < l.items ? (double)l.items / (double)l.slots + 0.3 : (double)((l.items + l.slots - 1) / l.slots);
    };
    if ((four.items < four.slots ? four.items : four.slots) <= 4 * kNumCU) step *= lone;
    return rounds(one) * one.steps / (rounds(four) * four.steps * step);
}
// The fewest x paths for it next to the solo kernels: with fewer the quads are half empty and do not pay however many there
// are (n x m, L = 64, order 0, d = 4: 1 x 8192 / 2 x 8192 / 5 x 4000 / 7 x 1000: 804 / 1050 / 677 / 261 us and 1248 / 1305 /
// 787 / 219; L = 100, order 1, d = 5: 3 x 4000 / 5 x 4000: 1403 / 2057 and 1401 / 1773; L = 40, order 2, d = 5: 5 x 1000 /
// 6 x 3000: 435 / 1243 and 490 / 1021).
// Nor is it taken below kFourMinQuads, counted as for K(X, Y): half a wavefront per SIMD.
constexpr int64_t kFourMinQuads = 512;
constexpr int four_min_paths(int BL) { return BL == 0 ? 7 : (BL == 1 ? 5 : 6); }
constexpr int kTileRowPad = 8;     // backward: node columns kept left of column 0 in the pair's bottom row (all 1)
constexpr int kTileCkChunks = 8;   // backward: chunks of 8 macro-steps between two checkpoints (kept in LDS)

// Split mode: waves of a workgroup of the second launch (two per SIMD, or one where what it keeps of eight macro-steps, all of it
// in registers, and the lane's increments and sums need the whole register file), columns of a wave's window of y-side sums
// for tasks of K chunks, and that launch's LDS: the y increments of the workgroup's tasks, the windows, two edge feeds per wave;
// afterwards the waves' x-side sums.
constexpr int split_seg_waves(int BL, int DT, int M) { return (M << BL) >= 4 || DT >= ((M << BL) == 2 ? 6 : 16) ? 4 : 8; }
constexpr int split_window(int K, int rs2) { return ((K * kLockCH1 + kWave - 2) >> rs2) + 2; }
inline size_t split_seg_lds(int BL, int DT, int M, int K, int rs2, size_t* off_gy = nullptr, size_t* off_feed = nullptr)
{
    const int W = split_seg_waves(BL, DT, M);
    const size_t row = (size_t)(DT | 1) * 8;
    const size_t y = align_up(split_window(W * K, rs2) * row, 256), gy = align_up(W * split_window(K, rs2) * row, 256);
    if (off_gy) *off_gy = y;
    if (off_feed) *off_feed = y + gy;
    const size_t sweep = y + gy + (size_t)W * 2 * kLockCH1 * (1 << BL) * 8, sums = (size_t)W * kWave * M * row;
    return sweep > sums ? sweep : sums;
}
// Chunks per task: a strip's tasks fill one workgroup, at most this many where that leaves other strips and pairs too little.
constexpr int kSplitMaxChunks = 8, kSplitMaxChunks4 = 16;   // (workgroups of eight and of four waves)
// Whether a forward and a backward call in that form, with the strips of a pair in one workgroup, are faster than the form they
// replace (Plan p: a kept forward sweep where there is one).  Nearly always; us for both calls on the GPU, before and now
// (476 shapes of 4 to 250 pairs, 16 to 400 points, orders 0 to 2; one / two / four strips 1.5 / 1.7 / 2.5 times faster in the mean):
//   128 pairs, L = 256, d = 3 (1): 171 and 105;  4 pairs, L = 16, d = 3 (0): 54 and 25;  128 pairs, L = 400, d = 8 (0): 599 and 369;
//   250 pairs, L = 128, d = 3 (0), two strips: 85 and 67
// With so many strips that two workgroups share a compute unit, the lock-step kernels' kept form loses little to their fewer
// sweeps: 250 pairs, two strips, lead-lag, L = 100, d = 8 (1): 164 and 190; L = 200, d = 3 (0): 158 and 182; sixteen channels,
// L = 100 (0): 149 and 155; four strips, L = 200 (0): 403 and 414.
inline bool split_pays(const Plan& p, int strips)
{
    if (p.npairs * strips <= 384 || p.gramM != 0 || p.io_elem != 8) return true;
    return p.lock ? p.ll == 0 && p.DT <= 8 : p.ll != 0 || p.DT <= 8;
}

// Wide mode: waves per workgroup at most, doubles per block of the stored edges (right edge, and bottom edge without the
// corner they share), macro-steps per chunk (what a wave holds of the coming chunk stays in registers), and the scratch that
// its resident workgroups may take together: forward no more than kWideForward once it keeps the chip busy with the waves of
// that many workgroups.  Gram 64 x 64, L = 600, d = 20 (0), forward, with 6.6, 4 and 2 GiB: 13.5, 13.1 and 12.7 ms.
constexpr int kWideMaxWaves = 8;
constexpr int wide_edge_values(int BL) { return 2 * (1 << BL) - 1; }
constexpr int wide_chunk(int BL) { return BL == 2 ? 4 : 8; }
constexpr size_t kWideScratch = (size_t)8 << 30, kWideForward = (size_t)2 << 30;

// Band mode: strips per workgroup, block columns per hand-over ring, coarse y columns per y ring (powers of
// two), chunks the data-moving wave works ahead, and the bound on its polls of another workgroup's counter.
constexpr int kBandStrips = 4, kBandRing = 64, kBandYRing = 512, kBandLead = 2, kBandSpin = 1 << 22, kBandSlack = 8, kBandLeadRev = 3;

// Band mode takes over from three strips on (a single band then: measured a little ahead of the cooperative kernels).
constexpr int kBandMinStrips = 2;
constexpr int64_t kCoopMaxPairs = 1024;   // above this, one wave per pair already fills the chip

// Whether the wide kernels take the place of the wave-per-pair or cooperative kernels that the plan has come to: above
// sixteen channels always, backward also where those keep the y side out of LDS (their sums are then an atomic addition per
// block and channel) and next to the cooperative kernels with sixteen channels.  us per call, those kernels and these
// (d channels, order in brackets):
//   Gram 66 x 593, L = 124, 76, d = 19 (1), forward: 39185 and 4711;  31 x 917, L = 16, d = 19 (1), step: 24879 and 2976
//   64 pairs, L = 889, 460, d = 19 (0), step: 74602 and 2411;  96 pairs, L = 38, 68, d = 17 (1), forward: 215 and 39
//   Gram 59 x 106, L = 232, 164, d = 10 (0), step: 185727 and 7894 (y in memory);  1500 pairs, L = 300, 700, backward, y in
//   memory, d = 5 (0) / (1): 49543 / 49937 and 7085 / 9599;  d = 8: 119663 / 121405 and 7265 / 9784
//   backward with sixteen channels, cooperative, (0) / (1) / (2): 8 pairs, L = 150: 279 / 416 / 500 and 168 / 217 / 357; 64 pairs,
//   L = 300: 586 / 959 / 1420 and 393 / 485 / 835; 300 pairs, L = 200, 250: 873 / 905 / 1531 and 575 / 785 / 1306
// Also with less scratch than they would fill, down to one workgroup's (the figures: those kernels, these with all of their
// scratch, and with no more than those need).  ms, backward: 32 pairs, L = 2048, d = 17 (2): 551, 48 and 159; 64 pairs, d = 8 (2):
// 112, 69 and 133; 256 pairs, L = 2048, 1500, d = 17 (0): 1281, 25 and 46; Gram 100 x 100, L = 128, d = 20 (1): 310, 6.0 and 6.1;
// forward: Gram 64 x 64, L = 600, d = 20 (0): 167, 12.7 and 40; Gram 256 x 256, L = 128, d = 20 (0): 111, 10.3 and 50.6.
// Not elsewhere: forward with sixteen channels, 300 pairs, L = 200, 250: 150 / 180 / 248 and 195 / 206 / 288; backward, sixteen
// channels, wave per pair, 1500 pairs, L = 90 (1) / (2): 624 / 894 and 763 / 1250; up to eight channels with y in LDS, 64 pairs,
// L = 1500, d = 3 (1), backward: 5140 and 9668; forward with y in memory, 1500 pairs, L = 300, 700, d = 8 (0): 1468 and 2530.
inline bool wide_pays(const Plan& p)
{
    if (p.lock || p.solo || p.tile || p.quad || p.four || p.band || p.split) return false;
    return p.DT == 0 || (p.backward && (!p.y_lds || (p.coop && p.DT == 16)));
}

constexpr int kUncomputeS = 8;   // macro-steps between checkpoints when the reverse sweep inverts Eq. (1)
constexpr size_t kSecondChanceBytes = (size_t)8 << 20;   // scratch of the launch that solves drifted pairs once more
// A recovered forward value may differ from the exact checkpoint by this fraction of the lane's largest forward
// value; beyond it the pair is solved once more by the replay kernel.  Measured: on Brownian-like paths (the
// benchmark configurations) the differences stay below 3e-12 (a tolerance of 1e-12 already sends such pairs to
// the replay kernel) and the gradients agree with the reference to a few 1e-13; on paths with a few increments of
// order one a pair that passes can lose accuracy where its kernel values cancel (seen: 1.6e-10 of the gradient's
// largest entry, against 3e-12 from the replay kernel).  SK_FLAG_BWD_REPLAY is the choice for such data.
constexpr double kDriftTol = 1e-11;

inline Plan make_plan(bool backward, bool gram, bool symmetric, int64_t nx, int64_t ny, int64_t L1, int64_t L2,
                      int64_t d, int lam1, int lam2, int io_elem, bool uncompute = true, bool keep = false,
                      bool second_chance = false, bool lead_lag = false, bool may_four = true, size_t wide_scratch = kWideScratch,
                      bool split = false)
{
    // lead_lag: the sweep of two lead-lag paths (Section 4) on the grid of the original increments; lam1 and lam2 then
    // count the lead-lag level as one more dyadic level (the caller's orders plus one), L1, L2 and d are the caller's.
    // The level lies inside the blocks when these hold every refined cell of a pair of increments, above them
    // otherwise (Plan::ll); the tile kernels have no such form.
    // wide_scratch: what the resident workgroups of a wide launch may take together (0: no wide mode).
    // split: a backward plan of the kernels that sweep forward and adjoint side by side; Plan::split says whether the shape has
    // one.
    // second_chance: the plan of the launch that solves the listed pairs once more (wave-per-pair replay kernel,
    // a bounded number of waves, no increment and accumulator areas of its own: it works on the main plan's).
    // keep: a backward plan whose forward sweep may be a launch of its own (a forward call that keeps its sweep for
    // the backward call).  Lock-step and band plans are laid out for that anyway; solo plans then get checkpoints and
    // a bottom row per pair instead of per wave.
    Plan p;
    p.uncompute = backward && uncompute;
    const int elem = 8;
    p.io_elem = io_elem;
    p.backward = backward;
    p.symmetric = symmetric;
    p.elem = elem;
    p.nx = nx;
    p.ny = ny;
    p.npairs = gram ? nx * ny : nx;
    p.kcount = p.npairs;
    p.gramM = gram ? ny : 0;
    p.L1 = (int)L1; p.L2 = (int)L2; p.d = (int)d;
    p.r = (int)L1 - 1; p.q = (int)L2 - 1;
    if (p.npairs <= 0 || p.r <= 0 || p.q <= 0) return p;   // nothing to sweep
    int mn = lam1 < lam2 ? lam1 : lam2;
    if (lead_lag) {
        if (mn < 1) return p;   // not valid: the lead-lag level counts as one dyadic level on either side
        // With unequal orders the blocks stay below the lead-lag level on both sides (a block then lies inside one
        // quadrant of that level, whichever side is refined more).
        if (lam1 != lam2) mn -= 1;
    }
    p.BL = mn < kMaxBL ? mn : kMaxBL;
    p.rs1 = lam1 - p.BL; p.rs2 = lam2 - p.BL;
    p.mb = p.r << p.rs1; p.nb = p.q << p.rs2;
    if (lead_lag) p.ll = (p.rs1 == 0 && p.rs2 == 0) ? 1 : 2;
    p.ns = (p.mb + kWave - 1) / kWave;
    const int C = 1 << p.BL, R = C;
    p.rowlen = (int)align_up((size_t)(p.nb + 8) * C + 1, 64);   // a few block columns beyond the grid (band mode)
    p.rpad = (int)align_up((size_t)p.r, 64);
    p.qpad = (int)align_up((size_t)p.q, 64);
    p.DT = 0;
    for (int t : kTemplD) if (d <= t) { p.DT = t; break; }
    p.DP = p.DT ? (p.DT | 1) : (int)d;   // odd row stride: LDS bank spread (see Sweep::DSc)
    p.xstride = (int64_t)p.DP * p.rpad;
    p.ystride = (int64_t)p.DP * p.qpad;

    int64_t slots = 1;           // wavefronts of a launch with one pair each that the chip holds at once
    const int NVR = R + C + 1;   // block input edges kept per macro-step in the ring
    const size_t ring_step = (size_t)kWave * NVR * elem;
    p.coop = (p.ns >= 2 && p.npairs <= kCoopMaxPairs && !second_chance) ? 1 : 0;
    if (p.coop) {
        // Workgroup-shared LDS: y (+ gradient accumulators), flags, ones/zeros/outbox rings; then one replay
        // ring per wave.
        const int maxw = (backward && p.BL == 2) ? 4 : 8;
        p.nw = p.ns < maxw ? p.ns : maxw;
        // Outbox rings long enough for a whole row need no back-pressure; otherwise 32 columns (set below).
        p.CH = 8;
        const int CW = backward ? 2 * C : C;   // values per column in the hand-over rings
        {
            int full = 32;
            while (full < p.nb + 1) full <<= 1;
            p.RB = ((size_t)(2 * p.nw + 2) * full * CW * elem <= 40 * 1024) ? full : 32;
        }
        const size_t ycopy = (size_t)p.q * p.DP * elem;
        const size_t fixed = 512 + (size_t)(2 * p.nw + 2) * p.RB * CW * elem;
        const size_t budget = kLdsPerCU - 1024;
        const size_t ring_min = (backward && !p.uncompute) ? (size_t)p.nw * 4 * ring_step : 0;
        const size_t yneed = ycopy * (backward ? 2 : 1);
        p.y_lds = (p.DT != 0 && align_up(yneed, 256) + fixed + ring_min <= budget) ? 1 : 0;
        size_t used = p.y_lds ? align_up(ycopy, 256) : 0;
        p.coop_off_gdy = used;
        if (p.y_lds && backward) used += align_up(ycopy, 256);
        p.coop_off_flags = used;
        used += 512;
        p.coop_off_obox = used;   // ones, zeros, nw outboxes, nw staging rings
        used += (size_t)(2 * p.nw + 2) * p.RB * CW * elem;
        used = align_up(used, 256);
        p.coop_off_ring = used;
        if (backward && p.uncompute) {
            p.S = kUncomputeS;
            p.nseg = (p.nb + kWave - 1 + p.S - 1) / p.S;
        } else if (backward) {
            int S = 64;
            while (S > 4 && used + (size_t)p.nw * S * ring_step > budget) S >>= 1;
            p.S = S;
            p.nseg = (p.nb + kWave - 1 + S - 1) / S;
            p.coop_ring_stride = (size_t)S * ring_step;
            used += (size_t)p.nw * p.coop_ring_stride;
        }
        p.lds_wave = 0;
        p.lds_bytes = align_up(used, 256);
        int wg_per_cu = (int)(kLdsPerCU / p.lds_bytes);
        if (wg_per_cu < 1) wg_per_cu = 1;
        if (wg_per_cu * p.nw > 8) wg_per_cu = 8 / p.nw > 0 ? 8 / p.nw : 1;
        int64_t cap = (int64_t)kNumCU * wg_per_cu;
        p.grid = (int)(p.npairs < cap ? p.npairs : cap);
        p.nslots = p.grid;
    } else {
        // LDS per wave: y increments (+ their gradient accumulators when going backward) and the replay ring.
        size_t ybytes = (size_t)p.DP * p.qpad * elem * (backward ? 2 : 1);
        p.y_lds = (p.DT != 0 && ybytes <= kLdsPerWave) ? 1 : 0;   // up to a whole compute unit for four waves
        size_t used = p.y_lds ? ybytes : 0;
        p.ring_off = used;
        if (backward && p.uncompute) {
            p.S = kUncomputeS;
            p.nseg = (p.nb + kWave - 1 + p.S - 1) / p.S;
        } else if (backward) {
            auto fit = [&](size_t before) {
                int S = 64;
                while (S > 4 && before + (size_t)S * ring_step > kLdsPerWave) S >>= 1;
                return S;
            };
            int S = fit(used);
            if (used + (size_t)S * ring_step > kLdsPerWave) {
                // not even the shortest ring fits next to the y increments: these stay in global memory
                p.y_lds = 0;
                used = 0;
                p.ring_off = 0;
                S = fit(0);
            }
            p.S = S;
            p.nseg = (p.nb + kWave - 1 + S - 1) / S;   // strips run nb + (lanes-1) macro-steps at most
            used += (size_t)S * ring_step;
        }
        p.lds_wave = align_up(used, 256);
        p.lds_bytes = p.lds_wave * kWavesPerWG;

        int wg_per_cu = (int)(kLdsPerCU / (p.lds_bytes ? p.lds_bytes : 1));
        if (wg_per_cu < 1) wg_per_cu = 1;
        if (wg_per_cu > 4) wg_per_cu = 4;
        if (backward && wg_per_cu > 2) wg_per_cu = 2;   // register file: the backward kernels run 2 waves per SIMD at most
        int64_t want = (p.npairs + kWavesPerWG - 1) / kWavesPerWG;
        int64_t cap = (int64_t)kNumCU * wg_per_cu;
        if (second_chance && cap > kNumCU) cap = kNumCU;
        slots = cap * kWavesPerWG;
        p.grid = (int)(want < cap ? want : cap);
        p.nslots = (int64_t)p.grid * kWavesPerWG;
    }
    if (second_chance) {
        // rows, adjoint rows and checkpoints per wave slot, held to kSecondChanceBytes (at least one workgroup)
        const int C2 = 1 << p.BL;
        const size_t slot_bytes = ((size_t)p.ns * p.rowlen + 4 * (size_t)p.rowlen +
                                   (size_t)p.ns * (p.nseg + 1) * (2 * C2 + 2) * kWave) * elem;
        int64_t g = (int64_t)(kSecondChanceBytes / (slot_bytes * kWavesPerWG));
        if (g < 1) g = 1;
        if (g < p.grid) p.grid = (int)g;
        p.nslots = (int64_t)p.grid * kWavesPerWG;
    }

    // Lock-step mode replaces the modes above when every pair can have a workgroup of its own resident at
    // once: the chip is then under-filled and the time of a call is the latency of one pair's chain of
    // macro-steps, which this mode shortens (fewer instructions in the wave that carries the recurrence,
    // fewer strips, no waits).
    if (lock_max_rows(backward, p.BL, p.DT) > 0 && (!backward || p.uncompute) && !second_chance) {
        const int maxM = lock_max_rows(backward, p.BL, p.DT);
        int M = 1;
        while (M < maxM && (p.mb + kWave * M - 1) / (kWave * M) > 2) M *= 2;
        const int lns = (p.mb + kWave * M - 1) / (kWave * M);
        const int NT = (int)align_up((size_t)p.nb + kWave - 1, 8);
        const int lrow = (int)align_up((size_t)kWave * C + (size_t)NT * C + C + 2, 2);
        size_t used = 0;
        auto lds_take = [&](size_t bytes) { size_t o = used; used = align_up(used + bytes, 256); return o; };
        const size_t ycopy = (size_t)p.q * p.DP * elem;
        const size_t o_y = lds_take(ycopy);
        const size_t o_gy = backward ? lds_take(ycopy) : 0;
        const size_t cstride = (size_t)16384 * M;   // 2 chunks x (8 steps x 16 B | 4 steps x 32 B) x 64 lanes x M
        const size_t o_cr = lds_take(cstride * lns);
        const size_t gstride = (size_t)2 * kLockCH2 * M * kWave * elem;
        const size_t o_gp = backward ? lds_take(gstride * lns) : 0;
        const size_t o_kr = lds_take((size_t)(lns + 1) * lrow * elem);
        const size_t o_ar = backward ? lds_take((size_t)(lns + 1) * lrow * elem) : 0;
        const size_t o_dump = lds_take((size_t)(kWave + 8) * C * elem);
        const size_t kstride = (size_t)2 * (M * R + 1 + C) * kWave * elem;   // two staged checkpoints per strip
        const size_t o_ck = backward ? lds_take(kstride * lns) : 0;
        const int waves = lns == 1 ? 3 : (lns == 2 ? 8 : 12);
        int wgpc = used ? (int)(kLdsPerCU / used) : 0;
        if (wgpc * waves > 16) wgpc = 16 / waves;
        if (lns <= (backward ? kLockMaxStripsBwd : kLockMaxStrips) && used <= kLdsPerCU - 1024 && wgpc >= 1 && p.npairs <= (int64_t)kNumCU * wgpc) {
            p.lock = 1; p.coop = 0;
            p.lk_M = M; p.lk_ns = lns; p.lk_NT = NT; p.lk_rowlen = lrow;
            p.lk_padb = lns * kWave * M - p.mb;
            p.lk_off_y = o_y; p.lk_off_gy = o_gy; p.lk_off_cring = o_cr; p.lk_off_gp = o_gp;
            p.lk_off_krows = o_kr; p.lk_off_arows = o_ar; p.lk_off_dump = o_dump;
            p.lk_cring_stride = cstride; p.lk_gp_stride = gstride;
            p.lk_off_ck = o_ck; p.lk_ck_stride = kstride;
            p.y_lds = 1;
            p.lds_wave = 0;
            p.lds_bytes = align_up(used, 256);
            p.grid = (int)p.npairs;
            p.nslots = p.npairs;
            p.S = kLockS;
            p.nseg = NT / kLockS;
        }
    }

    // Solo mode: enough pairs to fill the chip, and all block rows of a pair fit one strip of 64 M rows.
    if (!p.lock && solo_max_rows(backward, p.BL, p.DT) > 0 && (!backward || p.uncompute) && !second_chance) {
        const int M = p.mb > kWave ? 2 : 1;
        const int NT = (int)align_up((size_t)p.nb + kWave - 1, 8);
        size_t used = 0;
        auto lds_take = [&](size_t bytes) { size_t o = used; used = align_up(used + bytes, 256); return o; };
        const size_t ycopy = (size_t)p.q * p.DP * elem;
        lds_take(ycopy);
        const size_t o_gy = backward ? lds_take(ycopy) : 0;
        const size_t o_gyp = backward ? lds_take(ycopy) : 0;   // y-side sums of the pair in work
        const size_t o_kr = backward ? lds_take(((size_t)kWave * C + (size_t)NT * C + 2) * elem) : 0;
        const size_t o_dump = backward ? lds_take((size_t)kWave * C * elem) : 0;
        const int maxwg = backward ? solo_bwd_waves_per_simd(p.BL, M, p.DT) : 4;   // register file of the backward kernel
        if (M <= solo_max_rows(backward, p.BL, p.DT) && p.mb <= kWave * M && used * kWavesPerWG <= kLdsPerCU) {
            p.solo = 1; p.coop = 0;
            p.lk_M = M; p.lk_ns = 1; p.lk_NT = NT; p.lk_padb = kWave * M - p.mb;
            p.lk_off_y = 0; p.lk_off_gy = o_gy; p.lk_off_krows = o_kr; p.lk_off_dump = o_dump; p.lk_off_gyp = o_gyp;
            p.y_lds = 1;
            p.lds_wave = used;
            p.lds_bytes = used * kWavesPerWG;
            int wgpc = (int)(kLdsPerCU / p.lds_bytes);
            if (wgpc > maxwg) wgpc = maxwg;
            const int64_t want = (p.npairs + kWavesPerWG - 1) / kWavesPerWG;
            const int64_t cap = (int64_t)kNumCU * wgpc;
            slots = cap * kWavesPerWG;
            p.grid = (int)(want < cap ? want : cap);
            p.nslots = (int64_t)p.grid * kWavesPerWG;
            p.S = kLockS;
            p.nseg = NT / kLockS;
        }
    }

    // Tile mode: many pairs of at most 64 x 64 unrefined cells with 8 or 16 channels; the contractions over
    // the channels and over the rows / columns run as MFMA tiles, the sweep reads one number per cell from LDS.
    if (!p.lock && !lead_lag && p.BL == 0 && p.rs1 == 0 && p.rs2 == 0 && (p.DT == 8 || p.DT == 16) && p.mb > kWave / 2 &&
        p.mb <= kWave && p.nb > kWave / 2 && p.nb <= kWave && (!backward || p.uncompute) && !second_chance) {
        const int NT = (int)align_up((size_t)p.nb + kWave - 1, 8);
        size_t used = 0;
        auto lds_take = [&](size_t bytes) { size_t o = used; used = align_up(used + bytes, 256); return o; };
        lds_take((size_t)kTileCols * kTileStride * elem);
        // backward: compact checkpoints (two doubles per lane) every kTileCkChunks chunks of 8 macro-steps
        const int nck = backward ? (NT / kLockS - 1) / kTileCkChunks : 0;
        const size_t o_ck = nck ? lds_take((size_t)nck * 2 * kWave * elem) : 0;
        // backward: the pair's bottom row, node columns -kTileRowPad .. 64 and slack up to a multiple of eight
        const size_t o_kr = backward ? lds_take((size_t)(kTileRowPad + kWave + 8) * elem) : 0;
        p.tile = 1; p.solo = 0; p.coop = 0;
        p.lk_M = 1; p.lk_ns = 1; p.lk_NT = NT; p.lk_padb = kWave - p.mb;
        p.lk_off_y = 0; p.lk_off_gy = 0; p.lk_off_krows = o_kr; p.lk_off_dump = 0; p.lk_off_ck = o_ck;
        p.y_lds = 0;
        p.lds_wave = used;
        p.lds_bytes = used * kWavesPerWG;   // one workgroup per compute unit
        const int64_t want = (p.npairs + kWavesPerWG - 1) / kWavesPerWG;
        p.grid = (int)(want < kNumCU ? want : kNumCU);
        p.nslots = (int64_t)p.grid * kWavesPerWG;
        p.S = kLockS;
        p.nseg = NT / kLockS;
    }

    // Symmetric Gram matrix: k(x, y) = k(y, x) bit for bit, so the solo, four-pair and tile kernels solve the pairs n <= m
    // only, write both entries of K, and use the sum of the two upstream gradients.  Eq. (1) is symmetric under
    // a swap of the paths together with their dyadic orders, so this holds for equal orders only; with unequal
    // orders K(X, X) is not a symmetric matrix and all N^2 pairs are solved over the shared increment buffer.
    const bool may_tri = symmetric && gram && nx == ny && lam1 == lam2;

    // Four-pair mode: backward calls for Gram matrices, where it pays (four_gain).
    bool four = false;
    int64_t four_slots = 0;
    if (may_four && backward && gram && p.uncompute && !keep && !second_chance && !lead_lag && !p.tile && !p.lock && !p.coop &&
        p.DT >= 2 && gram_quads(false, nx, ny) >= kFourMinQuads && (!p.solo || nx >= four_min_paths(p.BL))) {
        const int DT = four_channels(p.DT, p.d), band = kWave / kQuadPairs * four_rows(p.BL, DT);
        const int bands = (p.mb + band - 1) / band;
        size_t used = 0;
        auto lds_take = [&](size_t bytes) { size_t o = used; used = align_up(used + bytes, 256); return o; };
        const size_t o_y = lds_take((size_t)(p.q + 1) * quad_y_stride(DT) * elem);
        const size_t o_gyp = lds_take((size_t)p.q * DT * elem);
        const size_t o_gring = lds_take((size_t)kQuadPairs * four_gring_stride(DT) * elem);
        const size_t o_ring = lds_take((size_t)(bands > 1 ? 3 : 1) * kWave * C * elem);
        const int occupancy = four_occupancy(p.BL, DT);
        int waves = used ? (int)(kLdsPerCU / used) : 0;                  // per compute unit
        if (waves > 4 * occupancy) waves = 4 * occupancy;
        if (waves >= 4) {
            const SweepLoad one = {may_tri && p.solo ? nx * (nx + 1) / 2 : nx * ny, slots,
                                   p.solo ? (double)p.lk_M * p.lk_NT : (double)p.ns * (p.nb + kWave - 1), p.npairs};
            const int64_t steps = (int64_t)bands * four_rows(p.BL, DT) * (p.nb + kWave / kQuadPairs - 1);
            SweepLoad quads = {gram_quads(may_tri, nx, ny), (int64_t)kNumCU * waves, (double)steps, 0};
            quads.even = four_even_share(quads.items, quads.items < quads.slots ? quads.items : quads.slots,
                                         steps * (C * C * 11 + 15 + 5 * DT));
            // (Eight channels and few columns, chained: the x-side sums, which both add to memory, are most of the time.
            // 64 x 64 paths of 200 and 30 points, order 0: 596 us and 690.)
            const bool sums = !p.solo && p.DT == 8 && p.nb < kWave;
            const bool alone = p.solo && occupancy == 2 && solo_bwd_waves_per_simd(p.BL, p.lk_M, p.DT) == 1;
            // (Nine to twelve channels are sixteen to the solo kernel: L = 34, order 1, d = 12, (54) / (89): 242 / 478 and 142 / 246.)
            const bool twelve = alone && DT < p.DT;
            const double step = !p.solo ? 0.65 : (twelve ? 1.1 : (alone ? 1.75 : (p.lk_M == 2 && p.DT >= 5 ? 0.88 : 1.0)));
            const double gain = four_gain(one, quads, step, twelve ? 0.6 : (alone && p.DT >= 8 ? 0.85 : 0.73));
            four = !sums && gain > 1.0;
            // A step with a kept sweep and one without (K(X, X) of n paths): two block rows per lane of few channels, L = 128,
            // order 1, d = 3, n = 92 / 112: 500 / 673 us and 595 / 611; order 2, n = 80 / 112: 973 / 1686 and 1015 / 1628;
            // L = 120, order 0, d = 3, n = 92 / 112: 310 / 401 and 383 / 400.  Elsewhere small gains are enough: L = 64, order 0,
            // d = 4, n = 128: 388 and 271; L = 100, order 1, d = 5, n = 128: 1240 and 1021.
            p.four_over_kept = four && gain >= (p.solo && p.lk_M == 2 && p.DT <= 4 ? 1.2 : 1.0);
            four_slots = quads.slots;
            if (four) p.qd_even = quads.even;
        }
        if (four) {
            p.lock = 0; p.coop = 0; p.solo = 0; p.four = 1;
            p.DT = DT;
            p.lk_M = bands > 1 ? 2 : 1;
            p.fv_bands = bands; p.lk_padb = bands * band - p.mb;
            p.lk_ns = 0;
            p.lk_NT = p.nb + kWave / kQuadPairs - 1;
            p.lk_off_y = o_y; p.lk_off_gyp = o_gyp; p.lk_off_gp = o_gring; p.lk_off_krows = o_ring;
            p.y_lds = 1;
            p.lds_wave = used;
            p.lds_bytes = used;                  // one wavefront per workgroup
            p.nseg = (p.lk_NT - 1) / kFourCkpt + 1;   // checkpoint places per band
        }
    }

    if (may_tri && (p.solo || p.tile || p.four)) {
        p.tri = 1;
        p.npairs = nx * (nx + 1) / 2;
        const int64_t want = (p.npairs + kWavesPerWG - 1) / kWavesPerWG;
        if (want < p.grid) p.grid = (int)want;
        p.nslots = (int64_t)p.grid * kWavesPerWG;
    }
    // The sequence of quads: rows of the Gram matrix in groups of four x paths (symmetric: the pairs n <= m of row m).
    if (gram) p.nquads = gram_quads(p.tri != 0, nx, ny);
    if (four) {
        p.grid = (int)(p.nquads < four_slots ? p.nquads : four_slots);
        p.nslots = p.grid;
    }
    // The four-pair launch's counter (bd_flags[0]); the other kernels of a backward Gram call leave its place free, so that
    // what follows it does not move with the launch mode.
    if (backward && gram && !keep) p.nflags = 1;

    // Quad mode: forward calls for Gram matrices (the four pairs of a wavefront share the y path) on the shapes of the
    // tile kernels and on those of the solo kernels whose blocks hold all of the refinement.  The sequence is the Gram
    // matrix row by row (y-major) in groups of four x paths; a symmetric Gram matrix has the pairs n <= m of row m
    // only.  Two workgroups of four waves per compute unit.
    if ((p.tile || p.solo) && !backward && gram && !lead_lag && p.rs1 == 0 && p.rs2 == 0) {
        const int lanes = kWave / kQuadPairs;
        // As few rows per lane as hold the pair: a row above the grid costs what any other does.  Gram 256 x 256, 94 block
        // rows, d = 6, order 1, eight rows and six: 676 and 506 us; d = 2, 79 block rows, order 0, eight and five: 311
        // and 213 us.  (Kernels of fewer than four rows are not built.)
        int M = (p.mb + lanes - 1) / lanes;
        if (M < kQuadMinRows) M = kQuadMinRows;
        const size_t ycopy = align_up((size_t)(p.nb + 1) * quad_y_stride(p.DT) * elem, 256);   // the y copy and a row of zeros
        const int64_t quad_slots = 4 * kNumCU * (2 * ycopy * kWavesPerWG <= kLdsPerCU ? 2 : 1);
        const bool pays = !p.solo || p.DT < 8 || M <= 4 ||
                          quad_pays(p.npairs, slots, (double)p.lk_M * p.lk_NT, p.nquads, quad_slots, (double)M * (p.nb + lanes - 1));
        if (M <= quad_max_rows(p.BL, p.DT) && p.mb <= M * lanes && ycopy * kWavesPerWG <= kLdsPerCU && pays) {
            p.tile = 0; p.solo = 0; p.quad = 1;
            p.lk_M = M; p.lk_ns = 1; p.lk_NT = p.nb + lanes - 1; p.lk_padb = M * lanes - p.mb;
            p.y_lds = 1;
            p.lds_wave = ycopy;
            p.lds_bytes = p.lds_wave * kWavesPerWG;
            const int64_t want = (p.nquads + kWavesPerWG - 1) / kWavesPerWG;
            const int64_t cap = (int64_t)kNumCU * (2 * p.lds_bytes <= kLdsPerCU ? 2 : 1);
            p.grid = (int)(want < cap ? want : cap);
            p.nslots = (int64_t)p.grid * kWavesPerWG;
        }
    }

    // Band mode: few pairs of long paths.  The strips of a pair are spread over workgroups (bands of kBandStrips
    // strips) that all run at once; chosen when that fills more of the chip than one workgroup per pair does.
    if (!p.lock && !p.tile && !p.solo && !p.four && (!backward || p.uncompute) && p.DT >= 2 && p.DT <= 8 && p.ns > kBandMinStrips &&
        !second_chance) {
        const int nbands = (p.ns + kBandStrips - 1) / kBandStrips;
        if (p.npairs * nbands <= kNumCU) {
            const int NT = (int)align_up((size_t)p.nb + kWave - 1, 8);
            size_t used = 0;
            auto lds_take = [&](size_t bytes) { size_t o = used; used = align_up(used + bytes, 256); return o; };
            const size_t ybytes = (size_t)kBandYRing * p.DP * elem;
            p.bd_off_y = lds_take(ybytes);
            p.bd_off_gy = backward ? lds_take(ybytes) : 0;
            // forward: hand-over rings; backward: adjoint rings, forward-value rings, checkpoint staging
            p.bd_off_rings = lds_take(((size_t)(kBandStrips + 1) * kBandRing * C +
                                       (backward ? (size_t)kBandStrips * kBandRing * C +
                                                       (size_t)kBandStrips * 2 * (R + 1 + C) * kWave : 0)) * elem);
            p.band = 1; p.coop = 0; p.bd_nbands = nbands;
            p.lk_M = 1; p.lk_ns = p.ns; p.lk_NT = NT; p.lk_padb = p.ns * kWave - p.mb;
            p.y_lds = 1;
            p.lds_wave = 0;
            p.lds_bytes = used;
            p.grid = (int)(p.npairs * nbands);
            p.nslots = p.npairs;
            p.S = kLockS;
            p.nseg = NT / kLockS;
            p.nflags = (int)(2 * p.npairs * nbands);
        }
    }

    // Split mode: few pairs, whose sweeps are chains that leave most of the chip idle.  In place of the lock-step kernels (up
    // to four strips here: the sweeps alone need less LDS and fewer waves) and of the band kernels.
    if (split && p.uncompute && !p.solo && !p.tile && !p.four && p.DT >= 2) {
        int M = 1, lns = 0, NT = (int)align_up((size_t)p.nb + kWave - 1, 8), lrow = 0;
        size_t used = 0, o_y = 0, o_cr = 0, o_kr = 0, o_dump = 0, cstride = 0;
        auto lds_take = [&](size_t bytes) { size_t o = used; used = align_up(used + bytes, 256); return o; };
        bool lock = lock_max_rows(true, p.BL, p.DT) > 0 && p.npairs <= kNumCU;
        if (lock) {
            const int maxM = lock_max_rows(true, p.BL, p.DT);
            while (M < maxM && (p.mb + kWave * M - 1) / (kWave * M) > 2) M *= 2;
            lns = (p.mb + kWave * M - 1) / (kWave * M);
            lrow = (int)align_up((size_t)kWave * C + (size_t)NT * C + C + 2, 2);
            o_y = lds_take((size_t)p.q * p.DP * elem);
            cstride = (size_t)16384 * M;
            o_cr = lds_take(cstride * lns);
            o_kr = lds_take((size_t)(lns + 1) * lrow * elem);
            o_dump = lds_take((size_t)(kWave + 8) * C * elem);
            lock = lns <= kLockMaxStrips && used <= kLdsPerCU - 1024 && split_pays(p, lns);
        }
        if (lock) {
            p.split = 1; p.lock = 1; p.band = 0; p.coop = 0;
            p.lk_M = M; p.lk_ns = lns; p.lk_NT = NT; p.lk_rowlen = lrow; p.lk_padb = lns * kWave * M - p.mb;
            p.lk_off_y = o_y; p.lk_off_cring = o_cr; p.lk_off_krows = o_kr; p.lk_off_dump = o_dump;
            p.lk_cring_stride = cstride;
            p.lds_bytes = used;
            p.grid = (int)(2 * p.npairs);
            p.nflags = 0;
        } else if (p.band) {
            p.split = 1;
            used = 0;
            p.bd_off_y = lds_take((size_t)kBandYRing * p.DP * elem);
            p.bd_off_rings = lds_take((size_t)(kBandStrips + 1) * kBandRing * C * elem);
            p.lds_bytes = used;
            p.grid = (int)(2 * p.npairs * p.bd_nbands);
        }
        if (p.split) {
            p.y_lds = 1; p.lds_wave = 0; p.nslots = p.npairs;
            p.S = kLockS; p.nseg = NT / kLockS;
            const int W = split_seg_waves(p.BL, p.DT, p.lk_M), most = W == 8 ? kSplitMaxChunks : kSplitMaxChunks4, nck = NT / kLockCH1;
            int K = p.band ? 8 : (nck + W - 1) / W;
            if (K > most) K = most;
            while (K > 1 && split_seg_lds(p.BL, p.DT, p.lk_M, K, p.rs2) > kLdsPerCU - 1024) K /= 2;
            p.sp_chunks = K;
            p.sp_tasks = (nck + K - 1) / K;
            p.sp_win = split_window(K, p.rs2);
            p.sp_lds = split_seg_lds(p.BL, p.DT, p.lk_M, K, p.rs2, &p.sp_off_gy, &p.sp_off_feed);
            p.sp_ackpt_slot = (int64_t)p.lk_ns * p.sp_tasks * (p.lk_M * R + 1 + C) * kWave;
        }
    }

    // Wide mode takes over what is left to the wave-per-pair and the cooperative kernels with more channels than those hold
    // in registers, or with y increments (and their sums) that do not fit in LDS.
    if (wide_scratch != 0 && wide_pays(p) && (!backward || p.uncompute) && !second_chance) {
        const int NT = (int)align_up((size_t)p.nb + kWave - 1, 8);
        const int64_t pairs = may_tri ? nx * (nx + 1) / 2 : p.npairs;
        const int64_t slot = (int64_t)p.ns * kWave * (NT + (backward ? (int64_t)(NT + 2) * wide_edge_values(p.BL) : 0));
        // As many waves per pair as fill the chip: two wavefronts per SIMD by registers, forward four.  Where the scratch
        // leaves room for fewer workgroups, they have more waves, up to one per strip.
        const int64_t resident = (backward ? 8 : 16) * kNumCU, waves = p.ns < kWideMaxWaves ? p.ns : kWideMaxWaves;
        int64_t most = (int64_t)(wide_scratch / ((size_t)slot * elem));   // workgroups
        if (!backward && most > resident / waves) {
            const int64_t enough = (int64_t)(kWideForward / ((size_t)slot * elem));
            if (most > enough) most = enough > resident / waves ? enough : resident / waves;
        }
        if (most > pairs) most = pairs;
        if (most >= 1) {
            int64_t nw = (resident + most - 1) / most;
            if (nw > waves) nw = waves;
            if (most > resident / nw) most = resident / nw;
            const int64_t rounds = (pairs + most - 1) / most;
            const int64_t grid = (pairs + rounds - 1) / rounds;   // the same rounds, evenly filled
            p.wide = 1; p.coop = 0;
            p.nw = (int)nw;
            p.tri = may_tri ? 1 : 0;
            p.npairs = pairs;
            p.lk_M = 1; p.lk_ns = p.ns; p.lk_NT = NT; p.lk_padb = p.ns * kWave - p.mb;
            p.wd_slot = slot;
            p.y_lds = 0;
            p.lds_wave = p.lds_bytes = 0;
            p.grid = (int)grid;
            p.nslots = grid;
        }
    }

    // Workspace layout (all offsets 256-byte aligned).
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    // first, so that their place does not depend on the rest of the layout: the error flag, the progress counters
    // of band mode directly behind it (cleared with it), and behind those the counter of drifted pairs
    p.off_err = take(256);
    p.off_flags = take((size_t)p.nflags * sizeof(int) + 4);
    p.off_badcnt = p.off_flags + (size_t)p.nflags * sizeof(int);
    if (!second_chance) {
        p.off_dxT = take((size_t)nx * p.xstride * elem);
        p.off_dyT = symmetric ? p.off_dxT : take((size_t)ny * p.ystride * elem);
    }
    if (p.wide) p.off_wd = take((size_t)p.nslots * p.wd_slot * elem);
    p.rows_slot = p.four ? (int64_t)p.fv_bands * kQuadPairs * p.rowlen : (p.split && p.lock ? 0 : (int64_t)p.ns * p.rowlen);
    p.off_rows = take((size_t)p.nslots * p.rows_slot * elem);
    if (backward) {
        if (!second_chance) {
            p.off_gdxT = take((size_t)nx * p.xstride * elem);
            p.off_gdyT = symmetric ? p.off_gdxT : take((size_t)ny * p.ystride * elem);
        }
        p.adj_slot = p.wide || p.split ? 0 : (p.band && p.bd_nbands > 4 ? p.bd_nbands : 4) * (int64_t)p.rowlen;   // two rows of 2C values per block column; band mode: one row per band
        p.off_adj = take((size_t)p.nslots * p.adj_slot * elem);
        // lane state kept per checkpoint: right edge, bottom edge, bottom-left corner
        const bool lean = p.lock || p.solo || p.tile || p.band || p.four;
        const int NVC = lean ? p.lk_M * R + C + 2 : R + C + 2;
        p.ckpt_slot = p.tile || p.wide ? 0 : (int64_t)(lean ? p.lk_ns : p.ns) * (p.nseg + 1) * NVC * kWave;
        if (p.four) {
            p.ckpt_slot = (int64_t)p.fv_bands * p.nseg * four_ckpt_values(p.BL, p.DT) * kWave;
            p.fv_gx_slot = p.fv_bands > 1 ? (int64_t)p.fv_bands * four_rows(p.BL, p.DT) * p.DT * kWave : 0;
            p.off_fvgx = take((size_t)p.nslots * p.fv_gx_slot * elem);
        }
        p.keep_solo = (keep && p.solo) ? 1 : 0;
        p.off_ckpt = take((size_t)(p.keep_solo ? p.npairs : p.nslots) * p.ckpt_slot * elem);
        if (p.keep_solo) {
            p.keep_len = (int64_t)kWave * C + (int64_t)p.lk_NT * C + 2;   // the bottom row as the kernel holds it in LDS
            p.off_keep = take((size_t)p.npairs * p.keep_len * elem);
            p.off_keep_tag = take(256);
        }
        if (p.lock) p.off_keep = take((size_t)p.npairs * (p.lk_ns + 1) * p.lk_rowlen * elem);
        else if (p.band) p.off_keep = take((size_t)p.kcount * elem);   // band mode: the kernel values of the kept sweep
        if (p.lock || p.band) p.off_keep_tag = take(256);   // which call's forward sweep the workspace holds
        if (p.split) {
            p.off_keep_tag = p.off_badcnt;   // (this mode counts no drifted pairs, and every other backward call clears that place)
            p.off_sp_arows = take((size_t)p.npairs * (p.lock ? (p.lk_ns + 1) * p.lk_rowlen : p.lk_ns * p.rowlen) * elem);
            p.off_sp_ackpt = take((size_t)p.npairs * p.sp_ackpt_slot * elem);
        }
    }
    if (io_elem != elem) {
        p.off_kio = take((size_t)p.kcount * elem);
        if (backward) p.off_gkio = take((size_t)p.kcount * elem);
    }
    if (backward && p.uncompute && !second_chance && !p.split) p.off_badlist = take((size_t)p.kcount * sizeof(long long));
    p.total = off;
    p.valid = true;
    if (p.four && p.total > kFourScratch) {
        const Plan one = make_plan(backward, gram, symmetric, nx, ny, L1, L2, d, lam1, lam2, io_elem, uncompute, keep,
                                   second_chance, lead_lag, false, wide_scratch);
        if (one.total < p.total) return one;
    }
    return p;
}

}  // namespace sk
