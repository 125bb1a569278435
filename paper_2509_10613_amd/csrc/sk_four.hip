// Backward sweep of Gram matrices with four path pairs per wavefront (gfx950).
//
// The solo backward kernel of sk_solo_impl.h gives a pair all 64 lanes: the skew of the anti-diagonal sweep
// (Section 3.3) leaves 63 of its nb + 63 macro-steps per lane outside the grid.  Here a pair has 16 lanes, each with
// two or four consecutive block rows, and the four groups of 16 lanes work on four pairs of a Gram row at once:
//
//  * a band of 16 lanes takes nb + 15 macro-steps; longer pairs are several bands, one after the other, whose bottom
//    rows (forward values, and the adjoints that go up from band to band) wait in the wavefront's global scratch;
//  * the four pairs share the y path: its increments sit in LDS once.  What the y side of the linear map of Section
//    3.4 adds up for a column travels with the column from lane to lane (the reverse sweep reaches a column's last
//    block row first and its first one 15 macro-steps later), in registers; only the first lane of a group writes it
//    to LDS, and once in sixteen macro-steps the four groups' sums are added to the quad's, without atomics;
//  * nothing is masked: a lane whose column lies outside the grid reads a row of zeros behind the y copy, works with
//    p = 0, i.e. A = B = 1, and adds zeros (its travelling sum belongs to no column and is dropped);
//  * rows above the grid fill the first band from the top; macro-steps in which only they would work are skipped.
//
// The reverse sweep inverts Eq. (1) between checkpoints of the lane state and is checked against them (sk_lane.h).  A pair
// that drifts is listed for the replay kernel, replaced by zeros, and the quad is swept again for the other three: the sums
// of a quad are never split by pair, so a drifted pair costs more than in the one-pair kernels and has to be rarer.  What
// decides is how far an error travels between two checkpoints, and a lane's four block rows take it twice as far per
// macro-step as two.  Pairs that drift of Gram 256 x 256, L = 128, order 1, d = 3, and milliseconds, by the squared length
// of the paths' increments (one-pair kernel: a checkpoint every 8 macro-steps):
//
//    spacing       squared length 4      10           20             30            50
//    one-pair        0    6.1        0   6.2      0    6.2      192   7.4    28850   167
//    32              0    3.8      345   6.3  12682   76.7    46700   267    65494   371
//    8               0    4.2        0   4.2     37    4.8     1682  15.4    24725   146
//    4               0    4.8        0   4.8      0    4.9        6   5.5     1132    13
//    by band         0    3.8        0   4.4      1    5.9      105   6.7     3884    29   (as built)
//
// Checkpoints are what the kernel moves through memory, so a band takes 16, 8 or 4 by the largest increment product that
// one of its blocks can have (kFourCalm, kFourSteady), with the guard at kFourDriftTol.  1 / B has a term more than in the
// other kernels: theirs is what drifts first on unrefined paths (L = 60, order 0, d = 5, squared length 10: 8315 pairs in
// the one-pair kernel, 12671 here without the term, 15 with it; no time is seen).
//
// Bound by fp64 issue: Gram 256 x 256, L = 128, order 1, d = 3: 5.9 -> 3.8 ms; K(X, X) of 300 paths, L = 100, order 1,
// d = 5: 4.6 -> 2.5 ms; Gram 128 x 128, L = 100, order 0, d = 16: 4.0 -> 2.7 ms.  Four block rows per lane
// up to six channels, two from eight on and for blocks of 4 x 4 cells: with more the lane state does not fit the 256
// registers of a wavefront that shares its SIMD (eight rows, d = 3: 1 KB of it in scratch, 22 ms), and a lone wavefront
// is slower (4.7 ms).  Sixteen channels, and twelve with 4 x 4 blocks, do not fit either way and run alone on their SIMD
// (L = 100, order 0, d = 16: 6.0 against 14.0 ms; order 2, L = 40, d = 12: 2.5 against 3.9 ms per step).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sk_dev.h"
#include "sk_kernels.h"
#include "sk_lane.h"
#include "sk_quad.h"

namespace sk {
namespace four {

constexpr real kSqrt3 = 1.7320508075688772, kRsqrt12 = 0.28867513459481287;

__device__ __forceinline__ real wave_max(real v)
{
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v = fmax(v, __shfl_xor(v, s));
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)), __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// M: 1 = the block rows of a pair fit one band of 16 lanes, 2 = several bands; TC: whether there is a time channel.
template <int BL, int D, int M, bool TC>
__device__ __forceinline__ void backward(const SweepArgs& a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LP = kWave / kQuadPairs, YS = quad_y_stride(D);
    constexpr int RL = four_rows(BL, D);         // block rows per lane
    using LK = Lock<BL, D, RL>;
    constexpr int C = LK::C, R = C, RR = LK::RR; // RR refined rows per lane
    constexpr int NVS = RR + 1 + C;              // checkpoint: right edge, bottom-left corner, bottom edge but its last value
    static_assert(NVS == four_ckpt_values(BL, D), "checkpoint layout");
    constexpr int GS = four_gring_stride(D);
    const int lane = threadIdx.x;
    const int g = lane >> 4, r = lane & (LP - 1);
    SK_LDS real* ylds = (SK_LDS real*)smem;                       // [q + 1][YS]
    SK_LDS real* gyp = (SK_LDS real*)(smem + a.lk_off_gyp);       // [q][D]: y-side sums of the quad
    // Sixteen columns at a time of what passes between a band and the outside, [group][column & 15][...]: the finished
    // y-side sums of the group's first lane (gring), forward values from below (kring; going forward: out of the last
    // lane), adjoints from below (aring; going forward: forward values from above), adjoints out of the first lane
    // (oring).  A lane moves one of the sixteen columns to or from global memory, so that the wavefront never waits
    // for a store that is still under way when it needs a value it has loaded.
    SK_LDS real* gring0 = (SK_LDS real*)(smem + a.lk_off_gp);
    SK_LDS real* gring = gring0 + g * GS;
    SK_LDS real* kring = (SK_LDS real*)(smem + a.lk_off_krows) + g * (LP * C);
    SK_LDS real* aring = kring + kWave * C;                       // (several bands only)
    SK_LDS real* oring = aring + kWave * C;                       // (several bands only)
    const long slot = blockIdx.x;
    const int nb = a.nb, q = a.q;
    const int ns = M == 1 ? 1 : a.fv_bands;
    const int NT = nb + LP - 1;
    const int nck = a.nseg;                                       // checkpoint places per band, the last for the band's end
    // Scratch of this wavefront.  rows[band][group]: the band's bottom row, node column n at [2 C - 1 + n] (1 up to
    // node column 0); adj[group]: the adjoints that enter a band from below, column J at [J C ...].
    real* const rows = a.rows + slot * a.rows_slot;
    real* const adj0 = a.adj + slot * a.adj_slot;
    real* const ckpt = a.ckpt + slot * a.ckpt_slot;
    const unsigned gRow = g * a.rowlen;
    auto row_of = [&](int s) { return rows + (long)s * kQuadPairs * a.rowlen; };
    for (int s = 0; s < ns; ++s)
        for (int t = r; t < 2 * C; t += LP) row_of(s)[gRow + t] = 1.0;
    for (int t = lane; t < YS; t += kWave) ylds[q * YS + t] = 0.0;   // the row of zeros
    for (int t = lane; t < q * D; t += kWave) gyp[t] = 0.0;

    long cur_y = -1;
    real ylen2 = 0.0;   // largest squared length of a y increment
    QuadQueue queue(a, slot, gridDim.x);
    unsigned out = 0;   // groups of the quad whose pairs drifted
    while (queue.more()) {
        const QuadCursor& cur = queue.cur;
        const long yi = cur.yi;
        if (yi != cur_y) {
            const real* dyg = a.dy + yi * a.ystride;
            for (int t = lane; t < q * D; t += kWave) {
                const int b = t / D, c = t - b * D;
                ylds[b * YS + c] = dyg[(long)b * a.DS + c];
            }
            cur_y = yi;
            ylen2 = 0.0;
            for (int b = lane; b < q; b += kWave) {
                real t = 0.0;
#pragma unroll
                for (int c = 0; c < D; ++c) t = fma(ylds[b * YS + c], ylds[b * YS + c], t);
                ylen2 = fmax(ylen2, t);
            }
            ylen2 = wave_max(ylen2);
        }
        // a group beyond the row's end, or whose pair has drifted: zero increments, no outputs
        const bool inrow = cur.xi0 + g < cur.npr, valid = inrow && ((out >> g) & 1u) == 0;
        const long xi = inrow ? cur.xi0 + g : cur.npr - 1;
        const long pid = a.tri ? xi * a.gramN + yi : xi * a.gramM + yi;
        const long pid2 = a.tri ? yi * a.gramN + xi : pid;

        const real gxs = a.sc * (1.0 / kSqrt3);   // of the x-side sums; the y-side sums hold sc / 2 (through dxr)
        real dxr[RL][D];
        // Increments of the lane's block rows in band s (zeros above the grid).  Returns log2 of the macro-steps between the
        // band's checkpoints, by the largest increment product that a block of the band can have.
        auto load_x = [&](int s) __attribute__((always_inline)) {
            const real* const dxp = a.dx + xi * a.xstride;
            const int I0 = (s * LP + r) * RL - a.lk_padb;
#pragma unroll
            for (int m = 0; m < RL; ++m) {
                const int I = I0 + m;
                const real* xp = dxp + ((I >= 0 ? I : 0) >> a.rs1) * a.DS;
#pragma unroll
                for (int c = 0; c < D; ++c) dxr[m][c] = xp[c];
            }
#pragma unroll
            for (int m = 0; m < RL; ++m) {
                const real sc = valid && I0 + m >= 0 ? a.sc * kRsqrt12 : 0.0;
#pragma unroll
                for (int c = 0; c < D; ++c) dxr[m][c] *= sc;
            }
            real xlen2 = 0.0;
#pragma unroll
            for (int m = 0; m < RL; ++m) {
                real t = 0.0;
#pragma unroll
                for (int c = 0; c < D; ++c) t = fma(dxr[m][c], dxr[m][c], t);
                xlen2 = fmax(xlen2, t);
            }
            const real unit = kRsqrt12 / (C * C) * four_calm_scale(BL, D);   // (the cells of a block share its product)
            const real most2 = wave_max(xlen2) * ylen2;
            return most2 <= (kFourCalm * unit) * (kFourCalm * unit) ? 4 : (most2 <= (kFourSteady * unit) * (kFourSteady * unit) ? 3 : 2);
        };
        // the D increments of the block column the lane is at in macro-step T
        auto fetch = [&](int T, real (&y)[D]) __attribute__((always_inline)) {
            const int b = (int)min((unsigned)(T - r) >> a.rs2, (unsigned)q);   // outside the grid: the row of zeros
            if constexpr (D % 2 == 0) {
                const SK_LDS real2* yp = (const SK_LDS real2*)(ylds + __mul24(b, YS));
#pragma unroll
                for (int c = 0; c < D / 2; ++c) {
                    const real2 v = yp[c];
                    y[2 * c] = v.x;
                    y[2 * c + 1] = v.y;
                }
            } else {
                const SK_LDS real* yp = ylds + __mul24(b, YS);
#pragma unroll
                for (int c = 0; c < D; ++c) y[c] = yp[c];
            }
        };
        // P = p / sqrt(12) of block row m (Eq. (1), third line): with that factor in the x increments A = 1 + P^2 + sqrt(3) P
        // and B = 1 - P^2 take an operation less; tcj: the time channel's constant inside the grid, else 0
        auto inner = [&](int m, int nabove, real tcj, const real (&y)[D]) __attribute__((always_inline)) {
            real t = dxr[m][0] * y[0];
#pragma unroll
            for (int c = 1; c < D; ++c) t = fma(dxr[m][c], y[c], t);
            if constexpr (TC) t += m >= nabove ? tcj : 0.0;
            return t;
        };
        auto tc_at = [&](int T) __attribute__((always_inline)) {
            if constexpr (TC) return valid && (unsigned)(T - r) < (unsigned)nb ? a.tc * kRsqrt12 : 0.0;
            else return 0.0;
        };

        // ---- forward, a checkpoint every 2^ckL macro-steps, every band's bottom row into global scratch ----
        int ckL = 0;   // of the band in work (the last band's serves both sweeps, as its increments do)
        for (int s = 0; s < ns; ++s) {
            ckL = load_x(s);
            const int nabove = a.lk_padb - (s * LP + r) * RL;
            const int Ts = s == 0 ? a.lk_padb / RL : 0;
            real left[RR + 1], bot[C], blc = 1.0;
#pragma unroll
            for (int i = 0; i <= RR; ++i) left[i] = 1.0;
#pragma unroll
            for (int i = 0; i < C; ++i) bot[i] = 1.0;
            const real* const above = row_of(s > 0 ? s - 1 : 0);
            real* const below = row_of(s);
            real* const ck = ckpt + (long)s * nck * NVS * kWave;
            auto store = [&](int k) __attribute__((always_inline)) {
                real* cp = ck + (long)k * NVS * kWave;
#pragma unroll
                for (int i = 0; i <= RR; ++i) cp[i * kWave + lane] = left[i];
                cp[(RR + 1) * kWave + lane] = blc;
#pragma unroll
                for (int i = 0; i + 1 < C; ++i) cp[(RR + 2 + i) * kWave + lane] = bot[i];
            };
            real y[D], pre[C], te[C];   // pre: the lane's column of the next sixteen of the row above; te: the next top edge
            auto load_above = [&](int J) __attribute__((always_inline)) {   // (beyond the grid: anything finite)
#pragma unroll
                for (int cc = 0; cc < C; ++cc) pre[cc] = ld_scratch(above + (gRow + 2 * C + min(J + r, nb - 1) * C + cc));
            };
            auto next_edge = [&](int T) __attribute__((always_inline)) {
                if ((T & (LP - 1)) == 0) {
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) aring[r * C + cc] = pre[cc];
                    load_above(T + LP);
                }
#pragma unroll
                for (int cc = 0; cc < C; ++cc) te[cc] = aring[(T & (LP - 1)) * C + cc];
            };
#pragma unroll
            for (int cc = 0; cc < C; ++cc) te[cc] = 1.0;
            if (M > 1 && s > 0) {
                load_above(0);
                next_edge(0);
            }
            fetch(Ts, y);
            for (int k = Ts >> ckL; k << ckL < NT; ++k) {
                if (k << ckL > Ts) store(k - 1);
                const int T0 = max(Ts, k << ckL), T1 = min(NT, (k + 1) << ckL);
                for (int T = T0; T < T1; ++T) {
                    const real tcj = tc_at(T);
                    real p[RL];
#pragma unroll
                    for (int m = 0; m < RL; ++m) p[m] = inner(m, nabove, tcj, y);
                    fetch(T + 1, y);
                    real top[C + 1];
                    top[0] = left[0];
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) top[cc + 1] = row_from_above_or(bot[cc], te[cc]);
                    left[0] = top[C];
                    if (M > 1 && s > 0) next_edge(T + 1);
#pragma unroll
                    for (int m = 0; m < RL; ++m) {
                        const real Bc = fma(-p[m], p[m], 1.0), Ac = fma(p[m], kSqrt3, fma(p[m], p[m], 1.0));
#pragma unroll
                        for (int rb = 0; rb < R; ++rb) {
                            const int rr = m * R + rb;
                            real now[C + 1];
                            now[0] = left[rr + 1];
#pragma unroll
                            for (int cc = 0; cc < C; ++cc) now[cc + 1] = fma(now[cc] + top[cc + 1], Ac, -(top[cc] * Bc));
                            left[rr + 1] = now[C];
#pragma unroll
                            for (int cc = 0; cc <= C; ++cc) top[cc] = now[cc];
                        }
                    }
                    blc = top[0];
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) bot[cc] = top[cc + 1];
                    const int J15 = (T + 1) & (LP - 1);   // the last lane's column, mod 16
                    if (r == LP - 1) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) kring[J15 * C + cc] = bot[cc];
                    }
                    if (T >= LP - 1 && (J15 == LP - 1 || T == NT - 1)) {
                        const int J = ((T - (LP - 1)) & ~(LP - 1)) + r;
                        if (J < nb) {
#pragma unroll
                            for (int cc = 0; cc < C; ++cc) below[gRow + 2 * C + J * C + cc] = kring[r * C + cc];
                        }
                    }
                }
            }
            store(nck - 1);
            if (s == ns - 1 && r == LP - 1 && valid && a.k_out) {
                a.k_out[pid] = bot[C - 1];
                a.k_out[pid2] = bot[C - 1];
            }
            scratch_fence();   // the next band reads this one's bottom row, the reverse sweep the checkpoints
        }

        // ---- reverse ----
        bool drift = false;
        const real gk = valid ? gram_weight(a, pid, pid2) : 0.0;   // dF/dk[m, n]: enters under the last lane
        for (int s = ns - 1; s >= 0; --s) {
            if (s < ns - 1) ckL = load_x(s);
            const int nabove = a.lk_padb - (s * LP + r) * RL;
            const int Ts = s == 0 ? a.lk_padb / RL : 0;
            real kR[RR + 1], accL[RR + 1], ktop[C], up[C], corner = 0.0, kscale = 1.0;
            real gacc[RL][D], gtr[D];
#pragma unroll
            for (int i = 0; i <= RR; ++i) { kR[i] = 1.0; accL[i] = 0.0; }
#pragma unroll
            for (int i = 0; i < C; ++i) { ktop[i] = 1.0; up[i] = 0.0; }
#pragma unroll
            for (int c = 0; c < D; ++c) gtr[c] = 0.0;
#pragma unroll
            for (int m = 0; m < RL; ++m)
#pragma unroll
                for (int c = 0; c < D; ++c) gacc[m][c] = 0.0;
            const real* const krow = row_of(s);
            const real* const ck = ckpt + (long)s * nck * NVS * kWave;
            const int laneup = r > 0 ? lane - 1 : lane;   // the bottom edge of the lane above travels with this lane's top edge
            auto restore = [&](int k, bool check) __attribute__((always_inline)) {
                const real* cp = ck + (long)k * NVS * kWave;
                real v[NVS];
#pragma unroll
                for (int i = 0; i <= RR; ++i) v[i] = ld_scratch(cp + (i * kWave + lane));
#pragma unroll
                for (int i = RR + 1; i < NVS; ++i) v[i] = ld_scratch(cp + (i * kWave + laneup));
#pragma unroll
                for (int i = 0; i <= RR; ++i) kscale = fmax(kscale, fabs(v[i]));
                if (check) {
#pragma unroll
                    for (int i = 0; i <= RR; ++i)   // written so that a NaN counts as drift
                        if (!(fabs(kR[i] - v[i]) <= kFourDriftTol * kscale)) drift = true;
                }
#pragma unroll
                for (int i = 0; i <= RR; ++i) kR[i] = v[i];
#pragma unroll
                for (int i = 0; i < C; ++i) ktop[i] = v[RR + 1 + i];
            };
            // the lane's column of the next sixteen of the row below (left of the grid: ones and zeros), and
            // what the last lane receives from below in the next macro-step
            real y[D], prek[C], prea[C], ek[C], ea[C];
            auto load_below = [&](int J0) __attribute__((always_inline)) {
                const int J = J0 + r;
#pragma unroll
                for (int cc = 0; cc < C; ++cc) { prek[cc] = 1.0; prea[cc] = 0.0; }
                if (J >= 0 && J < nb) {
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) prek[cc] = ld_scratch(krow + (gRow + 2 * C - 1 + J * C + cc));
                    if (M > 1 && s < ns - 1) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) prea[cc] = ld_scratch(adj0 + (gRow + J * C + cc));
                    }
                }
            };
            auto next_edge = [&](int T) __attribute__((always_inline)) {
                const int J15 = (T + 1) & (LP - 1);   // the last lane's column, mod 16
                if (J15 == LP - 1 || T == NT - 1) {
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) kring[r * C + cc] = prek[cc];
                    if (M > 1) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) aring[r * C + cc] = prea[cc];
                    }
                    load_below(((T - (LP - 1)) & ~(LP - 1)) - LP);
                }
#pragma unroll
                for (int cc = 0; cc < C; ++cc) {
                    ek[cc] = kring[J15 * C + cc];
                    ea[cc] = M > 1 ? aring[J15 * C + cc] : 0.0;
                }
            };
            load_below((nb - 1) & ~(LP - 1));
            next_edge(NT - 1);
            if (s == ns - 1) ea[C - 1] = gk;
            fetch(NT - 1, y);
            for (int k = (NT - 1) >> ckL; (k + 1) << ckL > Ts; --k) {
                const int T0 = max(Ts, k << ckL), T1 = min(NT, (k + 1) << ckL);
                restore(T1 == NT ? nck - 1 : k, T1 != NT);
                for (int T = T1 - 1; T >= T0; --T) {
                    real yn[D];
                    fetch(T - 1, yn);
                    const real tcj = tc_at(T);
                    real eb[C + 1], gb[C + 1];   // forward values and adjoints along the lower edge of a row of cells
                    gb[0] = 0.0;
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) {
                        eb[cc] = row_from_below_or(ktop[cc], ek[cc]);
                        gb[cc + 1] = row_from_below_or(up[cc], ea[cc]);
                    }
                    eb[C] = kR[RR];
                    gb[C] += accL[RR];
                    next_edge(T - 1);
#pragma unroll
                    for (int c = 0; c < D; ++c) gtr[c] = row_from_below(gtr[c]);
#pragma unroll
                    for (int m = RL - 1; m >= 0; --m) {
                        __builtin_amdgcn_sched_barrier(0);   // block by block: the lane state leaves no room
                        const real p = inner(m, nabove, tcj, y);
                        const real Bc = fma(-p, p, 1.0), r0 = fma(p, p, 1.0), Ac = fma(p, kSqrt3, r0);
                        const real ee = fma(-Bc, r0, 1.0), r1 = fma(ee, r0, r0);
                        const real iB = fma(ee * ee, r1, r1);   // 1 / B = r0 (1 + ee) (1 + ee^2 ...), see coef_rev in sk_lane.h
                        real gs = 0.0, gq = 0.0;
#pragma unroll
                        for (int rb = R - 1; rb >= 0; --rb) {
                            const int rr = m * R + rb;
                            real et[C + 1], gt[C + 1];
                            et[C] = kR[rr];
                            gt[C] = rr > 0 ? accL[rr] : corner;
#pragma unroll
                            for (int cc = C - 1; cc >= 0; --cc) {
                                const real sum = eb[cc] + et[cc + 1];
                                et[cc] = fma(sum, Ac, -eb[cc + 1]) * iB;   // Eq. (1) solved for its oldest term
                                const real go = gb[cc + 1];
                                gb[cc] = fma(go, Ac, gb[cc]);
                                gt[cc + 1] = fma(go, Ac, gt[cc + 1]);
                                gt[cc] = -(go * Bc);
                                const bool first = rb == R - 1 && cc == C - 1;
                                gs = first ? go * sum : fma(go, sum, gs);
                                gq = first ? go * et[cc] : fma(go, et[cc], gq);
                            }
                            kR[rr + 1] = eb[0];
                            accL[rr + 1] = gb[0];
#pragma unroll
                            for (int cc = 0; cc <= C; ++cc) { eb[cc] = et[cc]; gb[cc] = gt[cc]; }
                        }
                        // sqrt(3) dF/dp: A'(p) = P / sqrt(3) + 1/2, -B'(p) = P / sqrt(3); then the linear map of Section 3.4
                        // (the factors are taken back where the sums leave)
                        const real gp = fma(p, gs + gq, gs * (0.5 * kSqrt3));
#pragma unroll
                        for (int c = 0; c < D; ++c) {
                            gacc[m][c] = fma(gp, y[c], gacc[m][c]);
                            gtr[c] = fma(gp, dxr[m][c], gtr[c]);
                        }
                    }
                    kR[0] = eb[0];
                    corner = gb[0];
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) { up[cc] = gb[cc + 1]; ktop[cc] = eb[cc]; }
#pragma unroll
                    for (int c = 0; c < D; ++c) y[c] = yn[c];
                    // the group's first lane with rows has seen all of column col = T - Ts
                    const int col = T - Ts, c15 = col & (LP - 1);
                    if (r == Ts) {
#pragma unroll
                        for (int c = 0; c < D; ++c) gring[c15 * D + c] = gtr[c];
                        if (M > 1 && s > 0) {
#pragma unroll
                            for (int cc = 0; cc < C; ++cc) oring[c15 * C + cc] = up[cc];
                        }
                    }
                    if (c15 == 0 && col < nb) {   // sixteen columns (or the last few) are complete
                        for (int t = lane; t < min(LP, nb - col) * D; t += kWave) {
                            const real sum = (gring0[t] + gring0[GS + t]) + (gring0[2 * GS + t] + gring0[3 * GS + t]);
                            if (a.rs2 == 0) gyp[col * D + t] += sum;
                            else lds_atomic_add(gyp + ((col + t / D) >> a.rs2) * D + t % D, sum);
                        }
                        if (M > 1 && s > 0 && col + r < nb) {
#pragma unroll
                            for (int cc = 0; cc < C; ++cc) adj0[gRow + (col + r) * C + cc] = oring[r * C + cc];
                        }
                    }
                }
            }
            // the left end: the sweep started from the boundary value 1 in every lane
#pragma unroll
            for (int i = 0; i <= RR; ++i)
                if (!(fabs(kR[i] - 1.0) <= kFourDriftTol * kscale)) drift = true;
            // the x-side sums wait for the verdict on the whole pair: in registers if this is the only band
            if constexpr (M > 1) {
                real* gsp = a.fv_gx + slot * a.fv_gx_slot + (long)s * RL * D * kWave;
#pragma unroll
                for (int m = 0; m < RL; ++m)
#pragma unroll
                    for (int c = 0; c < D; ++c) gsp[(m * D + c) * kWave + lane] = gacc[m][c];
                scratch_fence();   // (the next band also reads the adjoints this one handed up)
            } else if (__ballot(drift && valid) == 0ull && a.want_gx && valid) {
                real* const gx = a.gdx + xi * a.xstride;
#pragma unroll
                for (int m = 0; m < RL; ++m) {
                    const int I = r * RL + m - a.lk_padb;
                    if (I >= 0) {
#pragma unroll
                        for (int c = 0; c < D; ++c) unsafeAtomicAdd(gx + (I >> a.rs1) * a.DS + c, gacc[m][c] * gxs);
                    }
                }
            }
        }
        // A pair that drifted: nothing of it is kept, and the quad is done again with zeros in its place.
        const unsigned long long bad = __ballot(drift && valid);
        if (bad != 0ull) {
            if (r == 0 && ((bad >> (16 * g)) & 0xffffull) != 0ull) list_drifted(a, pid, pid2);
            for (int i = 0; i < kQuadPairs; ++i) out |= ((bad >> (16 * i)) & 0xffffull) != 0ull ? 1u << i : 0u;
            for (int t = lane; t < q * D; t += kWave) gyp[t] = 0.0;
            if (__ballot(inrow && ((out >> g) & 1u) == 0) != 0ull) continue;
            // (no pair of the quad is left: nothing to sweep again)
        } else {
            if (M > 1 && a.want_gx && valid) {
                real* const gx = a.gdx + xi * a.xstride;
                for (int s = 0; s < ns; ++s) {
                    const real* gsp = a.fv_gx + slot * a.fv_gx_slot + (long)s * RL * D * kWave;
#pragma unroll
                    for (int m = 0; m < RL; ++m) {
                        const int I = (s * LP + r) * RL + m - a.lk_padb;
                        if (I >= 0) {
#pragma unroll
                            for (int c = 0; c < D; ++c)
                                unsafeAtomicAdd(gx + (I >> a.rs1) * a.DS + c, ld_scratch(gsp + ((m * D + c) * kWave + lane)) * gxs);
                        }
                    }
                }
            }
            if (a.want_gy) {
                real* gdy = a.gdy + yi * a.ystride;
                for (int t = lane; t < q * D; t += kWave) {
                    const int b = t / D, c = t - b * D;
                    unsafeAtomicAdd(&gdy[(long)b * a.DS + c], 2.0 * gyp[t]);
                    gyp[t] = 0.0;
                }
            } else {
                for (int t = lane; t < q * D; t += kWave) gyp[t] = 0.0;
            }
        }
        out = 0;
        queue.next(a);
    }
}

// OCC: wavefronts per SIMD the registers are allotted for.  Calls with a time channel have kernels of their own: together in
// one kernel the two copies of the sweep cost each other registers.
template <int BL, int D, int M, bool TC, int OCC>
__global__ __launch_bounds__(kWave, OCC) void four_bwd_kernel(SweepArgs a)
{
    backward<BL, D, M, TC>(a);
}

// ------------------------------------------------------------------------------------------------
// launcher
// ------------------------------------------------------------------------------------------------
template <int BL, int D, int M>
static hipError_t launch_t(const SweepArgs& a, int grid, size_t lds, hipStream_t st)
{
    if constexpr (four_occupancy(BL, D) > 0) {
        auto kernel = a.tc != 0.0 ? &four_bwd_kernel<BL, D, M, true, four_occupancy(BL, D)>
                                  : &four_bwd_kernel<BL, D, M, false, four_occupancy(BL, D)>;
        if (hipError_t e = allow_full_lds(reinterpret_cast<const void*>(kernel)); e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kWave), lds, st, a);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

template <int BL, int D>
static hipError_t launch_m(const SweepArgs& a, int grid, size_t lds, hipStream_t st)
{
    return a.lk_M == 1 ? launch_t<BL, D, 1>(a, grid, lds, st) : launch_t<BL, D, 2>(a, grid, lds, st);
}

template <int BL>
static hipError_t launch_bl(int DT, const SweepArgs& a, int grid, size_t lds, hipStream_t st)
{
    switch (DT) {
        case 2: return launch_m<BL, 2>(a, grid, lds, st);
        case 3: return launch_m<BL, 3>(a, grid, lds, st);
        case 4: return launch_m<BL, 4>(a, grid, lds, st);
        case 5: return launch_m<BL, 5>(a, grid, lds, st);
        case 6: return launch_m<BL, 6>(a, grid, lds, st);
        case 8: return launch_m<BL, 8>(a, grid, lds, st);
        case 12: return launch_m<BL, 12>(a, grid, lds, st);
        case 16: return launch_m<BL, 16>(a, grid, lds, st);
        default: return hipErrorInvalidValue;
    }
}
}  // namespace four

hipError_t launch_sweep_four(int BL, int DT, const SweepArgs& a, int grid, size_t lds, hipStream_t st)
{
    // what the kernel assumes about the launch
    if (four_occupancy(BL, DT) == 0) return hipErrorInvalidValue;
    const int lanerows = four_rows(BL, DT), bands = a.fv_bands, C = 1 << BL;
    const size_t rings = (size_t)(a.lk_M == 1 ? 1 : 3) * kWave * C * sizeof(real);
    if (!a.gramM || !a.bd_flags || a.qd_even < 0 || a.ll != 0 || a.lk_phase != 0 || bands < 1 || a.lk_M != (bands == 1 ? 1 : 2) || a.mb < 1 || a.nb < 1 ||
        a.lk_padb != bands * 16 * lanerows - a.mb || a.lk_padb < 0 || a.lk_padb >= 16 * lanerows || a.DS < DT || a.d > DT ||
        a.qd_nquads < 1 || a.nb != a.q << a.rs2 || a.mb != a.r << a.rs1 ||
        a.nseg < (a.nb + 14) / kFourCkpt + 1 || a.rowlen < (a.nb + 2) * C || !a.bad_list || !a.bad_count ||
        a.rows_slot < (long)bands * kQuadPairs * a.rowlen || a.adj_slot < (long)kQuadPairs * a.rowlen ||
        a.ckpt_slot < (long)bands * a.nseg * four_ckpt_values(BL, DT) * kWave ||
        (bands > 1 && (!a.fv_gx || a.fv_gx_slot < (long)bands * lanerows * DT * kWave)) ||
        a.lk_off_gyp < (size_t)(a.q + 1) * quad_y_stride(DT) * sizeof(real) ||
        a.lk_off_gp < a.lk_off_gyp + (size_t)a.q * DT * sizeof(real) ||
        a.lk_off_krows < a.lk_off_gp + (size_t)kQuadPairs * four_gring_stride(DT) * sizeof(real) ||
        a.lk_off_krows + rings > lds)
        return hipErrorInvalidValue;
    switch (BL) {
        case 0: return four::launch_bl<0>(DT, a, grid, lds, st);
        case 1: return four::launch_bl<1>(DT, a, grid, lds, st);
        case 2: return four::launch_bl<2>(DT, a, grid, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sk
