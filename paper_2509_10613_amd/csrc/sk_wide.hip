// Wide kernels (gfx950): any channel count, any number of strips.  For paths of more channels than the other kernels hold
// in registers (above 16), and backward, whatever the channel count, where the y increments and their sums do not fit in LDS
// or the cooperative kernels would hold sixteen channels (wide_pays).
//
// The contraction over the channels is taken out of the sweeps altogether: the wave that owns a strip of 64 block rows
// first writes p of Eq. (1) for every block of the strip into its scratch, formed on the matrix cores
// (v_mfma_f64_16x16x4_f64, sixteen rows by sixteen columns, four channels per instruction), in the order in which the sweep
// reads it: entry [T][lane] belongs to block column T - lane, so a macro-step is one coalesced load, and what lies outside
// the grid is stored as zero (A = B = 1 there, so no lane is masked).  The sweep then costs the same for every channel
// count.  Backward, the forward sweep also stores each block's right and bottom edge, so the reverse sweep needs no
// division, no checkpoint and no second try; dF/dp replaces p in place, and the linear map of Section 3.4 is two more
// contractions on the matrix cores.
//
// What bounds it: the scratch, (1 + 2^(BL+1) - 1) doubles per block written and read once or twice each.  Counters, backward, 59 x
// 106 pairs of 231 x 163 cells, d = 10: 25.4 GB in 6.8 ms, 3.7 TB/s where a copy reads and writes 4.6; vector instructions take a
// tenth of the issue slots.  Forward, 66 x 593 pairs, d = 19, order 1: 14.0 GB in 4.85 ms.  What it replaces looped over the
// channels of every block in memory, with an atomic addition per block, channel and side (measured, both sides: in front of
// wide_pays in sk_plan.h).
//
// Strips: strip s + 1 follows strip s at a fixed lag of macro-steps, one strip per wave, nw of them in a workgroup that
// advances in chunks separated by barriers; strips beyond that take further rounds.  With enough pairs to fill the chip a
// workgroup is one wave (nw = 1), which takes the strips of its pair one after the other and meets no barrier.  Every
// wave runs the same number of iterations, so every barrier is met by all of them and nothing is ever polled.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sk_dev.h"
#include "sk_kernels.h"
#include "sk_lane.h"

namespace sk {

typedef double real4w __attribute__((ext_vector_type(4)));

template <int BL, int LL>
struct Wide {
    using LK = Lock<BL, 1, 1, LL>;
    static constexpr int C = 1 << BL, R = 1 << BL;
    static constexpr int NV = wide_edge_values(BL);     // right edge (R values, the corner last), then the bottom edge without the corner
    static constexpr int CH = wide_chunk(BL);           // macro-steps per chunk
    // A strip reads its upper (reverse: lower) neighbour's row one chunk ahead: 64 lanes and two chunks behind it.
    static constexpr int LAG = (2 * CH + 62) / CH + 1;
    static constexpr int kFeed = CH * C + 1;            // values a chunk takes from a neighbour's row
};

// Waits for this wave's stores as well: the rows that cross waves are in global memory.
__device__ __forceinline__ void wide_barrier(int nw)
{
    if (nw > 1) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// p of strip s, [T][lane].
template <bool LL2>
__device__ __forceinline__ void wide_form_p(const SweepArgs& a, int s, int lane, const real* dx, const real* dy, real* P)
{
    const int n16 = lane & 15, g16 = lane >> 4;
    const int NT = a.lk_NT, nb = a.nb, d = a.d;
    const int Ibase = s * kWave - a.lk_padb;   // block row of lane 0; negative above the grid
    const int jt1 = (NT + 15) >> 4;
    // operand rows: lane l supplies row l % 16 of each of the four row tiles, channel 4 k + l / 16
    const real* xr[4];
    bool xok[4];
#pragma unroll
    for (int I = 0; I < 4; ++I) {
        const int row = Ibase + 16 * I + n16;
        xok[I] = row >= 0;
        xr[I] = dx + (long)((row >= 0 ? row : 0) >> a.rs1) * a.DS;
    }
    for (int jt = -4; jt < jt1; ++jt) {
        real4w acc[4];
#pragma unroll
        for (int I = 0; I < 4; ++I) acc[I] = real4w{0.0, 0.0, 0.0, 0.0};
        if (jt >= 0 && 16 * jt < nb) {
            const int J = 16 * jt + n16;
            const bool yok = J < nb;
            const real* yr = dy + (long)((yok ? J : nb - 1) >> a.rs2) * a.DS;
            for (int c0 = 0; c0 < d; c0 += 8) {
                real xv[2][4], yv[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = c0 + 4 * u + g16;
                    const int cc = c < d ? c : d - 1;
                    yv[u] = yr[cc];
#pragma unroll
                    for (int I = 0; I < 4; ++I) xv[u][I] = xr[I][cc];
                    if (!(yok && c < d)) yv[u] = 0.0;
#pragma unroll
                    for (int I = 0; I < 4; ++I) xv[u][I] = (xok[I] && c < d) ? xv[u][I] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int I = 0; I < 4; ++I) acc[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[u][I], yv[u], acc[I], 0, 0, 0);
            }
        }
        // result register r of lane l: row 16 I + l / 16 + 4 r, column 16 jt + l % 16
        const int J = 16 * jt + n16;
#pragma unroll
        for (int I = 0; I < 4; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int lr = 16 * I + g16 + 4 * r, T = J + lr, row = Ibase + lr;
                const bool in = row >= 0 && (unsigned)J < (unsigned)nb;
                real v = in ? fma(acc[I][r], a.sc, a.tc) : 0.0;
                if constexpr (LL2) {   // off the diagonal of the lead-lag level: the time channel's constant alone
                    if (in && (((row >> (a.rs1 - 1)) ^ (J >> (a.rs2 - 1))) & 1)) v = a.tc;
                }
                if ((unsigned)T < (unsigned)NT) P[(long)T * kWave + lr] = v;
            }
    }
}

// ------------------------------------------------------------------------------------------------
// forward sweep of the strips of one pair (EDGES: the blocks' edges are stored for the reverse sweep)
// ------------------------------------------------------------------------------------------------
template <int BL, int LL, bool EDGES>
__device__ __forceinline__ void wide_forward(const SweepArgs& a, int w, int nw, int lane, const real* Pall, real* Vall, real* rows,
                                             SK_LDS real* feed)
{
    using W = Wide<BL, LL>;
    using LK = typename W::LK;
    constexpr int C = W::C, R = W::R, CH = W::CH, NV = W::NV, LAG = W::LAG;
    const int NT = a.lk_NT, ns = a.lk_ns, nck = NT / CH;
    const int nbx = NT - (kWave - 1);   // block columns a strip's last lane visits
    for (int s0 = 0; s0 < ns; s0 += nw) {
        const int s = s0 + w;
        const bool active = s < ns;
        const int nsw = min(nw, ns - s0);
        const int niter = nck + (nsw - 1) * LAG;
        const real* P = Pall + (long)s * NT * kWave + lane;
        real* V = EDGES ? Vall + ((long)s * (NT + 2) + 2) * NV * kWave + lane : nullptr;
        const real* above = s > 0 ? rows + (long)(s - 1) * a.rowlen : nullptr;
        real* row = rows + (long)s * a.rowlen;
        typename LK::Fwd f;
        typename LK::Off off;
        f.init();
        off.setup(a, active ? s : 0, lane);
        real pq[CH];
        real ev = 1.0;
#pragma unroll
        for (int i = 0; i < CH; ++i) pq[i] = 0.0;
        auto load_edge = [&](int c) {   // lane q: node q % C of block column c CH + q / C of the row above
            const int col = c * CH + lane / C;
            return (above && lane < CH * C && col < nbx) ? ld_scratch(above + (long)col * C + 1 + lane % C) : 1.0;
        };
        for (int g = -1; g < niter; ++g) {
            const int c = g - w * LAG;
            if (active && c == -1) {
#pragma unroll
                for (int i = 0; i < CH; ++i) pq[i] = ld_scratch(P + i * kWave);
                ev = load_edge(0);
            }
            if (active && c >= 0 && c < nck) {
                if (lane < CH * C) feed[lane] = ev;
                __builtin_amdgcn_wave_barrier();
                const int T0 = c * CH;
                const real* pn = P + (long)(c + 1 < nck ? T0 + CH : T0) * kWave;   // (past the end: read again, unused)
                ev = load_edge(c + 1);
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const real p = pq[i];
                    pq[i] = ld_scratch(pn + i * kWave);
                    real Ac[1], Bc[1], A0[1], B0[1];
                    LK::coef_fwd(p, Ac[0], Bc[0]);
                    if constexpr (LL == 1) off.at(T0 + i, A0, B0);
                    else { A0[0] = Ac[0]; B0[0] = Bc[0]; }
                    real recv[C];
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) recv[cc] = wave_from_above_or(f.bot[cc], feed[i * C + cc]);
                    f.step(recv, Ac, Bc, A0, B0);
                    if constexpr (EDGES) {
                        real* vp = V + (long)(T0 + i) * NV * kWave;
#pragma unroll
                        for (int rr = 0; rr < R; ++rr) vp[rr * kWave] = f.left[rr + 1];
#pragma unroll
                        for (int cc = 0; cc + 1 < C; ++cc) vp[(R + cc) * kWave] = f.bot[cc];
                    }
                    const int Jw = T0 + i - (kWave - 1);
                    if (lane == kWave - 1 && Jw >= 0) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) row[(long)Jw * C + 1 + cc] = f.bot[cc];
                    }
                }
            }
            wide_barrier(nw);
        }
        scratch_fence();
    }
}

template <int BL, int LL>
__device__ __forceinline__ void wide_fwd(const SweepArgs& a)
{
    using W = Wide<BL, LL>;
    __shared__ real feeds[kWideMaxWaves][2 * W::kFeed + 1];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = a.nw;
    const int ns = a.lk_ns;
    real* rows = a.rows + (long)blockIdx.x * a.rows_slot;
    real* P = a.wd_scratch + (long)blockIdx.x * a.wd_slot;
    SK_LDS real* feed = (SK_LDS real*)&feeds[w][0];
    for (long q = blockIdx.x; q < a.npairs; q += gridDim.x) {
        long xi, yi, pid, pid2;
        gram_pair(a, q, xi, yi, pid, pid2);
        for (int s = w; s < ns; s += nw) {
            if (a.ll == 2) wide_form_p<true>(a, s, lane, a.dx + xi * a.xstride, a.dy + yi * a.ystride, P + (long)s * a.lk_NT * kWave);
            else wide_form_p<false>(a, s, lane, a.dx + xi * a.xstride, a.dy + yi * a.ystride, P + (long)s * a.lk_NT * kWave);
        }
        scratch_fence();
        wide_forward<BL, LL, false>(a, w, nw, lane, P, nullptr, rows, feed);
        if (threadIdx.x == 0) {
            const real k = ld_scratch(rows + (long)(ns - 1) * a.rowlen + (long)a.nb * W::C);
            a.k_out[pid] = k;
            if (pid2 != pid) a.k_out[pid2] = k;
        }
        wide_barrier(nw);   // the rows are about to be written again
    }
}

template <int BL, int LL>
__global__ __launch_bounds__(kWideMaxWaves* kWave, 2) void wide_fwd_kernel(SweepArgs a) { wide_fwd<BL, LL>(a); }

// ------------------------------------------------------------------------------------------------
// backward: forward sweep with the blocks' edges stored, reverse sweep, linear map
// ------------------------------------------------------------------------------------------------
// One reverse step on a block: the forward values of its nodes from the stored left edge (el), top edge (et) and corner,
// Eq. (1) inside; the adjoint recurrence and dF/dp as in Lock::Rev::step.
template <int BL, int LL>
struct WideRev {
    using W = Wide<BL, LL>;
    using LK = typename W::LK;
    static constexpr int C = W::C, R = W::R;
    real accL[R + 1];   // partial adjoints of the left edge nodes (index 0 unused)
    real corner;        // partial adjoint of the top-left node
    real up[C];         // adjoint contributions to the top edge nodes, handed to the lane above

    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int i = 0; i <= R; ++i) accL[i] = 0.0;
#pragma unroll
        for (int i = 0; i < C; ++i) up[i] = 0.0;
        corner = 0.0;
    }
    __device__ __forceinline__ real step(real ec, const real (&et)[C], const real (&el)[R], const real (&recv)[C], real p, real Ac,
                                         real Bc, real A0, real B0)
    {
        real e[R + 1][C + 1], gn[R + 1][C + 1];
        e[0][0] = ec;
#pragma unroll
        for (int cc = 0; cc < C; ++cc) e[0][cc + 1] = et[cc];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) e[rr + 1][0] = el[rr];
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int cc = 0; cc < C; ++cc) {
                const bool o = LK::cell_off(rr, cc);
                e[rr + 1][cc + 1] = fma(e[rr + 1][cc] + e[rr][cc + 1], o ? A0 : Ac, -(e[rr][cc] * (o ? B0 : Bc)));
            }
#pragma unroll
        for (int rr = 0; rr <= R; ++rr)
#pragma unroll
            for (int cc = 0; cc <= C; ++cc) gn[rr][cc] = 0.0;
#pragma unroll
        for (int rr = 1; rr <= R; ++rr) gn[rr][C] = accL[rr];
#pragma unroll
        for (int cc = 0; cc < C; ++cc) gn[R][cc + 1] += recv[cc];
        gn[0][C] = corner;
        real gs = 0.0, gk = 0.0;
#pragma unroll
        for (int rr = R - 1; rr >= 0; --rr)
#pragma unroll
            for (int cc = C - 1; cc >= 0; --cc) {
                const bool o = LK::cell_off(rr, cc);
                const real Aq = o ? A0 : Ac, Bq = o ? B0 : Bc;
                const real go = gn[rr + 1][cc + 1];
                gn[rr + 1][cc] = fma(go, Aq, gn[rr + 1][cc]);
                gn[rr][cc + 1] = fma(go, Aq, gn[rr][cc + 1]);
                gn[rr][cc] = fma(-go, Bq, gn[rr][cc]);
                if (o) continue;
                gs = fma(go, e[rr + 1][cc] + e[rr][cc + 1], gs);
                gk = fma(go, e[rr][cc], gk);
            }
#pragma unroll
        for (int cc = 0; cc < C; ++cc) up[cc] = gn[0][cc + 1];
        corner = gn[0][0];
#pragma unroll
        for (int rr = 1; rr <= R; ++rr) accL[rr] = gn[rr][0];
        const real p6 = p * (1.0 / 6.0);
        return fma(gs, p6 + 0.5, gk * p6);   // A'(p) = p / 6 + 1 / 2, -B'(p) = p / 6
    }
};

template <int BL, int LL>
__device__ __forceinline__ void wide_reverse(const SweepArgs& a, int w, int nw, int lane, real* Pall, const real* Vall, real* rows,
                                             real gk, SK_LDS real* feed)
{
    using W = Wide<BL, LL>;
    using LK = typename W::LK;
    constexpr int C = W::C, R = W::R, CH = W::CH, NV = W::NV, LAG = W::LAG, kFeed = W::kFeed;
    const int NT = a.lk_NT, ns = a.lk_ns, nck = NT / CH, nb = a.nb;
    const int nbx = NT - (kWave - 1);
    SK_LDS real* feed2 = feed + kFeed;
    for (int s0 = (ns - 1) / nw * nw; s0 >= 0; s0 -= nw) {
        const int s = s0 + w;
        const bool active = s < ns;
        const int nsw = min(nw, ns - s0);
        const int niter = nck + (nsw - 1) * LAG;
        const int lead = (nsw - 1 - w) * LAG;   // the round's last strip starts
        real* P = Pall + (long)s * NT * kWave + lane;
        const real* V = Vall + ((long)s * (NT + 2) + 2) * NV * kWave + lane;
        // The row above holds the forward values under the upper strip; the adjoint that this strip hands up replaces them
        // node by node, once they have been read.
        real* above = s > 0 ? rows + (long)(s - 1) * a.rowlen : nullptr;
        const real* below = s < ns - 1 ? rows + (long)s * a.rowlen : nullptr;
        WideRev<BL, LL> rv;
        typename LK::Off off;
        rv.init();
        off.setup(a, active ? s : 0, lane);
        real pq[CH], vq[CH][NV];
        real ek = 1.0, ea = 0.0;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            pq[i] = 0.0;
#pragma unroll
            for (int v = 0; v < NV; ++v) vq[i][v] = 1.0;
        }
        // lane q: forward value at node q of the row above from block column T0 on
        auto load_above = [&](int T0) {
            const int node = T0 * C + lane;
            return (above && lane < kFeed && node > 0 && node <= nbx * C) ? ld_scratch(above + node) : 1.0;
        };
        // lane q: what the strip below adds to node 1 + q % C of block column T0 - 63 + q / C
        auto load_below = [&](int T0) {
            const int J = T0 - (kWave - 1) + lane / C;
            if (lane >= CH * C || (unsigned)J >= (unsigned)nb) return 0.0;
            if (!below) return s == ns - 1 && J == nb - 1 && lane % C == C - 1 ? gk : 0.0;
            return ld_scratch(below + (long)J * C + 1 + lane % C);
        };
        for (int g = -1; g < niter; ++g) {
            const int rc = g - lead;
            if (active && rc == -1) {
                const int T0 = (nck - 1) * CH;
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    pq[i] = ld_scratch(P + (long)(T0 + i) * kWave);
#pragma unroll
                    for (int v = 0; v < NV; ++v) vq[i][v] = ld_scratch(V + ((long)(T0 + i - 1) * NV + v) * kWave);
                }
                ek = load_above(T0);
                ea = load_below(T0);
            }
            if (active && rc >= 0 && rc < nck) {
                const int T0 = (nck - 1 - rc) * CH;
                if (lane < kFeed) feed[lane] = ek;
                if (lane < CH * C) feed2[lane] = ea;
                __builtin_amdgcn_wave_barrier();
                const int Tn = T0 >= CH ? T0 - CH : 0;   // (past the end: read again, unused)
                ek = load_above(Tn);
                ea = load_below(T0 - CH);
                real* pt = P + (long)T0 * kWave;
                const real* pn = P + (long)Tn * kWave;
                const real* vn = V + (long)(Tn - 1) * NV * kWave;
#pragma unroll
                for (int i = CH - 1; i >= 0; --i) {
                    const real p = pq[i];
                    pq[i] = ld_scratch(pn + i * kWave);
                    real el[R], et[C], recv[C];
#pragma unroll
                    for (int rr = 0; rr < R; ++rr) el[rr] = vq[i][rr];
                    real Ac[1], Bc[1], A0[1], B0[1];
                    LK::coef_fwd(p, Ac[0], Bc[0]);
                    if constexpr (LL == 1) off.at(T0 + i, A0, B0);
                    else { A0[0] = Ac[0]; B0[0] = Bc[0]; }
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) {
                        et[cc] = wave_from_above_or(cc + 1 < C ? vq[i][R + (cc + 1 < C ? cc : 0)] : vq[i][R - 1], feed[i * C + cc + 1]);
                        recv[cc] = wave_from_below_or(rv.up[cc], feed2[i * C + cc]);
                    }
#pragma unroll
                    for (int v = 0; v < NV; ++v) vq[i][v] = ld_scratch(vn + ((long)i * NV + v) * kWave);
                    // (two steps back: the next slot down, or the last slot of the next chunk, which has just been requested)
                    const real ec = wave_from_above_or(vq[(i + CH - 1) % CH][R - 1], feed[i * C]);
                    const real gp = rv.step(ec, et, el, recv, p, Ac[0], Bc[0], A0[0], B0[0]);
                    pt[i * kWave] = gp;
                    if (lane == 0 && above && T0 + i < nb) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) above[(long)(T0 + i) * C + 1 + cc] = rv.up[cc];
                    }
                }
            }
            wide_barrier(nw);
        }
        scratch_fence();
    }
}

// dF/d(increments) from dF/dp (Section 3.4); LL2: blocks off the diagonal of the lead-lag level have no increment.
template <bool LL2>
__device__ __forceinline__ void wide_map(const SweepArgs& a, int w, int nw, int lane, const real* G, long xi, long yi)
{
    const int n16 = lane & 15, g16 = lane >> 4;
    const int NT = a.lk_NT, ns = a.lk_ns, nb = a.nb, d = a.d;
    auto at = [&](const real* Gs, int row, int lr, int J) -> real {
        bool ok = row >= 0 && J < nb;
        if constexpr (LL2) ok = ok && (((row >> (a.rs1 - 1)) ^ (J >> (a.rs2 - 1))) & 1) == 0;
        const real v = ld_scratch(Gs + (long)(min(J, nb - 1) + lr) * kWave + lr);
        return ok ? v : 0.0;
    };
    if (a.want_gx) {
        const real* dy = a.dy + yi * a.ystride;
        real* gdx = a.gdx + xi * a.xstride;
        for (int s = w; s < ns; s += nw) {
            const real* Gs = G + (long)s * NT * kWave;
            const int Ibase = s * kWave - a.lk_padb;
            for (int n0 = 0; n0 < d; n0 += 32) {
                const int c0 = n0 + n16, c1 = c0 + 16;
                const bool two = n0 + 16 < d;
                real4w acc[2][4];
#pragma unroll
                for (int I = 0; I < 4; ++I) acc[0][I] = acc[1][I] = real4w{0.0, 0.0, 0.0, 0.0};
                for (int J0 = 0; J0 < nb; J0 += 4) {
                    const int J = J0 + g16;
                    const real* yr = dy + (long)(min(J, nb - 1) >> a.rs2) * a.DS;
                    real gv[4];
#pragma unroll
                    for (int I = 0; I < 4; ++I) gv[I] = at(Gs, Ibase + 16 * I + n16, 16 * I + n16, J);
                    const real b0 = c0 < d ? yr[c0] : 0.0, b1 = c1 < d ? yr[c1] : 0.0;
#pragma unroll
                    for (int I = 0; I < 4; ++I) acc[0][I] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[I], b0, acc[0][I], 0, 0, 0);
                    if (two) {
#pragma unroll
                        for (int I = 0; I < 4; ++I) acc[1][I] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[I], b1, acc[1][I], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int I = 0; I < 4; ++I)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = Ibase + 16 * I + g16 + 4 * r;
                        if (row < 0) continue;
                        real* gq = gdx + (long)(row >> a.rs1) * a.DS;
                        if (c0 < d) unsafeAtomicAdd(gq + c0, acc[0][I][r] * a.sc);
                        if (c1 < d) unsafeAtomicAdd(gq + c1, acc[1][I][r] * a.sc);
                    }
            }
        }
    }
    if (a.want_gy) {
        const real* dx = a.dx + xi * a.xstride;
        real* gdy = a.gdy + yi * a.ystride;
        for (int j0 = w * kWave; j0 < nb; j0 += nw * kWave) {
            for (int n0 = 0; n0 < d; n0 += 32) {
                const int c0 = n0 + n16, c1 = c0 + 16;
                const bool two = n0 + 16 < d;
                real4w acc[2][4];
#pragma unroll
                for (int I = 0; I < 4; ++I) acc[0][I] = acc[1][I] = real4w{0.0, 0.0, 0.0, 0.0};
                for (int s = 0; s < ns; ++s) {
                    const real* Gs = G + (long)s * NT * kWave;
                    const int Ibase = s * kWave - a.lk_padb;
                    for (int ka = 0; ka < 16; ++ka) {
                        const int lr = 4 * ka + g16, row = Ibase + lr;
                        const real* xr = dx + (long)(max(row, 0) >> a.rs1) * a.DS;
                        real gv[4];
#pragma unroll
                        for (int Jt = 0; Jt < 4; ++Jt) gv[Jt] = at(Gs, row, lr, j0 + 16 * Jt + n16);
                        const real b0 = c0 < d ? xr[c0] : 0.0, b1 = c1 < d ? xr[c1] : 0.0;
#pragma unroll
                        for (int Jt = 0; Jt < 4; ++Jt) acc[0][Jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[Jt], b0, acc[0][Jt], 0, 0, 0);
                        if (two) {
#pragma unroll
                            for (int Jt = 0; Jt < 4; ++Jt) acc[1][Jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[Jt], b1, acc[1][Jt], 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int Jt = 0; Jt < 4; ++Jt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int J = j0 + 16 * Jt + g16 + 4 * r;
                        if (J >= nb) continue;
                        real* gq = gdy + (long)(J >> a.rs2) * a.DS;
                        if (c0 < d) unsafeAtomicAdd(gq + c0, acc[0][Jt][r] * a.sc);
                        if (c1 < d) unsafeAtomicAdd(gq + c1, acc[1][Jt][r] * a.sc);
                    }
            }
        }
    }
}

template <int BL, int LL>
__global__ __launch_bounds__(kWideMaxWaves* kWave, 2) void wide_bwd_kernel(SweepArgs a)
{
    using W = Wide<BL, LL>;
    constexpr int NV = W::NV;
    __shared__ real feeds[kWideMaxWaves][2 * W::kFeed + 1];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = a.nw, ns = a.lk_ns, NT = a.lk_NT;
    real* rows = a.rows + (long)blockIdx.x * a.rows_slot;
    real* P = a.wd_scratch + (long)blockIdx.x * a.wd_slot;
    real* V = P + (long)ns * NT * kWave;   // [ns][2 + NT][NV][64]: two macro-steps of ones in front
    SK_LDS real* feed = (SK_LDS real*)&feeds[w][0];
    for (int s = w; s < ns; s += nw)
        for (int v = 0; v < 2 * NV; ++v) V[((long)s * (NT + 2) * NV + v) * kWave + lane] = 1.0;
    for (long q = blockIdx.x; q < a.npairs; q += gridDim.x) {
        long xi, yi, pid, pid2;
        gram_pair(a, q, xi, yi, pid, pid2);
        for (int s = w; s < ns; s += nw) {
            if (a.ll == 2) wide_form_p<true>(a, s, lane, a.dx + xi * a.xstride, a.dy + yi * a.ystride, P + (long)s * NT * kWave);
            else wide_form_p<false>(a, s, lane, a.dx + xi * a.xstride, a.dy + yi * a.ystride, P + (long)s * NT * kWave);
        }
        scratch_fence();
        wide_forward<BL, LL, true>(a, w, nw, lane, P, V, rows, feed);
        if (threadIdx.x == 0 && a.k_out) {
            const real k = ld_scratch(rows + (long)(ns - 1) * a.rowlen + (long)a.nb * W::C);
            a.k_out[pid] = k;
            if (pid2 != pid) a.k_out[pid2] = k;
        }
        wide_reverse<BL, LL>(a, w, nw, lane, P, V, rows, gram_weight(a, pid, pid2), feed);
        wide_barrier(nw);   // dF/dp of every strip is in place
        if (a.ll == 2) wide_map<true>(a, w, nw, lane, P, xi, yi);
        else wide_map<false>(a, w, nw, lane, P, xi, yi);
        wide_barrier(nw);   // P is about to be written again
        scratch_fence();
    }
}

// ------------------------------------------------------------------------------------------------
// launcher
// ------------------------------------------------------------------------------------------------
template <int BL, int LL>
static hipError_t launch_wide_t(bool backward, const SweepArgs& a, int grid, hipStream_t st)
{
    const dim3 block((unsigned)a.nw * kWave);
    if (backward) hipLaunchKernelGGL((wide_bwd_kernel<BL, LL>), dim3((unsigned)grid), block, 0, st, a);
    else hipLaunchKernelGGL((wide_fwd_kernel<BL, LL>), dim3((unsigned)grid), block, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_sweep_wide(bool backward, int BL, const SweepArgs& a, int grid, hipStream_t st)
{
    // what the kernels assume about the launch
    const long blocks = (long)a.lk_ns * kWave;
    if (a.nw < 1 || a.nw > kWideMaxWaves || grid < 1 || a.lk_ns < 1 || (a.lk_NT & 7) != 0 || a.lk_NT < a.nb + kWave - 1 ||
        a.lk_NT >= a.nb + kWave - 1 + 8 || a.lk_padb != blocks - a.mb || a.rowlen < (a.nb + 8) * (1 << BL) + 1 ||
        a.rows_slot < (long)a.lk_ns * a.rowlen || !a.wd_scratch ||
        a.wd_slot < blocks * (a.lk_NT + (backward ? (long)(a.lk_NT + 2) * wide_edge_values(BL) : 0)))
        return hipErrorInvalidValue;
    if (a.ll == 1) {
        if (BL == 1) return launch_wide_t<1, 1>(backward, a, grid, st);
        if (BL == 2) return launch_wide_t<2, 1>(backward, a, grid, st);
        return hipErrorInvalidValue;
    }
    switch (BL) {
        case 0: return launch_wide_t<0, 0>(backward, a, grid, st);
        case 1: return launch_wide_t<1, 0>(backward, a, grid, st);
        case 2: return launch_wide_t<2, 0>(backward, a, grid, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sk
