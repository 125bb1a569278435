// Split sweeps (gfx950), second launch: dF/dp of every block and the linear map of Section 3.4, from the checkpoints that the
// forward and the adjoint sweep have left (sk_split_lock.hip says what for).  No chain of macro-steps longer than a task.
//
// A wave takes a task, a few chunks of eight macro-steps of one strip, from the last to the first: it replays a chunk's
// forward values from the checkpoint in front of it, keeping each macro-step's left edge and the edge from the lane above in
// registers (the eight steps are unrolled), then walks the chunk back with the adjoint, which it carries from the checkpoint
// behind the task.  x-side sums stay in registers, y-side sums in a window of LDS of the wave's own; the waves of a
// workgroup take neighbouring tasks of one strip and add both up, in a fixed order, before they go to memory.  (A strip of up to
// 64 chunks is one workgroup's: the gradients of pairs of at most two such strips are the same bits in every call.  More strips or
// workgroups, and the pairs of a Gram matrix, add in the order in which they arrive.)
//
// What bounds it: instruction issue of a wave alone on its SIMD, half of it the forward values (replayed once to keep the edges,
// formed once more block by block), and its LDS instructions, which nothing hides.  Counters: 128 pairs of 256 points, d = 5, order
// 1: 14100 vector and 1150 LDS instructions per wave, 8.0 clocks per vector instruction (4 to issue it), 54 us, where the
// reverse sweep took 135; 32 pairs of 2048 points, d = 8, order 2: 15700 and 1230, 7.9 clocks, 2.0 ms for 3.65.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sk_dev.h"
#include "sk_kernels.h"
#include "sk_lane.h"

namespace sk {

namespace split {

template <int BL, int D, int M, int LL>
__global__ __launch_bounds__(split_seg_waves(BL, D, M) * kWave, split_seg_waves(BL, D, M) / 4) void seg_kernel(SweepArgs a)
{
    constexpr int kSegWaves = split_seg_waves(BL, D, M);
    extern __shared__ __align__(16) unsigned char smem[];
    using LK = Lock<BL, D, M, LL>;
    constexpr int C = LK::C, RR = LK::RR, DSc = LK::DSc, CH = kLockCH1, NVC = LK::NVC, NVA = LK::Adj::NVA;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ns = a.lk_ns, nb = a.nb, nck = a.lk_NT / CH;
    const int ntask = a.sp_tasks, ngrp = (ntask + kSegWaves - 1) / kSegWaves;
    const int grp = blockIdx.x % ngrp;
    const long rest = blockIdx.x / ngrp;
    const int strip = (int)(rest % ns);
    const long pid = rest / ns;
    long xi, yi;
    pair_ids(a, pid, xi, yi);
    const int task = grp * kSegWaves + w;
    const bool active = task < ntask;
    const int K = a.sp_chunks;   // chunks per task
    const int c0 = task * K, c1 = min(nck, c0 + K);
    // y increments of the columns the workgroup's tasks touch; the wave's own window of sums
    const int gJ0 = max(grp * kSegWaves * K * CH - (kWave - 1), 0);
    const int gJ1 = min(min(nck, (grp + 1) * kSegWaves * K) * CH - 1, nb - 1);
    const int gb0 = gJ0 >> a.rs2, gn = (gJ1 >> a.rs2) - gb0 + 1;
    SK_LDS real* yl = (SK_LDS real*)smem;                                         // [gn][DSc]
    SK_LDS real* gyl = (SK_LDS real*)(smem + a.sp_off_gy) + (long)w * a.sp_win * DSc;   // [sp_win][DSc] per wave
    SK_LDS real* feed = (SK_LDS real*)(smem + a.sp_off_feed) + w * (2 * CH * C);
    SK_LDS real* feed2 = feed + CH * C;
    const int wb0 = max(c0 * CH - (kWave - 1), 0) >> a.rs2;
    const int wn = active ? (min(c1 * CH - 1, nb - 1) >> a.rs2) - wb0 + 1 : 0;    // columns of the wave's window
    {
        const real* dyg = a.dy + yi * a.ystride + (long)gb0 * DSc;
        for (int t = threadIdx.x; t < gn * DSc; t += blockDim.x) yl[t] = dyg[t];
        for (int t = lane; t < wn * DSc; t += kWave) gyl[t] = 0.0;
    }
    __syncthreads();
    typename LK::Coef cf;
    typename LK::Off off;
    typename LK::Adj ad;
    // (the copy starts at column gb0; LDS addresses are 32-bit integers)
    cf.setup(a, strip, lane, a.dx + xi * a.xstride, (const SK_LDS real*)(size_t)((unsigned)(size_t)yl - (unsigned)(gb0 * DSc * (int)sizeof(real))));
    off.setup(a, strip, lane);
    ad.init();
    real gacc[M][D];
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int c = 0; c < D; ++c) gacc[m][c] = 0.0;
    if (active) {
        const real* ckpt = a.ckpt + pid * a.ckpt_slot + (long)strip * (nck + 1) * NVC * kWave + lane;
        if (c1 < nck) ad.load(a.sp_ackpt + pid * a.sp_ackpt_slot + ((long)strip * ntask + task + 1) * NVA * kWave + lane);
        // The rows between the strips.  Forward values: node n of the row above the strip at rowk[n]; adjoints: what the strip
        // below hands up at block column J at rowa[J C ..].
        const real *rowk, *rowa;
        if (a.band) {
            rowk = strip > 0 ? a.rows + pid * a.rows_slot + (long)(strip - 1) * a.rowlen : nullptr;
            rowa = strip < ns - 1 ? a.sp_arows + (pid * (long)ns + strip + 1) * a.rowlen : nullptr;
        } else {
            rowk = strip > 0 ? a.lk_keep + (pid * (long)(ns + 1) + strip) * a.lk_rowlen + LK::PADF : nullptr;
            rowa = strip < ns - 1 ? a.sp_arows + (pid * (long)(ns + 1) + strip + 1) * a.lk_rowlen + LK::PADF : nullptr;
        }
        const int nbx = a.lk_NT - (kWave - 1);   // block columns a strip's last lane visits: its row ends there
        real cp[RR + 1 + C], fk = 1.0, fa = 0.0;
        auto load_chunk = [&](int c) {
            const real* p = ckpt + (long)c * NVC * kWave;
#pragma unroll
            for (int i = 0; i < RR + 1 + C; ++i) cp[i] = p[i * kWave];
            const int J = c * CH + lane / C;
            fk = (rowk && lane < CH * C && J < nbx) ? rowk[(long)J * C + 1 + lane % C] : 1.0;
            const int Ja = J - (kWave - 1);
            fa = 0.0;
            if (lane < CH * C && (unsigned)Ja < (unsigned)nb) {
                if (rowa) fa = rowa[(long)Ja * C + lane % C];
                else fa = (Ja == nb - 1 && lane % C == C - 1) ? 1.0 : 0.0;
            }
        };
        load_chunk(c1 - 1);
        auto chunk = [&](auto edge_c, auto plain_c, int T0, bool more) __attribute__((always_inline)) {
            constexpr bool EDGE = decltype(edge_c)::value, PLAIN = decltype(plain_c)::value;
            if (lane < CH * C) { feed[lane] = fk; feed2[lane] = fa; }
            __builtin_amdgcn_wave_barrier();
            // ---- replay: p, left edge and top edge of every macro-step ----
            real left0, el[CH][RR], et[CH][C], pp[CH][M];
            {
                typename LK::Fwd f;
                left0 = cp[0];
#pragma unroll
                for (int i = 0; i <= RR; ++i) f.left[i] = cp[i];
#pragma unroll
                for (int i = 0; i < C; ++i) f.bot[i] = cp[RR + 1 + i];
                if (more) load_chunk(T0 / CH - 1);
                int J[2], b[2];
                real y[2][D];
                real edge[2][C];
                cf.template fetch<EDGE>(T0, J[0], b[0], y[0]);
#pragma unroll
                for (int cc = 0; cc < C; ++cc) edge[0][cc] = feed[cc];
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    if (i + 1 < CH) {
                        cf.template fetch<EDGE>(T0 + i + 1, J[(i + 1) & 1], b[(i + 1) & 1], y[(i + 1) & 1]);
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) edge[(i + 1) & 1][cc] = feed[(i + 1) * C + cc];
                    }
                    real Ac[M], Bc[M], A0[M], B0[M], recv[C];
#pragma unroll
                    for (int m = 0; m < M; ++m) pp[i][m] = cf.template inner<EDGE>(m, J[i & 1], y[i & 1]);
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) et[i][cc] = recv[cc] = wave_from_above_or(f.bot[cc], edge[i & 1][cc]);
#pragma unroll
                    for (int rr = 0; rr < RR; ++rr) el[i][rr] = f.left[rr + 1];
                    if (i + 1 < CH) {
#pragma unroll
                        for (int m = 0; m < M; ++m) LK::coef_fwd(pp[i][m], Ac[m], Bc[m]);
                        if constexpr (LL == 1) off.at(T0 + i, A0, B0);
                        else {
#pragma unroll
                            for (int m = 0; m < M; ++m) { A0[m] = Ac[m]; B0[m] = Bc[m]; }
                        }
                        f.step(recv, Ac, Bc, A0, B0);
                    }
                }
            }
            // ---- back, with the adjoint ----
            int J[2], b[2];
            real y[2][D];
            real edge[2][C];
            cf.template fetch<EDGE>(T0 + CH - 1, J[(CH - 1) & 1], b[(CH - 1) & 1], y[(CH - 1) & 1]);
#pragma unroll
            for (int cc = 0; cc < C; ++cc) edge[(CH - 1) & 1][cc] = feed2[(CH - 1) * C + cc];
#pragma unroll
            for (int i = CH - 1; i >= 0; --i) {
                // What the replay kept goes through opaque moves (no instructions): the block's values formed from it below are
                // those the replay went through, and the compiler would keep all of them instead, up to 900 bytes per lane in
                // scratch.
#pragma unroll
                for (int m = 0; m < M; ++m) asm volatile("" : "+v"(pp[i][m]));
#pragma unroll
                for (int rr = 0; rr < RR; ++rr) asm volatile("" : "+v"(el[i][rr]));
#pragma unroll
                for (int cc = 0; cc < C; ++cc) asm volatile("" : "+v"(et[i][cc]));
                // LDS reads a macro-step or most of one ahead of their use: the column's sums (the lane below wrote them in the
                // step before), then what the next step needs
                SK_LDS real* const gq = gyl + __mul24(b[i & 1] - wb0, DSc);
                const bool mine = !EDGE || (unsigned)J[i & 1] < (unsigned)nb;
                real sum[D];
                if constexpr (PLAIN) {
#pragma unroll
                    for (int c = 0; c < D; ++c) sum[c] = gq[c];
                }
                if (i > 0) {
                    cf.template fetch<EDGE>(T0 + i - 1, J[(i - 1) & 1], b[(i - 1) & 1], y[(i - 1) & 1]);
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) edge[(i - 1) & 1][cc] = feed2[(i - 1) * C + cc];
                }
                real Ac[M], Bc[M], A0[M], B0[M], recv[C];
#pragma unroll
                for (int m = 0; m < M; ++m) LK::coef_fwd(pp[i][m], Ac[m], Bc[m]);
                if constexpr (LL == 1) off.at(T0 + i, A0, B0);
                else {
#pragma unroll
                    for (int m = 0; m < M; ++m) { A0[m] = Ac[m]; B0[m] = Bc[m]; }
                }
#pragma unroll
                for (int cc = 0; cc < C; ++cc) recv[cc] = wave_from_below_or(ad.up[cc], edge[i & 1][cc]);
                real e[RR + 1][C + 1], gn[RR + 1][C + 1];
                e[0][0] = i > 0 ? et[i > 0 ? i - 1 : 0][C - 1] : left0;
#pragma unroll
                for (int cc = 0; cc < C; ++cc) e[0][cc + 1] = et[i][cc];
#pragma unroll
                for (int rr = 0; rr < RR; ++rr) e[rr + 1][0] = el[i][rr];
#pragma unroll
                for (int rr = 0; rr < RR; ++rr)
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) {
                        const bool o = LK::cell_off(rr, cc);
                        const int m = rr >> BL;
                        e[rr + 1][cc + 1] = fma(e[rr + 1][cc] + e[rr][cc + 1], o ? A0[m] : Ac[m], -(e[rr][cc] * (o ? B0[m] : Bc[m])));
                    }
                ad.begin(gn, recv);
                real gs[M], gk[M], gp[M];
#pragma unroll
                for (int rr = RR - 1; rr >= 0; --rr) {
                    const int m = rr >> BL;
#pragma unroll
                    for (int cc = C - 1; cc >= 0; --cc) {
                        const bool o = LK::cell_off(rr, cc);
                        const real Aq = o ? A0[m] : Ac[m], Bq = o ? B0[m] : Bc[m];
                        const real go = gn[rr + 1][cc + 1];
                        gn[rr + 1][cc] = fma(go, Aq, gn[rr + 1][cc]);
                        gn[rr][cc + 1] = fma(go, Aq, gn[rr][cc + 1]);
                        gn[rr][cc] = fma(-go, Bq, gn[rr][cc]);
                        if (o) continue;
                        const real s = e[rr + 1][cc] + e[rr][cc + 1];
                        const bool first = (rr & (C - 1)) == C - 1 && cc == C - 1;   // the block's first cell in this order
                        gs[m] = first ? go * s : fma(go, s, gs[m]);
                        gk[m] = first ? go * e[rr][cc] : fma(go, e[rr][cc], gk[m]);
                    }
                }
                ad.finish(gn);
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    // (left of the grid the adjoint that has left it is not zero; rows above the grid have no increments;
                    // lead-lag: blocks off the diagonal of that level have none either)
                    const real p6 = pp[i][m] * (1.0 / 6.0);
                    const real v = fma(gs[m], p6 + 0.5, gk[m] * p6);   // A'(p) = p / 6 + 1 / 2, -B'(p) = p / 6
                    gp[m] = ((!EDGE || (unsigned)J[i & 1] < (unsigned)cf.nbl[m]) && !cf.off_block(m, J[i & 1])) ? v : 0.0;
                }
                // (both sides whether wanted or not: a branch here costs more than the few multiply-adds)
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int c = 0; c < D; ++c) gacc[m][c] = fma(gp[m], y[i & 1][c], gacc[m][c]);
                if constexpr (PLAIN) {
#pragma unroll
                    for (int c = 0; c < D; ++c) {
#pragma unroll
                        for (int m = 0; m < M; ++m) sum[c] = fma(gp[m], cf.dxr[m][c], sum[c]);
                    }
                    if (mine) {
#pragma unroll
                        for (int c = 0; c < D; ++c) gq[c] = sum[c];
                    }
                } else if (mine) {
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        real t = gp[0] * cf.dxr[0][c];
#pragma unroll
                        for (int m = 1; m < M; ++m) t = fma(gp[m], cf.dxr[m][c], t);
                        lds_atomic_add(gq + c, t);
                    }
                }
            }
        };
        for (int c = c1 - 1; c >= c0; --c) {
            // (refinement above the blocks: lanes share y rows, and their sums meet in LDS atomics; otherwise 64 lanes are at 64
            // different rows, and a plain read-modify-write is safe)
            if (a.rs2 != 0) chunk(std::true_type(), std::false_type(), c * CH, c > c0);
            else if (cf.interior(c * CH, CH)) chunk(std::false_type(), std::true_type(), c * CH, c > c0);
            else chunk(std::true_type(), std::true_type(), c * CH, c > c0);
        }
    }
    // ---- the workgroup's sums, times the upstream gradient (NaN if the workspace holds another call's sweeps) ----
    real scale = a.grad_k[pid];
    if (*a.keep_tag != a.keep_tag_val) scale = __builtin_nan("");
    __syncthreads();
    if (a.want_gy) {
        real* gdy = a.gdy + yi * a.ystride;
        for (int t = threadIdx.x; t < gn * DSc; t += blockDim.x) {
            const int b = t / DSc, c = t - b * DSc;
            real v = 0.0;
#pragma unroll
            for (int u = 0; u < kSegWaves; ++u) {
                const int tk = grp * kSegWaves + u, k0 = tk * K;
                if (tk >= ntask) break;
                const int u0 = max(k0 * CH - (kWave - 1), 0) >> a.rs2;
                const int u1 = min(min(nck, k0 + K) * CH - 1, nb - 1) >> a.rs2;
                const int bb = gb0 + b;
                if (bb >= u0 && bb <= u1) v += ((SK_LDS real*)(smem + a.sp_off_gy))[((long)u * a.sp_win + (bb - u0)) * DSc + c];
            }
            v *= scale;
            if (c < a.d && v != 0.0) unsafeAtomicAdd(&gdy[(long)(gb0 + b) * DSc + c], v);
        }
    }
    if (a.want_gx) {
        // (over the y increments and sums, which are no longer needed)
        __syncthreads();
        SK_LDS real* gxl = (SK_LDS real*)smem;   // [waves][64 M][DSc]
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int c = 0; c < D; ++c) gxl[((w * kWave + lane) * M + m) * DSc + c] = gacc[m][c];
        __syncthreads();
        real* gdx = a.gdx + xi * a.xstride;
        for (int t = threadIdx.x; t < kWave * M * DSc; t += blockDim.x) {
            const int row = t / DSc, c = t - row * DSc;
            const int I = strip * kWave * M + row - a.lk_padb;
            if (I < 0 || c >= a.d) continue;
            real v = 0.0;
#pragma unroll
            for (int u = 0; u < kSegWaves; ++u) v += gxl[u * (kWave * M * DSc) + t];
            v *= scale * a.sc;
            if (v != 0.0) unsafeAtomicAdd(&gdx[(long)(I >> a.rs1) * DSc + c], v);
        }
    }
    // the kernel value: the last node of the last strip's bottom row
    if (a.k_out && strip == ns - 1 && grp == 0 && threadIdx.x == 0)
        a.k_out[pid] = a.band ? (*a.err != 0 ? __builtin_nan("") : a.rows[pid * a.rows_slot + (long)(ns - 1) * a.rowlen + (long)nb * C])
                              : a.lk_keep[(pid * (long)(ns + 1) + ns) * a.lk_rowlen + LK::PADF + nb * C];
}

template <int BL, int D, int M, int LL>
hipError_t launch_seg_t(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if (hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&seg_kernel<BL, D, M, LL>)); e != hipSuccess) return e;
    constexpr int W = split_seg_waves(BL, D, M);
    const long groups = (a.sp_tasks + W - 1) / W;
    hipLaunchKernelGGL((seg_kernel<BL, D, M, LL>), dim3((unsigned)(a.npairs * a.lk_ns * groups)), dim3(W * kWave), lds, st, a);
    return hipGetLastError();
}

template <int BL, int D, int LL>
hipError_t launch_seg_m(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if constexpr (D <= 8 || lock_max_rows(true, BL, D) >= 1) {
        if (a.lk_M == 1) return launch_seg_t<BL, D, 1, LL>(a, lds, st);
    }
    if constexpr (lock_max_rows(true, BL, D) >= 2) {
        if (a.lk_M == 2) return launch_seg_t<BL, D, 2, LL>(a, lds, st);
    }
    return hipErrorInvalidValue;
}

template <int BL, int D>
hipError_t launch_seg_ll(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if (a.ll == 0) return launch_seg_m<BL, D, 0>(a, lds, st);
    if constexpr (BL >= 1) {
        if (a.ll == 1 && a.rs1 == 0 && a.rs2 == 0) return launch_seg_m<BL, D, 1>(a, lds, st);
    }
    if (a.ll == 2 && a.rs1 >= 1 && a.rs2 >= 1) return launch_seg_m<BL, D, 2>(a, lds, st);
    return hipErrorInvalidValue;
}

template <int BL>
hipError_t launch_seg_bl(int DT, const SweepArgs& a, size_t lds, hipStream_t st)
{
    switch (DT) {
        case 2: return launch_seg_ll<BL, 2>(a, lds, st);
        case 3: return launch_seg_ll<BL, 3>(a, lds, st);
        case 4: return launch_seg_ll<BL, 4>(a, lds, st);
        case 5: return launch_seg_ll<BL, 5>(a, lds, st);
        case 6: return launch_seg_ll<BL, 6>(a, lds, st);
        case 8: return launch_seg_ll<BL, 8>(a, lds, st);
        case 16: return launch_seg_ll<BL, 16>(a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace split

hipError_t launch_split_seg(int BL, int DT, const SweepArgs& a, size_t lds, hipStream_t st)
{
    // what the kernel assumes about the launch
    const int RR = a.lk_M << BL, C = 1 << BL, nck = a.lk_NT / kLockCH1;
    if (a.fused || a.lk_ns < 1 || (a.lk_NT & 7) != 0 || !a.ckpt || !a.sp_arows || !a.sp_ackpt || !a.keep_tag || !a.grad_k ||
        (a.band ? (!a.rows || !a.err) : !a.lk_keep) || a.ckpt_slot < (long)a.lk_ns * (nck + 1) * (RR + C + 2) * kWave ||
        a.sp_chunks < 1 || a.sp_tasks != (nck + a.sp_chunks - 1) / a.sp_chunks || a.sp_ackpt_slot < (long)a.lk_ns * a.sp_tasks * (RR + 1 + C) * kWave ||
        a.sp_win < split_window(a.sp_chunks, a.rs2) || lds > kLdsPerCU ||
        lds < split_seg_lds(BL, DT, a.lk_M, a.sp_chunks, a.rs2))
        return hipErrorInvalidValue;
    switch (BL) {
        case 0: return split::launch_seg_bl<0>(DT, a, lds, st);
        case 1: return split::launch_seg_bl<1>(DT, a, lds, st);
        case 2: return split::launch_seg_bl<2>(DT, a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sk
