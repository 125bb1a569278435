// The forward sweep of the band kernels (sk_band.hip, where the scheme is described), as a function of the workgroup's band
// and pair: a launch of its own there, and beside the adjoint sweep in sk_split_band.hip.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sk_dev.h"
#include "sk_kernels.h"
#include "sk_lane.h"

namespace sk {

__device__ __forceinline__ void band_barrier()
{
    // LDS traffic of this wave has completed; global traffic may stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ void st_agent(real* p, real v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_agent_int(const int* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent_int(int* p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every vector memory operation this wave has issued has completed (stores acknowledged).  The rows that cross
// workgroups are written with agent-scope atomic stores and read with agent-scope atomic loads, which are
// coherent at the device's memory side by themselves (no cache has to be written back or invalidated); what
// is left to do is to keep the order: a counter is advanced only after the data it announces has arrived.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Polls *ctr until it is at least `want` (bounded).  Returns the last value read (below `want`: the wait ran out).
__device__ __forceinline__ int wait_progress(const int* ctr, int want, int limit)
{
    int v = ld_agent_int(ctr);
    for (int spin = 1; v < want && spin < limit; ++spin) {
        __builtin_amdgcn_s_sleep(4);
        v = ld_agent_int(ctr);
    }
    return v;
}

template <int BL, int D, int LL>
struct Band {
    using LK = Lock<BL, D, 1, LL>;
    static constexpr int C = LK::C, DSc = LK::DSc;
    static constexpr int RM = kBandRing - 1, YM = kBandYRing - 1;

    // y increments of the block column lane `lane` is at in macro-step T, from the ring
    template <bool EDGE>
    static __device__ __forceinline__ void fetch(const typename LK::Coef& cf, const SK_LDS real* yring, int T, int& J,
                                                 int& b, real (&y)[D])
    {
        J = T - cf.lane;
        b = (EDGE ? clamp_col(J, cf.nbm1) : J) >> cf.rs2;
        const SK_LDS real* yp = yring + __mul24(b & YM, DSc);
#pragma unroll
        for (int c = 0; c < D; ++c) y[c] = yp[c];
    }
};

// ------------------------------------------------------------------------------------------------
// forward (CKPT: phase 1 of the backward pass: checkpoints and every strip's bottom row go to global memory)
// ------------------------------------------------------------------------------------------------
template <int BL, int D, bool CKPT, int LL>
__device__ __forceinline__ void band_forward(const SweepArgs& a, unsigned char* smem, int band, long pid)
{
    using BD = Band<BL, D, LL>;
    using LK = Lock<BL, D, 1, LL>;
    constexpr int C = LK::C, DSc = LK::DSc, CH = kLockCH1, NVC = LK::NVC, SPB = kBandStrips;
    constexpr int RM = BD::RM, YM = BD::YM;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    long xi, yi;
    pair_ids(a, pid, xi, yi);
    SK_LDS real* yring = (SK_LDS real*)(smem + a.bd_off_y);
    SK_LDS real* rings = (SK_LDS real*)(smem + a.bd_off_rings);   // [SPB + 1][kBandRing][C]: ring s is read by strip s
    const int ns = a.lk_ns, nb = a.nb;
    // A strip's last lane visits block columns up to nbx - 1, a few beyond the grid (the macro-steps are rounded up to
    // whole chunks).  The values it computes there are of no interest by themselves, but the reverse sweep inverts
    // those macro-steps too and needs them under the last lane exactly as they were: the bottom rows cover them.
    const int nbx = a.lk_NT - (kWave - 1);
    const int s0 = band * SPB;
    const int nsw = ns - s0 < SPB ? ns - s0 : SPB;   // strips of this band
    const int nck = a.lk_NT / CH;
    const int lagc = kLockLag1 / CH;
    const int niter = nck + (SPB - 1) * lagc;
    real* rowsg = a.rows + pid * a.rows_slot;        // [ns][rowlen], by node column
    int* prog = a.bd_flags + pid * a.bd_nbands;      // per band: chunks of its last strip whose row is in global memory

    for (int t = threadIdx.x; t < (SPB + 1) * kBandRing * C; t += blockDim.x) rings[t] = 1.0;
    __syncthreads();

    if (w < SPB) {
        // ---------------- a strip ----------------
        const int sg = s0 + w;
        const bool active = w < nsw;
        const bool laststrip = sg == ns - 1;
        typename LK::Coef cf;
        typename LK::Fwd f;
        cf.setup(a, active ? sg : 0, lane, a.dx + xi * a.xstride, yring);
        f.init();
        real kfin = 0.0;   // k[m, n], in the last lane of the pair's last strip
        const SK_LDS real* rin = rings + w * (kBandRing * C);
        SK_LDS real* rout = rings + (w + 1) * (kBandRing * C);
        real* ckpt = CKPT ? a.ckpt + pid * a.ckpt_slot + (long)sg * (nck + 1) * NVC * kWave + lane : nullptr;

        auto chunk = [&](auto edge_c, int T0) {
            constexpr bool EDGE = decltype(edge_c)::value;
            // top edge of the strip's first lane for the whole chunk (the row above the strip)
            real edge[CH][C];
#pragma unroll
            for (int i = 0; i < CH; ++i)
#pragma unroll
                for (int cc = 0; cc < C; ++cc) edge[i][cc] = 1.0;
            if (lane == 0) {
#pragma unroll
                for (int i = 0; i < CH; ++i)
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) edge[i][cc] = rin[((T0 + i) & RM) * C + cc];
            }
            int J[2], b[2];
            real y[2][D];
            BD::template fetch<EDGE>(cf, yring, T0, J[0], b[0], y[0]);
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                if (i + 1 < CH) BD::template fetch<EDGE>(cf, yring, T0 + i + 1, J[(i + 1) & 1], b[(i + 1) & 1], y[(i + 1) & 1]);
                real Ac[1], Bc[1], A0[1], B0[1];
                LK::coef_fwd(cf.template inner<EDGE>(0, J[i & 1], y[i & 1]), Ac[0], Bc[0]);
                if constexpr (LL == 1) LK::coef_fwd(cf.template inner_off<EDGE>(0, J[i & 1]), A0[0], B0[0]);
                else { A0[0] = Ac[0]; B0[0] = Bc[0]; }
                real recv[C];
#pragma unroll
                for (int cc = 0; cc < C; ++cc) recv[cc] = wave_from_above_or(f.bot[cc], edge[i][cc]);
                f.step(recv, Ac, Bc, A0, B0);
                if (lane == kWave - 1) {
                    const int Jw = T0 + i - (kWave - 1);
                    if (!EDGE || Jw >= 0) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) rout[(Jw & RM) * C + cc] = f.bot[cc];
                        if (EDGE && Jw == nb - 1) kfin = f.bot[C - 1];
                    }
                }
            }
        };

        for (int g = -kBandLead; g <= niter + 1; ++g) {
            const int lc = g - w * lagc;
            if (active && lc >= 0 && lc < nck) {
                if (CKPT) f.store_ckpt(ckpt + (long)lc * NVC * kWave);
                if (cf.interior(lc * CH, CH)) chunk(std::false_type(), lc * CH);
                else chunk(std::true_type(), lc * CH);
                if (CKPT && lc == nck - 1) f.store_ckpt(ckpt + (long)nck * NVC * kWave);
            }
            band_barrier();
        }
        // A wait that ran out in this band or in one above it (their counters were read after their flag was set)
        // leaves rows that were never written behind: the value is not to be trusted.
        if (laststrip && active && lane == kWave - 1 && a.k_out)
            a.k_out[pid] = ld_agent_int(a.err) != 0 ? __builtin_nan("") : kfin;
    } else {
        // ---------------- the data-moving wave ----------------
        const real* dyg = a.dy + yi * a.ystride;
        const real* rowprev = band > 0 ? rowsg + (long)(s0 - 1) * a.rowlen : nullptr;
        const int* progprev = band > 0 ? prog + band - 1 : nullptr;
        const bool publish = band < a.bd_nbands - 1;
        int ynext = 0;              // next coarse y column to stage
        int yh0 = 0, yhn = 0;       // columns [yh0, yh0 + yhn) are held in registers, on their way into the ring
        real yh[2] = {0.0, 0.0};
        real inh = 1.0;             // one value of the incoming row piece held in registers
        int seen = 0;               // progress of the band above, as last read
        int pub = 0;                // progress of this band to announce at the start of the next iteration
        bool dead = false;
        if (CKPT && lane < nsw) st_agent(rowsg + (long)(s0 + lane) * a.rowlen, 1.0);   // node column 0 of each row

        for (int g = -kBandLead; g <= niter + 1; ++g) {
            // (0) the row pieces written out in the last iteration have had a whole chunk to arrive: announce them
            if (pub > 0) {
                stores_done();
                if (lane == 0) st_agent_int(prog + band, pub);
                pub = 0;
            }
            // (1) y increments: what was loaded in the last iteration goes into the ring; columns for the first
            //     strip's chunk g + 2 are requested (block columns up to (g + 2) CH + CH - 1)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int t = lane + u * kWave;
                if (t < yhn * DSc) yring[__mul24((yh0 + t / DSc) & YM, DSc) + t % DSc] = yh[u];
            }
            {
                const int cneed = g + 2;
                int upto = cneed >= 0 ? (((cneed + 1) * CH - 1) >> a.rs2) + 1 : 0;
                if (upto > a.q) upto = a.q;
                int n = upto - ynext;
                if (n > CH) n = CH;           // at most CH columns (2 values per lane) per iteration
                if (n < 0) n = 0;
                yh0 = ynext; yhn = n; ynext += n;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int t = lane + u * kWave;
                    if (t < n * DSc) yh[u] = dyg[(long)yh0 * DSc + t];
                }
            }
            // (2) the row above the band: the piece for the first strip's chunk g + 1 (loaded in the last
            //     iteration) goes into ring 0; the piece for chunk g + 2 is requested once the band above has it
            if (band > 0) {
                const int cw = g + 1;
                if (cw >= 0 && cw < nck && lane < CH * C) rings[((cw * CH + lane / C) & RM) * C + lane % C] = inh;
                const int cr = g + 2;
                if (cr >= 0 && cr < nck) {
                    // nodes of block columns [cr CH, cr CH + CH): written by the upper strip's chunks <= cr + 8
                    int need = cr + 9;
                    if (need > nck) need = nck;
                    if (seen < need && !dead) {
                        // ask for some chunks more than needed, so that the counter is read once in a while and
                        // not in every iteration (a read is a round trip to the memory side)
                        int want = need + kBandSlack;
                        if (want > nck) want = nck;
                        seen = wait_progress(progprev, want, a.bd_spin);
                        if (seen < need) {
                            dead = true;
                            if (lane == 0) atomicExch(a.err, 1);
                        }
                    }
                    const int col = cr * CH + lane / C;
                    inh = (lane < CH * C && col < nbx) ? ld_scratch(rowprev + (long)col * C + 1 + lane % C) : 1.0;
                }
            }
            // (3) bottom rows: the pieces the strips finished in the last iteration go out to global memory
#pragma unroll
            for (int u = 0; u < (SPB * CH * C + kWave - 1) / kWave; ++u) {
                const int t = lane + u * kWave;
                const int ws = t / (CH * C), off = t % (CH * C);
                const int lc = g - 1 - ws * lagc;
                const bool wanted = CKPT || (publish && ws == nsw - 1);
                if (ws < nsw && wanted && lc >= 0 && lc < nck) {
                    const int col = lc * CH - (kWave - 1) + off / C;
                    if (col >= 0)
                        st_agent(rowsg + (long)(s0 + ws) * a.rowlen + (long)col * C + 1 + off % C,
                                 rings[(ws + 1) * (kBandRing * C) + (col & RM) * C + off % C]);
                }
            }
            if (publish) {
                const int lc = g - 1 - (nsw - 1) * lagc;
                if (lc >= 0 && lc < nck) pub = lc + 1;
            }
            band_barrier();
        }
    }
}

}  // namespace sk
