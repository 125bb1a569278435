// Split sweeps (gfx950), first launch for a few pairs of long paths: the band kernels' forward sweep (sk_band.h) and, beside it
// on the same compute units, the sweep of the adjoint recurrence alone (what this is for: sk_split_lock.hip).
//
// The forward pipeline of 32 strips is half empty while it fills and drains, and the adjoint pipeline, which runs the other
// way, fills it: its first strips are the forward sweep's last ones.  Workgroups alternate between the two directions in the
// order in which their bands start, so that a band waits only for one that was dispatched before it, whatever is resident.
// 32 pairs of 2048 points, eight channels, order 2: both sweeps 1.66 ms, the forward one alone 1.45 (step 5.13 -> 3.57 ms).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sk_band.h"
#include "sk_dev.h"
#include "sk_kernels.h"
#include "sk_lane.h"

namespace sk {

namespace split {

// The adjoint sweep of one band, the mirror image in time of band_forward: the band's last strip starts, each strip follows
// the one below it at the same lag, and every strip's top row (what its first lane hands up) goes to global memory.
template <int BL, int D, int LL>
__device__ __forceinline__ void band_adjoint(const SweepArgs& a, unsigned char* smem, int band, long pid)
{
    using BD = Band<BL, D, LL>;
    using LK = Lock<BL, D, 1, LL>;
    constexpr int C = LK::C, DSc = LK::DSc, CH = kLockCH1, SPB = kBandStrips, NVA = LK::Adj::NVA;
    constexpr int RM = BD::RM, YM = BD::YM, RSZ = kBandRing * C;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int npairs = (int)a.npairs, nbands = a.bd_nbands;
    long xi, yi;
    pair_ids(a, pid, xi, yi);
    SK_LDS real* yring = (SK_LDS real*)(smem + a.bd_off_y);
    SK_LDS real* rings = (SK_LDS real*)(smem + a.bd_off_rings);   // ring s is written by strip s and read by the strip above it
    const int ns = a.lk_ns, nb = a.nb;
    const int s0 = band * SPB;
    const int nsw = ns - s0 < SPB ? ns - s0 : SPB;
    const int nck = a.lk_NT / CH;
    const int lagc = kLockLag1 / CH;
    const int niter = nck + (SPB - 1) * lagc;
    real* arows = a.sp_arows + pid * (long)ns * a.rowlen;   // [ns][rowlen]: what strip s hands up, block column J at J C
    int* prog = a.bd_flags + (long)npairs * nbands + pid * nbands;   // per band: chunks of its first strip whose row is in global memory

    for (int t = threadIdx.x; t < (SPB + 1) * RSZ; t += blockDim.x) rings[t] = 0.0;
    __syncthreads();
    // the adjoint of k[m, n] enters under the last lane of the pair's last strip, at the last column
    if (band == nbands - 1 && threadIdx.x == 0) rings[nsw * RSZ + ((nb - 1) & RM) * C + (C - 1)] = 1.0;
    __syncthreads();

    if (w < SPB) {
        // ---------------- a strip ----------------
        const int sg = s0 + w;
        const bool active = w < nsw;
        const int rs = nsw - 1 - w;
        typename LK::Coef cf;
        typename LK::Adj ad;
        cf.setup(a, active ? sg : 0, lane, a.dx + xi * a.xstride, yring);
        ad.init();
        const SK_LDS real* rin = rings + (w + 1) * RSZ;
        SK_LDS real* rout = rings + w * RSZ;
        real* ackpt = a.sp_ackpt + pid * a.sp_ackpt_slot + (long)sg * a.sp_tasks * NVA * kWave + lane;
        auto chunk = [&](auto edge_c, int T0) {
            constexpr bool EDGE = decltype(edge_c)::value;
            real edge[CH][C];   // what the strip below hands to the last lane
#pragma unroll
            for (int i = 0; i < CH; ++i)
#pragma unroll
                for (int cc = 0; cc < C; ++cc) edge[i][cc] = 0.0;
            if (lane == kWave - 1) {
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int Jl = T0 + i - (kWave - 1);
                    if (!EDGE || (unsigned)Jl < (unsigned)nb) {
#pragma unroll
                        for (int cc = 0; cc < C; ++cc) edge[i][cc] = rin[(Jl & RM) * C + cc];
                    }
                }
            }
            int J[2], b[2];
            real y[2][D];
            BD::template fetch<EDGE>(cf, yring, T0 + CH - 1, J[(CH - 1) & 1], b[(CH - 1) & 1], y[(CH - 1) & 1]);
#pragma unroll
            for (int i = CH - 1; i >= 0; --i) {
                if (i >= 1) BD::template fetch<EDGE>(cf, yring, T0 + i - 1, J[(i - 1) & 1], b[(i - 1) & 1], y[(i - 1) & 1]);
                real Ac[1], Bc[1], A0[1], B0[1], recv[C];
                LK::coef_fwd(cf.template inner<EDGE>(0, J[i & 1], y[i & 1]), Ac[0], Bc[0]);
                if constexpr (LL == 1) LK::coef_fwd(cf.template inner_off<EDGE>(0, J[i & 1]), A0[0], B0[0]);
                else { A0[0] = Ac[0]; B0[0] = Bc[0]; }
#pragma unroll
                for (int cc = 0; cc < C; ++cc) recv[cc] = wave_from_below_or(ad.up[cc], edge[i][cc]);
                ad.step(recv, Ac, Bc, A0, B0);
                if (lane == 0 && (!EDGE || T0 + i < nb)) {
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) rout[((T0 + i) & RM) * C + cc] = ad.up[cc];
                }
            }
        };
        for (int g = -kBandLead; g <= niter + 1; ++g) {
            const int rc = g - rs * lagc;
            if (active && rc >= 0 && rc < nck) {
                const int fc = nck - 1 - rc;
                if (rc > 0 && (fc + 1) % a.sp_chunks == 0) ad.store(ackpt + (long)((fc + 1) / a.sp_chunks) * NVA * kWave);
                if (cf.interior(fc * CH, CH)) chunk(std::false_type(), fc * CH);
                else chunk(std::true_type(), fc * CH);
            }
            band_barrier();
        }
    } else {
        // ---------------- the data-moving wave ----------------
        const real* dyg = a.dy + yi * a.ystride;
        const real* rowprev = band < nbands - 1 ? arows + (long)(s0 + SPB) * a.rowlen : nullptr;   // the first strip of the band below
        const int* progprev = band < nbands - 1 ? prog + band + 1 : nullptr;
        const bool publish = band > 0;
        constexpr int NY = (CH * DSc + kWave - 1) / kWave;
        int ylow = a.q;              // coarse y columns >= ylow are staged
        int yh0 = 0, yhn = 0;
        real yh[NY];
        real inh = 0.0;              // one value of the incoming row piece held in registers
        int seen = 0, pub = 0;
        bool dead = false;
#pragma unroll
        for (int u = 0; u < NY; ++u) yh[u] = 0.0;
        auto chunk_T0 = [&](int rc) { return (nck - 1 - rc) * CH; };
        for (int g = -kBandLead; g <= niter + 1; ++g) {
            // (0) the row pieces written out in the last iteration have had a whole chunk to arrive: announce them
            if (pub > 0) {
                stores_done();
                if (lane == 0) st_agent_int(prog + band, pub);
                pub = 0;
            }
            // the seed has been taken (the pair's last strip passes the last column in its first chunk): its ring slot serves
            // other columns from now on
            if (band == nbands - 1 && g == 4 && lane == 0) rings[nsw * RSZ + ((nb - 1) & RM) * C + (C - 1)] = 0.0;
            // (1) y increments of the coming columns, from the right
#pragma unroll
            for (int u = 0; u < NY; ++u) {
                const int t = lane + u * kWave;
                if (t < yhn * DSc) yring[__mul24((yh0 + t / DSc) & YM, DSc) + t % DSc] = yh[u];
            }
            {
                const int rcn = g + 2 < nck ? g + 2 : nck - 1;
                int lo = chunk_T0(rcn) - (kWave - 1);
                if (lo < 0) lo = 0;
                if (lo > nb - 1) lo = nb - 1;
                lo >>= a.rs2;
                int n = ylow - lo;
                if (n > CH) n = CH;
                if (n < 0) n = 0;
                yh0 = ylow - n; yhn = n; ylow -= n;
#pragma unroll
                for (int u = 0; u < NY; ++u) {
                    const int t = lane + u * kWave;
                    if (t < n * DSc) yh[u] = dyg[(long)yh0 * DSc + t];
                }
            }
            // (2) the row from the band below: the piece for the last strip's chunk g + 1 goes into its ring, the piece for chunk
            //     g + 2 is requested once the band below has it
            if (band < nbands - 1) {
                const int cw = g + 1;
                if (cw >= 0 && cw < nck && lane < CH * C) {
                    const int col = chunk_T0(cw) - (kWave - 1) + lane / C;
                    if ((unsigned)col < (unsigned)nb) rings[nsw * RSZ + (col & RM) * C + lane % C] = inh;
                }
                const int cr = g + 2;
                if (cr >= 0 && cr < nck) {
                    // block columns from chunk_T0(cr) - 63 on: written by the lower strip's chunks <= cr + 8
                    int need = cr + 9;
                    if (need > nck) need = nck;
                    if (seen < need && !dead) {
                        int want = need + kBandSlack;
                        if (want > nck) want = nck;
                        seen = wait_progress(progprev, want, a.bd_spin);
                        if (seen < need) {
                            dead = true;
                            if (lane == 0) atomicExch(a.err, 1);
                        }
                    }
                    const int col = chunk_T0(cr) - (kWave - 1) + lane / C;
                    inh = (lane < CH * C && (unsigned)col < (unsigned)nb) ? ld_scratch(rowprev + (long)col * C + lane % C) : 0.0;
                }
            }
            // (3) top rows: the pieces the strips finished in the last iteration go out to global memory
#pragma unroll
            for (int u = 0; u < (SPB * CH * C + kWave - 1) / kWave; ++u) {
                const int t = lane + u * kWave;
                const int ws = t / (CH * C), off = t % (CH * C);
                const int rc = g - 1 - (nsw - 1 - ws) * lagc;
                if (ws < nsw && rc >= 0 && rc < nck) {
                    const int col = chunk_T0(rc) + off / C;
                    if (col < nb)
                        st_agent(arows + (long)(s0 + ws) * a.rowlen + (long)col * C + off % C, rings[ws * RSZ + (col & RM) * C + off % C]);
                }
            }
            if (publish) {
                const int rc = g - 1 - (nsw - 1) * lagc;
                if (rc >= 0 && rc < nck) pub = rc + 1;
            }
            band_barrier();
        }
    }
}

template <int BL, int D, int LL>
__global__ __launch_bounds__((kBandStrips + 1) * kWave, 3) void band_split_kernel(SweepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int npairs = (int)a.npairs, turn = blockIdx.x / npairs;
    const long pid = blockIdx.x - turn * npairs;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.keep_tag = a.keep_tag_val;
    if ((turn & 1) == 0) band_forward<BL, D, true, LL>(a, smem, turn >> 1, pid);
    else band_adjoint<BL, D, LL>(a, smem, a.bd_nbands - 1 - (turn >> 1), pid);
}

template <int BL, int D, int LL>
hipError_t launch_band_t(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if (hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&band_split_kernel<BL, D, LL>)); e != hipSuccess) return e;
    hipLaunchKernelGGL((band_split_kernel<BL, D, LL>), dim3((unsigned)(2 * a.npairs * a.bd_nbands)), dim3((kBandStrips + 1) * kWave), lds, st,
                       a);
    return hipGetLastError();
}

template <int BL, int D>
hipError_t launch_band_ll(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if (a.ll == 0) return launch_band_t<BL, D, 0>(a, lds, st);
    if constexpr (BL >= 1) {
        if (a.ll == 1 && a.rs1 == 0 && a.rs2 == 0) return launch_band_t<BL, D, 1>(a, lds, st);
    }
    if (a.ll == 2 && a.rs1 >= 1 && a.rs2 >= 1) return launch_band_t<BL, D, 2>(a, lds, st);
    return hipErrorInvalidValue;
}

template <int BL>
hipError_t launch_band_bl(int DT, const SweepArgs& a, size_t lds, hipStream_t st)
{
    switch (DT) {
        case 2: return launch_band_ll<BL, 2>(a, lds, st);
        case 3: return launch_band_ll<BL, 3>(a, lds, st);
        case 4: return launch_band_ll<BL, 4>(a, lds, st);
        case 5: return launch_band_ll<BL, 5>(a, lds, st);
        case 6: return launch_band_ll<BL, 6>(a, lds, st);
        case 8: return launch_band_ll<BL, 8>(a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace split

hipError_t launch_split_band(int BL, int DT, const SweepArgs& a, size_t lds, hipStream_t st)
{
    // what the kernels assume about the launch
    const int C = 1 << BL, nck = a.lk_NT / kLockCH1;
    if (a.lk_M != 1 || a.lk_ns < 1 || a.bd_nbands != (a.lk_ns + kBandStrips - 1) / kBandStrips || (a.lk_NT & 7) != 0 ||
        a.lk_NT < a.nb + kWave - 1 || a.lk_NT >= a.nb + kWave - 1 + 8 || a.lk_padb != a.lk_ns * kWave - a.mb || !a.bd_flags || !a.ckpt ||
        a.rowlen < (a.lk_NT - (kWave - 1)) * C + 1 || a.rows_slot < (long)a.lk_ns * a.rowlen || !a.sp_arows || !a.sp_ackpt || !a.err || !a.keep_tag ||
        a.ckpt_slot < (long)a.lk_ns * (nck + 1) * (2 * C + 2) * kWave || a.sp_chunks < 1 || a.sp_tasks != (nck + a.sp_chunks - 1) / a.sp_chunks ||
        a.sp_ackpt_slot < (long)a.lk_ns * a.sp_tasks * (2 * C + 1) * kWave)
        return hipErrorInvalidValue;
    switch (BL) {
        case 0: return split::launch_band_bl<0>(DT, a, lds, st);
        case 1: return split::launch_band_bl<1>(DT, a, lds, st);
        case 2: return split::launch_band_bl<2>(DT, a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sk
