// Split sweeps (gfx950), first launch, one workgroup per pair and direction: the forward sweep and, beside it, the sweep of
// the adjoint recurrence alone.
//
// A few pairs leave most of the chip idle, and the time of a training step is the length of its chains of macro-steps.  The
// reverse sweep of the lock-step and band kernels is one such chain, three times as long as the forward one, because the wave
// that carries it recovers the forward values and forms dF/dp on the way.  Neither has to be in the chain: the first relation
// of Section 3.4 needs the coefficients only.  So a forward call whose sweep is kept for the backward call runs both
// recurrences at once, on different compute units, each leaving a checkpoint of its lane state every few macro-steps (the
// adjoint for the upstream gradient 1; it is linear in it), and the backward call is one launch without any chain: its waves
// take a few macro-steps of a strip each, replay the forward values from the checkpoint in front of them, walk back with the
// adjoint from the checkpoint behind them, form dF/dp and map it to the increments (sk_split_seg.hip).  Nothing is divided by,
// so no pair drifts.
//
// This file: pairs whose strips fit one workgroup (roles, rings and hand-over rows as in sk_lockstep.hip).  128 pairs of 256
// points, five channels, order 1 with time: the forward sweep with checkpoints 52 us alone, 56 us
// with the adjoint sweep beside it; the second launch 54 us, where the reverse sweep took 135 (step 182 -> 108 us).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sk_dev.h"
#include "sk_kernels.h"
#include "sk_lane.h"

namespace sk {

namespace split {

__device__ __forceinline__ void chunk_barrier()
{
    // LDS traffic of this wave has completed; global traffic (checkpoints) may stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Roles of the waves (sk_lockstep.hip): the stencil waves first, on SIMDs of their own where there are at most two, then two
// waves per strip that form the coefficients one chunk ahead, each for half of the macro-steps.
enum { kStencil = 0, kCoefEven = 1, kCoefOdd = 2, kIdle = 3 };
__host__ __device__ inline int waves(int ns) { return ns == 1 ? 3 : (ns == 2 ? 8 : 12); }
__device__ __forceinline__ void role_of(int w, int ns, int& role, int& strip)
{
    role = kIdle;
    strip = 0;
    if (w < ns) { role = kStencil; strip = w; return; }
    const int c0 = ns <= 2 ? ns : 4;
    if (w >= c0 && w < c0 + ns) { role = kCoefEven; strip = w - c0; return; }
    const int g0 = ns == 1 ? 2 : (ns == 2 ? 6 : 8);
    if (w >= g0 && w < g0 + ns) { role = kCoefOdd; strip = w - g0; }
}

template <int BL, int D, int M, int LL>
__global__ __launch_bounds__(12 * kWave) void lock_split_kernel(SweepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    using LK = Lock<BL, D, M, LL>;
    constexpr int C = LK::C, CH = LK::CH1, NVC = LK::NVC, NVA = LK::Adj::NVA;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ns = a.lk_ns;
    int role, strip;
    role_of(w, ns, role, strip);
    const bool adjoint = (long)blockIdx.x >= a.npairs;
    const long pid = adjoint ? blockIdx.x - a.npairs : blockIdx.x;
    long xi, yi;
    pair_ids(a, pid, xi, yi);
    const real* dxp = a.fused ? a.xraw + xi * (long)a.L1 * a.d : a.dx + xi * a.xstride;
    const int rowlen = a.lk_rowlen;
    SK_LDS real* y = (SK_LDS real*)(smem + a.lk_off_y);
    SK_LDS real* cring = (SK_LDS real*)(smem + a.lk_off_cring + (size_t)strip * a.lk_cring_stride);
    SK_LDS real* rows = (SK_LDS real*)(smem + a.lk_off_krows);   // [ns + 1][rowlen]: forward values or adjoints between the strips
    SK_LDS real* dump = (SK_LDS real*)(smem + a.lk_off_dump);
    {
        const int n = a.q * LK::DSc;
        if (a.fused) {
            const real* yp = a.yraw + yi * (long)a.L2 * a.d;
            for (int t = threadIdx.x; t < n; t += blockDim.x) {
                const int b = t / LK::DSc, c = t - b * LK::DSc;
                y[t] = c < a.d ? yp[(long)(b + 1) * a.d + c] - yp[(long)b * a.d + c] : 0.0;
            }
        } else {
            const real* dyg = a.dy + yi * a.ystride;
            for (int t = threadIdx.x; t < n; t += blockDim.x) y[t] = dyg[t];
        }
    }
    for (int t = threadIdx.x; t < (ns + 1) * rowlen; t += blockDim.x) rows[t] = adjoint ? 0.0 : 1.0;
    __syncthreads();
    // the adjoint of k[m, n] enters through the row under the last strip
    if (adjoint && threadIdx.x == 0) rows[ns * rowlen + LK::PADF + (a.nb - 1) * C + (C - 1)] = 1.0;
    const SK_LDS real* above = rows + strip * rowlen + LK::PADF;
    SK_LDS real* below = rows + (strip + 1) * rowlen + LK::PADF;
    const int nck = a.lk_NT / CH;
    const int lagc = kLockLag1 / CH;
    const int niter = nck + (ns - 1) * lagc;
    typename LK::Coef cf;
    typename LK::Off off;
    if (role == kCoefEven || role == kCoefOdd) cf.setup(a, strip, lane, dxp, y);
    off.setup(a, strip, lane);
    if (!adjoint) {
        real* ckpt = a.ckpt + pid * a.ckpt_slot + (long)strip * (nck + 1) * NVC * kWave + lane;
        typename LK::Fwd f;
        f.init();
        for (int g = -1; g < niter; ++g) {
            const int lc = g - strip * lagc;
            if (role == kStencil) {
                if (lc >= 0 && lc < nck) {
                    f.store_ckpt(ckpt + (long)lc * NVC * kWave);
                    f.chunk(lc * CH, lane, cring + (lc & 1) * LK::CR1, above, below, dump, off);
                }
            } else if (role != kIdle) {
                const int hc = lc + 1;
                if (hc >= 0 && hc < nck) cf.produce_fwd(hc * CH, cring + (hc & 1) * LK::CR1, role);
            }
            chunk_barrier();
        }
        if (threadIdx.x == 0) a.k_out[pid] = rows[ns * rowlen + LK::PADF + a.nb * C];
    } else {
        // The mirror image in time: strips bottom-up, chunks and macro-steps from the last to the first.  Outside the grid the
        // adjoint is exactly zero on the right; what leaves it on the left meets nothing any more.
        real* ackpt = a.sp_ackpt + pid * a.sp_ackpt_slot + (long)strip * a.sp_tasks * NVA * kWave + lane;
        SK_LDS real* out = lane == 0 ? rows + strip * rowlen + LK::PADF : dump + lane * C;
        typename LK::Adj ad;
        ad.init();
        auto chunk = [&](int T0, const SK_LDS real* half) __attribute__((always_inline)) {
            const SK_LDS real* cp = half + lane * 2;
            const SK_LDS real* ip = below + (T0 - (kWave - 1)) * C;   // what the strip below hands to the last lane
            SK_LDS real* op = lane == 0 ? out + T0 * C : out;
            constexpr int PF = 2;   // coefficient and edge reads are issued PF macro-steps ahead
            real2 ab[CH][M];
            real edge[CH][C];
            auto load = [&](int i) {
#pragma unroll
                for (int m = 0; m < M; ++m) ab[i][m] = *(const SK_LDS real2*)(cp + (i * M + m) * (kWave * 2));
#pragma unroll
                for (int cc = 0; cc < C; ++cc) edge[i][cc] = ip[i * C + cc];
            };
#pragma unroll
            for (int i = CH - 1; i > CH - 1 - PF; --i) load(i);
#pragma unroll
            for (int i = CH - 1; i >= 0; --i) {
                if (i - PF >= 0) load(i - PF);
                real Ac[M], Bc[M], A0[M], B0[M], recv[C];
#pragma unroll
                for (int m = 0; m < M; ++m) { Ac[m] = ab[i][m].x; Bc[m] = ab[i][m].y; }
                if constexpr (LL == 1) off.at(T0 + i, A0, B0);
                else {
#pragma unroll
                    for (int m = 0; m < M; ++m) { A0[m] = Ac[m]; B0[m] = Bc[m]; }
                }
#pragma unroll
                for (int cc = 0; cc < C; ++cc) recv[cc] = wave_from_below_or(ad.up[cc], edge[i][cc]);
                ad.step(recv, Ac, Bc, A0, B0);
#pragma unroll
                for (int cc = 0; cc < C; ++cc) op[i * C + cc] = ad.up[cc];
            }
        };
        const int rs = ns - 1 - strip;
        for (int g = -1; g < niter; ++g) {
            const int rc = g - rs * lagc;
            if (role == kStencil) {
                if (rc >= 0 && rc < nck) {
                    const int fc = nck - 1 - rc;
                    if (rc > 0 && (fc + 1) % a.sp_chunks == 0) ad.store(ackpt + (long)((fc + 1) / a.sp_chunks) * NVA * kWave);
                    chunk(fc * CH, cring + (rc & 1) * LK::CR1);
                }
            } else if (role != kIdle) {
                const int hc = rc + 1;
                if (hc >= 0 && hc < nck) cf.produce_fwd((nck - 1 - hc) * CH, cring + (hc & 1) * LK::CR1, role);
            }
            chunk_barrier();
        }
    }
    // the rows between the strips, for the launch that takes the sweeps over
    real* keep = (adjoint ? a.sp_arows : a.lk_keep) + pid * (long)(ns + 1) * rowlen;
    for (int t = threadIdx.x; t < (ns + 1) * rowlen; t += blockDim.x) keep[t] = rows[t];
    if (!adjoint && pid == 0 && threadIdx.x == 0) {
        *a.keep_tag = a.keep_tag_val;
        if (a.fused) *a.err = 0;   // (no preparation launch has cleared it)
    }
}

template <int BL, int D, int M, int LL>
hipError_t launch_t(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if (hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&lock_split_kernel<BL, D, M, LL>)); e != hipSuccess) return e;
    hipLaunchKernelGGL((lock_split_kernel<BL, D, M, LL>), dim3((unsigned)(2 * a.npairs)), dim3(waves(a.lk_ns) * kWave), lds, st, a);
    return hipGetLastError();
}

template <int BL, int D, int LL>
hipError_t launch_m(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if constexpr (lock_max_rows(true, BL, D) >= 1) {
        if (a.lk_M == 1) return launch_t<BL, D, 1, LL>(a, lds, st);
    }
    if constexpr (lock_max_rows(true, BL, D) >= 2) {
        if (a.lk_M == 2) return launch_t<BL, D, 2, LL>(a, lds, st);
    }
    return hipErrorInvalidValue;
}

template <int BL, int D>
hipError_t launch_ll(const SweepArgs& a, size_t lds, hipStream_t st)
{
    if (a.ll == 0) return launch_m<BL, D, 0>(a, lds, st);
    if constexpr (BL >= 1) {
        if (a.ll == 1 && a.rs1 == 0 && a.rs2 == 0) return launch_m<BL, D, 1>(a, lds, st);
    }
    if (a.ll == 2 && a.rs1 >= 1 && a.rs2 >= 1) return launch_m<BL, D, 2>(a, lds, st);
    return hipErrorInvalidValue;
}

template <int BL>
hipError_t launch_bl(int DT, const SweepArgs& a, size_t lds, hipStream_t st)
{
    switch (DT) {
        case 2: return launch_ll<BL, 2>(a, lds, st);
        case 3: return launch_ll<BL, 3>(a, lds, st);
        case 4: return launch_ll<BL, 4>(a, lds, st);
        case 5: return launch_ll<BL, 5>(a, lds, st);
        case 6: return launch_ll<BL, 6>(a, lds, st);
        case 8: return launch_ll<BL, 8>(a, lds, st);
        case 16: return launch_ll<BL, 16>(a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace split

hipError_t launch_split_lock(int BL, int DT, const SweepArgs& a, size_t lds, hipStream_t st)
{
    // what the kernel assumes about the launch
    const int RR = a.lk_M << BL, C = 1 << BL, nck = a.lk_NT / kLockCH1;
    if (a.lk_ns < 1 || a.lk_ns > kLockMaxStrips || (a.lk_NT & 7) != 0 || a.lk_NT < a.nb + kWave - 1 || a.lk_NT >= a.nb + kWave - 1 + 8 ||
        a.lk_padb != a.lk_ns * kWave * a.lk_M - a.mb || !a.lk_keep || !a.keep_tag || !a.sp_arows || !a.sp_ackpt || !a.ckpt || !a.k_out ||
        a.lk_rowlen < kWave * C + a.lk_NT * C + C + 1 || a.ckpt_slot < (long)a.lk_ns * (nck + 1) * (RR + C + 2) * kWave ||
        a.sp_chunks < 1 || a.sp_tasks != (nck + a.sp_chunks - 1) / a.sp_chunks || a.sp_ackpt_slot < (long)a.lk_ns * a.sp_tasks * (RR + 1 + C) * kWave)
        return hipErrorInvalidValue;
    switch (BL) {
        case 0: return split::launch_bl<0>(DT, a, lds, st);
        case 1: return split::launch_bl<1>(DT, a, lds, st);
        case 2: return split::launch_bl<2>(DT, a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sk
