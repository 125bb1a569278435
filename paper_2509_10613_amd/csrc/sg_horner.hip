// Batched truncated signatures by Horner's scheme (paper Section 2.3) for gfx950.
//
// One step of the scheme for the increment z of a segment, read word by word (v a word, c a letter, |v| its length):
//     G_k[empty] = 1,   G_k[v c] = G_k[v] z[c] / (k - |v|) + A_{|v|+1}[v c]   for |v| + 1 < k,
//     A_k[w c] += G_k[w] z[c]                                                  for |w| = k - 1,
// levels k = N, ..., 1 in that order so that every right-hand side still holds the values before the step
// (G_k[w] is B_k[w] + A_{k-1}[w] of Section 2.3).  Starting from A = (1, 0, 0, ...), the first step gives the tensor
// exponential of the first increment (Proposition 2.1), so no separate initialisation is needed.
//
// A value at a word depends only on values at its prefixes.  A lane therefore owns a prefix u of Q letters, S
// consecutive letters after it, and all continuations by up to M more letters, in registers for the whole path, plus
// its own copies of the Q entries at the prefixes of u.  No lane talks to another one.  All lanes of a wave work on
// the same path: the D increments of a step are wave-uniform and come in by scalar loads into scalar registers, the
// few that a lane selects by its own letters come in by ordinary loads; both are fetched one step ahead.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sg_dev.h"
#include "sg_kernels.h"

namespace sg {

namespace {

// The owned entries of level Q + 1 + m go to the words u (blk S + s) v: `first` is the number of the word u (blk S) in
// base D, at[m] the start of that level in the flattened signature.
template <int m, int D, int M, int S, int TOT, typename TO>
__device__ __forceinline__ void store_owned(const double (&A)[TOT], TO* out, const long (&at)[M + 1], int Dn,
                                            long first, int c0)
{
    constexpr int pm = ipow(D, m);
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if (c0 + s < Dn) {
            TO* o = out + at[m] + (first + s) * pm;
#pragma unroll
            for (int v = 0; v < pm; ++v) o[v] = (TO)A[Tree<D, M, S>::off(m) + s * pm + v];
        }
    }
    if constexpr (m < M) store_owned<m + 1, D, M, S, TOT>(A, out, at, Dn, first, c0);
}

// A lane's entries of one signature: its own words, the carried prefix entries (written by the lane whose remaining
// letters are all zero) and, by the first lane, the empty word's.
template <int D, int M, int S, int QC, int TOT, int QA, typename TO>
__device__ __forceinline__ void store_signature(const double (&A)[TOT], const double (&preR)[QA], TO* out, int Dn, int Q,
                                                long ti, long rest, int blk)
{
    // start of level k in the flattened signature: 1 + D + ... + D^(k-1)
    auto lvl = [&](int k) {
        long o = 0, p = 1;
        for (int i = 0; i < k; ++i) {
            o += p;
            p *= Dn;
        }
        return o;
    };
    if (ti == 0) out[0] = (TO)1;
    {
        long pw = 1;
#pragma unroll
        for (int r = 0; r < QC; ++r) {
            if (has<QC>(r, Q) && blk == 0 && rest % pw == 0) out[lvl(Q - r) + rest / pw] = (TO)preR[r];
            pw *= Dn;
        }
    }
    long at[M + 1];
#pragma unroll
    for (int m = 0; m <= M; ++m) at[m] = lvl(Q + 1 + m);
    store_owned<0, D, M, S, TOT>(A, out, at, Dn, rest * Dn + blk * S, blk * S);
}

// One wave's share of one path, all steps.  DT > 0: D = DT channels, increments of a step in scalar registers.
// DT == 0: any number of channels, M = 0, S = 1 (a lane owns one word of the top level).
// LEADLAG: the rows alternate between a move of the lead half (even rows) and of the lag half (odd rows) of the
// channels; the multiply-adds with the half that stands still are left out.
template <int DT, int M, int S, int QC, bool LEADLAG>
__device__ __forceinline__ void run(const Args& a)
{
    constexpr int DD = DT > 0 ? DT : 1;
    constexpr int QA = QC > 0 ? QC : 1;
    using T = Tree<DD, M, S>;
    const int D = DT > 0 ? DT : a.D;
    const int Q = QC <= kQExact ? QC : a.Q;
    const int lane = threadIdx.x & (kWave - 1);
    // Workgroups go to the 8 XCDs (each with an L2 of its own) in turn: number them so that the workgroups of one
    // path, which read the same increments, sit on the same XCD.
    long wg = blockIdx.x;
    if (gridDim.x % kXcds == 0) wg = (long)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    const long wt = wg * kWavesPerWG + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (wt >= a.NW) return;
    const long b = wt / a.WP;
    long ti = (wt - b * a.WP) * kWave + lane;
    const bool valid = ti < a.LP;
    if (!valid) ti = 0;
    const int blk = (int)(ti % a.NB);
    const long rest = ti / a.NB;      // the prefix u as a number in base D, first letter most significant
    int uR[QA];
    {
        long t = rest;
#pragma unroll
        for (int r = 0; r < QA; ++r) {
            uR[r] = (r < QC && has<QC>(r, Q)) ? (int)(t % D) : 0;
            t /= D;
        }
    }
    int cs[S];
#pragma unroll
    for (int s = 0; s < S; ++s) cs[s] = min(blk * S + s, D - 1);

    double A[T::TOT];
#pragma unroll
    for (int i = 0; i < T::TOT; ++i) A[i] = 0.0;
    double preR[QA];
#pragma unroll
    for (int r = 0; r < QA; ++r) preR[r] = 0.0;

    const double* zrow = a.dz + b * a.np * a.Dpad;
    double zz[DD], zc[S], zuR[QA];
    double zzn[DD], zcn[S], zuRn[QA];
    auto fetch = [&](long step, double (&z_)[DD], double (&zc_)[S], double (&zu_)[QA]) {
        const double* zp = zrow + step * a.Dpad;
        if constexpr (DT > 0 && M > 0) {
            uniform_ptr zs = (uniform_ptr)(zp);
#pragma unroll
            for (int c = 0; c < DD; ++c) z_[c] = zs[c];
        }
#pragma unroll
        for (int s = 0; s < S; ++s) zc_[s] = zp[cs[s]];
#pragma unroll
        for (int r = 0; r < QA; ++r) zu_[r] = (r < QC && has<QC>(r, Q)) ? zp[uR[r]] : 0.0;
    };
#pragma unroll
    for (int c = 0; c < DD; ++c) zz[c] = zzn[c] = 0.0;
    // Two steps per iteration with two sets of registers for the increments, each set requested one step before the
    // arithmetic that reads it.  Two things keep the compiler from moving a load next to its use: the body has no
    // branch (loads get moved into the block that uses them), and the set carried round the loop starts as constants,
    // not as a load (a value that is a load on every path into the loop becomes one load at the top of the body).
    // So the first step is a zero increment, which changes nothing, the rows follow in pairs, and the stored row count
    // np is odd with zero rows after the last segment.
#pragma unroll
    for (int s = 0; s < S; ++s) zc[s] = 0.0;
#pragma unroll
    for (int r = 0; r < QA; ++r) zuR[r] = 0.0;
    for (long step = 0; step < a.np; step += 2) {
        // the set carried round the loop holds the odd rows (lag half; the zero increment at the start fits any
        // half), the other set the even rows (lead half)
        fetch(step, zzn, zcn, zuRn);
        owned_levels<M, DD, M, S, QC, T::TOT, QA, LEADLAG ? 2 : 0>(A, Q, preR, zuR, zc, zz);
        prefix_levels<QC, QA>(Q, preR, zuR);
        fetch(step + 1 < a.np ? step + 1 : step, zz, zc, zuR);
        owned_levels<M, DD, M, S, QC, T::TOT, QA, LEADLAG ? 1 : 0>(A, Q, preR, zuRn, zcn, zzn);
        prefix_levels<QC, QA>(Q, preR, zuRn);
    }

    if (!valid) return;
    if (a.out_f32)
        store_signature<DD, M, S, QC>(A, preR, static_cast<float*>(a.out) + b * a.sig_len, D, Q, ti, rest, blk);
    else
        store_signature<DD, M, S, QC>(A, preR, static_cast<double*>(a.out) + b * a.sig_len, D, Q, ti, rest, blk);
}

// LDS written by one lane of a wave and read by another one
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Several short paths side by side in a wave (at most 32 lanes per path): lane groups of LP lanes, each a path (or a
// piece of one) of its own.
// The arithmetic of such paths is little, and what bounds them is memory traffic and launches: with the increments and the
// double signatures of float callers going through memory between three launches, 100000 paths of 10 points in 2
// channels to level 3, float, took 13.6 us, 10.7 us and 5.0 us.  Here a wave copies the points of its paths to LDS, 64
// consecutive numbers per load, forms the increments as it reads them back (a broadcast within a path), and its
// signatures, which are consecutive too, go out the same way if they fit there: 10.9 us in one launch, about 3 us of it
// memory at 4.6 TB/s and the rest instructions.  Fewer paths than 1024 waves hold are spread (the plan's rule on PW):
// 1000 paths of 100 points in 6 channels to level 2 took 21.9 us at first, 23.9 with ten paths in each of 100 waves
// (copying a chunk waits for memory, and nothing else runs meanwhile), 14.5 with two.
template <int DT, int M, int QC, bool LEADLAG>
__device__ __forceinline__ void run_shared(const Args& a, double* lds)
{
    constexpr int DD = DT > 0 ? DT : 1;
    constexpr int QA = QC > 0 ? QC : 1;
    constexpr int NW = 1 + QC;                         // letters a lane selects: its own one, those of its prefix
    constexpr bool kStatic = DT > 0 && M > 0;          // increments of all channels in registers
    using T = Tree<DD, M, 1>;
    const int D = DT > 0 ? DT : a.D, d = a.d;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const long wt = (long)blockIdx.x * kWavesPerWG + wave;
    if (wt >= a.NW) return;
    const long b0 = wt * a.PW;
    const int LP = (int)a.LP, here = (int)min((long)a.PW, a.B - b0);
    int g = lane / LP, ti = lane - g * LP;
    const bool valid = g < here;
    if (!valid) {           // idle lanes follow the wave's first path and write nothing
        g = 0;
        ti = 0;
    }
    const int rest = ti / a.NB, blk = ti - rest * a.NB;
    int at[NW];             // channel of the points that letter i moves with
    bool lead[NW], lag[NW], clock[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        int c = blk, t = rest;
        if (i > 0) {
            for (int r = 1; r < i; ++r) t /= D;
            c = t % D;
        }
        clock[i] = a.time && c == D - 1;
        const bool second = a.leadlag && !clock[i] && c >= d;
        lead[i] = !clock[i] && !second;
        lag[i] = second;
        at[i] = clock[i] ? 0 : (second ? c - d : c);
    }

    // the points of the wave's paths, one chunk after the other
    const SharedLds sh = shared_lds(a.PW, d, (int)min(a.L, 1L << 20), a.sig_len);
    double* buf = lds + wave * sh.doubles;
    const int per = a.leadlag ? 2 : 1;                          // rows per segment of the points
    const long step = a.n / per;                                // segments of a piece
    const int shift = __builtin_ctz((unsigned)a.P);
    const long first = ((b0 + g) & (a.P - 1)) * step;           // first segment of this lane's piece
    const long mine = min(step, max(0L, a.total / per - first));// its segments
    // ... and those that every piece of the wave has: the last pieces of a path may have fewer
    const long least = max(0L, min(step, a.total / per - min((long)a.P - 1, (b0 & (a.P - 1)) + here - 1) * step));
    // number e of the chunk of path gg, 64 apart: q paths and `rem` numbers on; between the chunks of two whole paths lie
    // `skip` numbers of x
    auto stage = [&](auto* x, long c0, int count) {
        const int len = count * d, q = kWave / len, rem = kWave - q * len;
        const long skip = a.L * d - len;
        int gg = lane / len, e = lane - gg * len;
        const auto* whole = x + (b0 * a.L + c0) * d + lane + gg * skip;
        constexpr int U = 8;
        while (gg < here) {
            double v[U];
            int to[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                to[u] = -1;
                if (gg < here) {
                    if (a.P == 1) {
                        v[u] = (double)*whole;
                    } else {
                        const long bp = b0 + gg;
                        long k = ((bp & (a.P - 1)) * step + c0) * d + e;    // number within the path
                        if (k >= a.L * d) k = (a.L - 1) * d + e % d;        // past its end: the last point again
                        v[u] = (double)x[(bp >> shift) * a.L * d + k];
                    }
                    to[u] = gg * sh.stride + e;
                }
                gg += q;
                e += rem;
                whole += kWave + q * skip;
                if (e >= len) {
                    e -= len;
                    ++gg;
                    whole += skip;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (to[u] >= 0) buf[to[u]] = v[u];
        }
    };

    double A[T::TOT], preR[QA], prev[DD], prevL[NW];
#pragma unroll
    for (int i = 0; i < T::TOT; ++i) A[i] = 0.0;
#pragma unroll
    for (int r = 0; r < QA; ++r) preR[r] = 0.0;
#pragma unroll
    for (int c = 0; c < DD; ++c) prev[c] = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) prevL[i] = 0.0;
    const double tick = a.time && a.total > 0 ? 1.0 / (double)a.total : 0.0;
    const double* own = buf + g * sh.stride;
    // one row: half 0 moves all channels, 1 the lead half, 2 the lag half
    auto row = [&](auto half, int which, const double (&dl)[NW], const double (&dp)[DD], double t) {
        constexpr int H = decltype(half)::value;
        double zz[DD], zc[1], zuR[QA];
        zuR[0] = 0.0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const bool moves = which == 0 || (which == 1 ? lead[i] : lag[i]);
            const double z = clock[i] ? t : (moves ? dl[i] : 0.0);
            if (i == 0) zc[0] = z;
            else zuR[i - 1] = z;
        }
#pragma unroll
        for (int c = 0; c < DD; ++c) {
            if constexpr (kStatic) {
                // channel c of the transformed path: the lag half follows the lead half, an odd count has the time last
                const bool second = which != 0 && c >= DD / 2;
                const int ch = (LEADLAG || DD < 4) && second ? (c - DD / 2 < DD ? c - DD / 2 : 0) : c;
                const bool moves = which == 0 || (which == 2) == second;
                zz[c] = (a.time && c == DD - 1) ? t : (moves ? dp[ch] : 0.0);
            } else {
                zz[c] = 0.0;
            }
        }
        owned_levels<M, DD, M, 1, QC, T::TOT, QA, H>(A, QC, preR, zuR, zc, zz);
        prefix_levels<QC, QA>(QC, preR, zuR);
    };
    for (long c0 = 0; c0 <= step; c0 += sh.points) {
        const int count = (int)min((long)sh.points, step + 1 - c0);
        wave_sync();
        if (a.x_f32) stage(static_cast<const float*>(a.x), c0, count);
        else stage(static_cast<const double*>(a.x), c0, count);
        wave_sync();
        double cur[DD], curL[NW];
        auto read = [&](int j) {
#pragma unroll
            for (int i = 0; i < NW; ++i) curL[i] = own[j * d + at[i]];
            if constexpr (kStatic) {
                // (channels past d, of the time and of the lag half, read a number that is not used: the buffer is
                // longer by D)
#pragma unroll
                for (int c = 0; c < DD; ++c) cur[c] = own[j * d + c];
            }
        };
        int j = 0;
        read(0);
        if (c0 == 0) {                                          // the path's first point
#pragma unroll
            for (int i = 0; i < NW; ++i) prevL[i] = curL[i];
#pragma unroll
            for (int c = 0; c < DD; ++c) prev[c] = kStatic ? cur[c] : 0.0;
            j = 1;
            read(count > 1 ? 1 : 0);
        }
        // (segments past a piece's end do not move: by a difference of equal points they would where those are infinite)
        auto segments = [&](auto all, int end) {
            constexpr bool ALL = decltype(all)::value;
#pragma unroll(ALL ? 2 : 1)
            for (; j < end; ++j) {
                const bool inside = ALL || c0 + j <= mine;
                double dl[NW], dp[DD];
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    dl[i] = inside ? curL[i] - prevL[i] : 0.0;
                    prevL[i] = curL[i];
                }
#pragma unroll
                for (int c = 0; c < DD; ++c) {
                    dp[c] = kStatic && inside ? cur[c] - prev[c] : 0.0;
                    prev[c] = kStatic ? cur[c] : 0.0;
                }
                read(j + 1 < count ? j + 1 : j);
                const double t = inside ? tick : 0.0;
                if constexpr (LEADLAG) {
                    row(std::integral_constant<int, 1>(), 1, dl, dp, t);
                    row(std::integral_constant<int, 2>(), 2, dl, dp, t);
                } else {
                    bool both = true;
                    if constexpr (DT < 4) {
                        if (a.leadlag) {
                            row(std::integral_constant<int, 0>(), 1, dl, dp, t);
                            row(std::integral_constant<int, 0>(), 2, dl, dp, t);
                            both = false;
                        }
                    }
                    if (both) row(std::integral_constant<int, 0>(), 0, dl, dp, t);
                }
            }
        };
        segments(std::true_type(), (int)min((long)count, least - c0 + 1));
        segments(std::false_type(), count);
    }

    const long lenS = a.sig_len, base = b0 * lenS;
    if (sh.staged) {
        wave_sync();
        if (valid) store_signature<DD, M, 1, QC>(A, preR, buf + g * lenS, D, QC, ti, rest, blk);
        wave_sync();
        const int total = here * (int)lenS;
        if (a.out_f32) {
            float* out = static_cast<float*>(a.out) + base;
            for (int i = lane; i < total; i += kWave) out[i] = (float)buf[i];
        } else {
            double* out = static_cast<double*>(a.out) + base;
            for (int i = lane; i < total; i += kWave) out[i] = buf[i];
        }
    } else if (valid) {
        if (a.out_f32)
            store_signature<DD, M, 1, QC>(A, preR, static_cast<float*>(a.out) + base + g * lenS, D, QC, ti, rest, blk);
        else
            store_signature<DD, M, 1, QC>(A, preR, static_cast<double*>(a.out) + base + g * lenS, D, QC, ti, rest, blk);
    }
}

template <int DT, int M, int S, int QC, bool SHARED, bool LEADLAG>
__global__ __launch_bounds__(kWave * kWavesPerWG) void horner_kernel(const Args a)
{
    if constexpr (SHARED) {
        extern __shared__ double lds[];
        run_shared<DT, M, QC, LEADLAG>(a, lds);
    } else {
        run<DT, M, S, QC, LEADLAG>(a);
    }
}

// Increments of the transformed paths (Section 4), one row of Dpad doubles per segment: channels of the path (after
// the lead-lag transform: lead half, then lag half; a segment of the transformed path moves one half only, the lead
// first), then the time channel 1/n if asked for, then zero padding.  A path is stored as P pieces of np rows: piece p
// holds the segments p Lc .. p Lc + Lc - 1 (those below n), then zero rows.
// I: type of the entries' numbers.  Three divisions per entry are what the kernel is bound by: in 64 bits 13.0 us for
// 100000 paths of 10 points, where the entries' numbers fit 32 bits and are divided as such 10.7 us.
// zero: doubles to clear beside them (the backward pass's sums).
template <typename TI, typename I>
__global__ __launch_bounds__(256) void increments_kernel(const TI* __restrict__ x, double* __restrict__ dz,
                                                         double* __restrict__ zero, I total, long L,
                                                         int d, int D, int Dpad, long n, int P, long Lc, long np,
                                                         int time_aug, int lead_lag)
{
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (I)gridDim.x * blockDim.x) {
        const int c = (int)(i % (I)Dpad);
        const I bs = i / (I)Dpad;
        const long j = bs % (I)np;
        const I bp = bs / (I)np;
        const long piece = P == 1 ? 0 : (long)(bp % (I)P);
        const long b = P == 1 ? (long)bp : (long)(bp / (I)P);
        const long s = piece * Lc + j;
        double v = 0.0;
        if (j >= Lc || s >= n) {
            // a zero row: past the piece or past the path
        } else if (time_aug && c == D - 1) {
            v = 1.0 / (double)n;
        } else if (c < D) {
            long seg = s;
            int ch = c;
            bool moves = true;
            if (lead_lag) {
                seg = s >> 1;
                const bool lag_half = c >= d;
                ch = lag_half ? c - d : c;
                moves = ((s & 1) != 0) == lag_half;
            }
            if (moves) {
                const TI* xp = x + (b * L + seg) * d + ch;
                v = (double)xp[d] - (double)xp[0];
            }
        }
        dz[i] = v;
        if (zero) zero[i] = 0.0;
    }
}

template <int DT, int M, int S, int QC, bool SHARED>
hipError_t launch_one(const Args& a, long grid, hipStream_t st)
{
    const size_t lds = SHARED ? kWavesPerWG * sizeof(double) * shared_lds(a.PW, a.d, (int)(a.L < (1L << 20) ? a.L : 1L << 20), a.sig_len).doubles : 0;
    // kernels that skip the half of the channels a lead-lag segment does not move: where a lane has registers over
    // those channels at all (M >= 1) and at least four channels
    if constexpr (DT >= 4 && M >= 1) {
        if (a.leadlag) {
            hipLaunchKernelGGL((horner_kernel<DT, M, S, QC, SHARED, true>), dim3((unsigned)grid), dim3(kWave * kWavesPerWG), lds, st, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((horner_kernel<DT, M, S, QC, SHARED, false>), dim3((unsigned)grid), dim3(kWave * kWavesPerWG), lds, st, a);
    return hipGetLastError();
}

// prefix lengths up to kQExact have kernels of their own; longer ones share the kernel that tests against Q, which
// exists for the channel counts that can reach them (kLongPrefixMaxD).  Kernels whose waves hold several paths exist
// for prefixes up to kSharedMaxQ letters and up to kSharedMaxD channels (beyond that a path fills a wave anyway).
template <int DT, int M, int S>
hipError_t launch_variant(const Args& a, long grid, hipStream_t st)
{
    if (a.PW > 1) {
        // (a path has D^(Q + 1) lanes, and at most half a wave)
        if constexpr (DT <= kSharedMaxD) {
            if (a.Q == 0) return launch_one<DT, M, S, 0, true>(a, grid, st);
            if constexpr (DT * DT <= kWave / 2) {
                if (a.Q == 1) return launch_one<DT, M, S, 1, true>(a, grid, st);
            }
            if constexpr (DT * DT * DT <= kWave / 2) {
                if (a.Q == 2) return launch_one<DT, M, S, 2, true>(a, grid, st);
            }
        }
        return hipErrorInvalidValue;
    }
    switch (a.Q) {
    case 0: return launch_one<DT, M, S, 0, false>(a, grid, st);
    case 1: return launch_one<DT, M, S, 1, false>(a, grid, st);
    case 2: return launch_one<DT, M, S, 2, false>(a, grid, st);
    case 3: return launch_one<DT, M, S, 3, false>(a, grid, st);
    case 4: return launch_one<DT, M, S, 4, false>(a, grid, st);
    default:
        if constexpr (DT <= kLongPrefixMaxD) return launch_one<DT, M, S, kQMax, false>(a, grid, st);
        else return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_horner(int DT, int M, int S, const Args& a, long grid, hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    if ((a.np > 0 && !(a.np & 1)) || a.np < a.n || a.Q < 0 || a.Q > kQMax || a.LP <= 0 || a.WP * kWave < a.LP || a.NB * (long)S < (DT ? DT : a.D))
        return hipErrorInvalidValue;
    if (a.PW < 1 || (a.PW > 1 && (a.WP != 1 || a.PW * a.LP > kWave || a.NW * a.PW < a.B)) || (a.PW == 1 && a.NW != a.B * a.WP) ||
        grid * kWavesPerWG < a.NW)
        return hipErrorInvalidValue;
    // several paths per wave: lanes of one letter each, points of at most as many channels as a path has lanes
    if (a.PW > 1 && (!a.x || S != 1 || a.d < 1 || a.d > a.LP || a.NB != (DT ? DT : a.D) || a.L < 1 || a.P < 1 || (a.P & (a.P - 1)) || a.B % a.P))
        return hipErrorInvalidValue;
    if (a.leadlag && (a.n & 1)) return hipErrorInvalidValue;      // pieces of a lead-lag path start with a lead move
    if (DT == 0) return (M == 0 && S == 1) ? launch_variant<0, 0, 1>(a, grid, st) : hipErrorInvalidValue;
#define SG_CASE(D_, M_, S_) \
    if (DT == D_ && M == M_ && S == S_) return launch_variant<D_, M_, S_>(a, grid, st);
    SG_VARIANTS(SG_CASE)
#undef SG_CASE
    return hipErrorInvalidValue;
}

template <typename TI>
hipError_t launch_increments(const TI* x, double* dz, double* zero, long B, long L, int d, int D, int Dpad, long n, int P, long Lc,
                             long np, int time_aug, int lead_lag, hipStream_t st)
{
    if (P < 1 || np < Lc || P * Lc < n || (np > 0 && !(np & 1))) return hipErrorInvalidValue;
    const long total = B * P * np * Dpad;
    if (total <= 0) return hipSuccess;
    long grid = (total + 255) / 256;
    if (grid > 65536) grid = 65536;
    if (total < (1L << 31))       // (a step of the loop adds at most 2^24)
        hipLaunchKernelGGL((increments_kernel<TI, unsigned>), dim3((unsigned)grid), dim3(256), 0, st, x, dz, zero, (unsigned)total, L, d,
                           D, Dpad, n, P, Lc, np, time_aug, lead_lag);
    else
        hipLaunchKernelGGL((increments_kernel<TI, unsigned long>), dim3((unsigned)grid), dim3(256), 0, st, x, dz, zero,
                           (unsigned long)total, L, d, D, Dpad, n, P, Lc, np, time_aug, lead_lag);
    return hipGetLastError();
}

template hipError_t launch_increments<float>(const float*, double*, double*, long, long, int, int, int, long, int, long, long, int, int, hipStream_t);
template hipError_t launch_increments<double>(const double*, double*, double*, long, long, int, int, int, long, int, long, long, int, int, hipStream_t);

}  // namespace sg
