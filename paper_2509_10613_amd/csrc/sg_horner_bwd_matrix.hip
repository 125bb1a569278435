// Gradient of batched truncated signatures (paper Section 2.4) with the top level's sum over words on the matrix cores, for
// gfx950.
//
// Walking a path backwards (sg_horner_bwd.hip), the adjoints Ab_N of the entries of the top level never change: nothing is
// computed from these entries.  With G_t[w] the chain value of the word w of N - 1 letters at segment t, their share of the
// gradient is
//     dF/dz_t[c] += sum_w G_t[w] Ab_N[w c],
// over sixteen segments at a time a matrix product.  So a lane has one or two words w = u c of N - 1 letters (the last
// letters of a prefix u side by side over 4, 8 or 16 lanes), their rows of Ab_N once for its own arithmetic and, other
// words' rows, once as the operand of v_mfma_f64_16x16x4_f64, and goes through the path sixteen segments at a time:
//
//  * segment by segment, everything per lane: the entries at w and its prefixes before the segment (the step with the
//    increment negated), G_t[w], its adjoint sum_c Ab_N[w c] z_t[c] (increments in scalar registers), and the adjoints of
//    levels 1 .. N - 1, where, as in the other kernel, the adjoints of the carried prefixes are shares that are never summed;
//  * the shares of dF/dz at the letters of w are summed over lanes through LDS four segments at a time;
//  * G goes through LDS, from lanes of words to lanes of segments, and the product adds up what the whole wavefront has.
//
// The other kernel sums dF/dz over its lanes segment by segment, 24 LDS instructions each, and is bound by them; here the
// sums wait for no LDS round trip of their own segment.  (128 paths of 1024 points, 16 channels, level 4) as a whole call:
// 2.19 -> 1.48 ms; (128, 256, 7, 4): 203 -> 109 us.  Bound by fp64 issue, vector and matrix together: the two do not overlap
// (the adjoints Ab_N z as sixteen more matrix instructions per sixteen segments, and the last letters' sums as products with
// unit vectors, took 3.9 ms).  Two wavefronts per SIMD, which costs sixteen channels 92 bytes per lane of scratch: one, with
// all of the register file, takes 2.0 ms there.
#include <hip/hip_runtime.h>

#include "sg_dev.h"
#include "sg_kernels.h"
#include "sk_kernels.h"

namespace sg {

namespace {

typedef double double4v __attribute__((ext_vector_type(4)));

template <int D, int Q, int S>
__global__ __launch_bounds__(kWave * kWavesPerWG, 2) void horner_bwd_matrix_kernel(const BwdArgs a)
{
    constexpr int DP = matrix_lanes(D, S), NP = kWave / DP;   // lanes per prefix, prefixes of the wavefront
    constexpr int T = kMatrixSteps, F = kMatrixFlush;
    static_assert(T == 16 && F == 4 && Q >= 1 && DP <= 16 && DP >= F, "sixteen segments at a time, sums every four");
    extern __shared__ double lds[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    long wg = blockIdx.x;
    if (gridDim.x % kXcds == 0) wg = (long)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    const long wt = wg * kWavesPerWG + wave;
    if (wt >= a.NW) return;
    const long b = wt / a.WP;
    const int w0 = (int)(wt - b * a.WP) * NP;             // the wavefront's first prefix
    constexpr int NU = ipow(D, Q);
    double* zs = lds + (size_t)wave * matrix_lds_doubles(S);  // [T][16]: gradients of the sixteen segments
    double* fb = zs + T * 16;                             // [F][64], column ^ 9 row: one value per segment and lane
    double* gb = fb + F * kWave;                          // [S][T][64], column ^ row: the chain values

    const int g = lane >> 4, i = lane & 15;
    // word s of lane l: prefix w0 + l / DP, last letter (l % DP) S + s
    const int blk = lane % DP;
    const bool inside = w0 + lane / DP < NU;
    const int u = inside ? w0 + lane / DP : 0;
    int uR[Q], cs[S];
    bool valid[S];
    {
        int t = u;
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            uR[r] = t % D;
            t /= D;
        }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
        valid[s] = inside && blk * S + s < D;
        cs[s] = min(blk * S + s, D - 1);
    }
    auto lvl = [](int k) {
        long o = 0, p = 1;
        for (int j = 0; j < k; ++j) {
            o += p;
            p *= D;
        }
        return o;
    };
    // the adjoints of the top level: of the lane's own words, and of word s of lane 16 g + k at channel i
    double top[S][D], b2[S][16];
    double A[S], Ab[S], preR[Q], prb[Q];
    const long own = lvl(Q + 1) + (long)u * D;
    auto load_sig = [&](const auto* sig) {
#pragma unroll
        for (int s = 0; s < S; ++s) A[s] = (double)sig[own + cs[s]];
        int pw = 1;
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            preR[r] = (double)sig[lvl(Q - r) + u / pw];
            pw *= D;
        }
    };
    auto load_gout = [&](const auto* gout) {
        const auto* gt = gout + lvl(Q + 2);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const auto* o = gt + ((long)u * D + cs[s]) * D;
#pragma unroll
            for (int c = 0; c < D; ++c) top[s][c] = (double)o[c];
#pragma unroll
            for (int c = 0; c < D; ++c) top[s][c] = valid[s] ? top[s][c] : 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int uw = w0 + (16 * g + k) / DP, cw = k % DP * S + s;
                const bool ok = uw < NU && cw < D && i < D;
                const double v = (double)gt[ok ? ((long)uw * D + cw) * D + i : 0];
                b2[s][k] = ok ? v : 0.0;
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const double v = (double)gout[own + cs[s]];
            Ab[s] = valid[s] ? v : 0.0;
        }
        int pw = 1;
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            // one lane starts with the upstream value
            prb[r] = (inside && blk == 0 && u % pw == 0) ? (double)gout[lvl(Q - r) + u / pw] : 0.0;
            pw *= D;
        }
    };
    if (a.sig_f32) load_sig(static_cast<const float*>(a.sig) + b * a.sig_len);
    else load_sig(static_cast<const double*>(a.sig) + b * a.sig_len);
    if (a.gout_f32) load_gout(static_cast<const float*>(a.gout) + b * a.sig_len);
    else load_gout(static_cast<const double*>(a.gout) + b * a.sig_len);
    const double* zrow = a.dz + b * a.np * a.Dpad;
    double* grow = a.gz + b * a.np * a.Dpad;
    const long n = a.n;
    if (n <= 0) return;

    // increments of one segment: all of them in scalar registers, those at the lane's own letters in vector registers
    struct Inc {
        double z[D], c[S], u[Q];
    };
    auto fetch = [&](long row, Inc& v) {
        const double* zp = zrow + row * a.Dpad;
        uniform_ptr zu = (uniform_ptr)(zp);
#pragma unroll
        for (int c = 0; c < D; ++c) v.z[c] = zu[c];
#pragma unroll
        for (int s = 0; s < S; ++s) v.c[s] = zp[cs[s]];
#pragma unroll
        for (int r = 0; r < Q; ++r) v.u[r] = zp[uR[r]];
    };
    // four segments first .. first + 3 backwards, of the sixteen the segments t0 .. t0 + 3
    auto four = [&](long first, int t0, Inc& v, double (&zub)[F][Q], double (&zcb)[F][S]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = F - 1; f >= 0; --f) {
            Inc next;
            const long row = first + f - 1;
            fetch(row > 0 ? row : 0, next);
            const int t = t0 + f;
            double nzc[S], nzu[Q], unused[D], gP = 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) nzc[s] = -v.c[s];
#pragma unroll
            for (int r = 0; r < Q; ++r) {
                nzu[r] = -v.u[r];
                zub[f][r] = 0.0;
            }
            // the entries before the segment: the forward step with the increment negated
            owned_levels<0, D, 0, S, Q, S, Q>(A, Q, preR, nzu, nzc, unused);
            prefix_levels<Q, Q>(Q, preR, nzu);
            // the adjoint of the forward step, levels 1 .. N - 1
            prefix_levels_rev<Q, Q>(Q, preR, v.u, prb, zub[f]);
            double h[Q + 1], hb = 0.0;
            gP = prefix_chain_keep<1, Q, Q>(Q, preR, v.u, h);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                hb = __builtin_fma(Ab[s], v.c[s], hb);
                zcb[f][s] = Ab[s] * gP;
            }
            prefix_chain_rev<1, Q, Q>(Q, v.u, h, hb, prb, zub[f]);
            // level N: the chain value of each word and its adjoint
            const double g0 = 0.5 * prefix_chain_keep<2, Q, Q>(Q, preR, v.u, h);
            hb = 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                gb[(s * T + t) * kWave + (lane ^ t)] = __builtin_fma(g0, v.c[s], A[s]);
                double p0 = top[s][0] * v.z[0], p1 = top[s][1] * v.z[1];
#pragma unroll
                for (int c = 2; c < D; ++c) {
                    double& p = c & 1 ? p1 : p0;
                    p = __builtin_fma(top[s][c], v.z[c], p);
                }
                const double P = p0 + p1;
                Ab[s] += P;
                zcb[f][s] = __builtin_fma(P, g0, zcb[f][s]);
                hb = __builtin_fma(P, v.c[s], hb);
            }
            prefix_chain_rev<2, Q, Q>(Q, v.u, h, 0.5 * hb, prb, zub[f]);
            v = next;
        }
    };
    // one value per lane of four segments to LDS, and the four of one segment a lane takes from there
    const int ft = lane % F;
    auto exchange = [&](const auto& put, int col, int stride, double (&got)[F]) __attribute__((always_inline)) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int f = 0; f < F; ++f) fb[f * kWave + (lane ^ (9 * f))] = put(f);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < F; ++k) got[k] = fb[ft * kWave + ((col + k * stride) ^ (9 * ft))];
    };
    const int zc_blk = lane / F % DP, zc_part = lane / (F * DP);        // letters: the prefixes F zc_part .. + 3
    const int zu_pre = lane / F % NP, zu_part = lane / (F * NP);        // prefixes: the lanes F zu_part .. + 3 of one
    int zu_letter[Q];
    {
        int t = w0 + zu_pre < NU ? w0 + zu_pre : 0;                     // (beyond the last prefix the sums are zero)
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            zu_letter[r] = t % D;
            t /= D;
        }
    }

    // Sixteen segments first .. first + 15 at a time from the path's end.  The last ones may begin before the path: such
    // segments repeat the first increment after all others are done, and what they give is not written (nothing of one
    // segment enters the sums of another).
    Inc v;
    fetch(n - 1, v);
    for (long first = n - T; first > -T; first -= T) {
#pragma unroll
        for (int k = 0; k < 4; ++k) zs[k * kWave + lane] = 0.0;
        for (int t0 = T - F; t0 >= 0 && first + t0 > -F; t0 -= F) {
            double zub[F][Q], zcb[F][S];
            four(first + t0, t0, v, zub, zcb);
            // The shares at the letters: over the lanes with the same last letters, over the lanes of a prefix.  (LDS
            // executes a wavefront's instructions in order: one buffer serves all of them without a wait in between.)
            double got[S + Q][F];
#pragma unroll
            for (int s = 0; s < S; ++s)
                exchange([&](int f) { return zcb[f][s]; }, (zc_part * F) * DP + zc_blk, DP, got[s]);
#pragma unroll
            for (int r = 0; r < Q; ++r)
                exchange([&](int f) { return zub[f][r]; }, zu_pre * DP + zu_part * F, 1, got[S + r]);
            __builtin_amdgcn_wave_barrier();
            double* zsum = zs + (t0 + ft) * 16;
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (zc_blk * S + s < D) unsafeAtomicAdd(&zsum[zc_blk * S + s], (got[s][0] + got[s][1]) + (got[s][2] + got[s][3]));
#pragma unroll
            for (int r = 0; r < Q; ++r)
                unsafeAtomicAdd(&zsum[zu_letter[r]], (got[S + r][0] + got[S + r][1]) + (got[S + r][2] + got[S + r][3]));
        }
        __builtin_amdgcn_wave_barrier();
        // Z[t, c] = sum_w G_t[w] Ab_N[w c]: lane (g, t) holds segment t of the words of lanes 16 g .. 16 g + 15
        double4v Z[2] = {double4v{0.0, 0.0, 0.0, 0.0}, double4v{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (k % DP * S + s < D)
                    Z[k & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(gb[(s * T + i) * kWave + ((16 * g + k) ^ i)], b2[s][k], Z[k & 1], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long row = first + g + 4 * r;
            if (row >= 0 && i < D) unsafeAtomicAdd(&grow[row * a.Dpad + i], zs[(g + 4 * r) * 16 + i] + (Z[0][r] + Z[1][r]));
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int D, int S>
hipError_t launch_matrix_q(const BwdArgs& a, long grid, hipStream_t st)
{
    const size_t lds = (size_t)kWavesPerWG * matrix_lds_doubles(S) * sizeof(double);
    auto kernel = a.Q == 1 ? &horner_bwd_matrix_kernel<D, 1, S> : (a.Q == 2 ? &horner_bwd_matrix_kernel<D, 2, S> : &horner_bwd_matrix_kernel<D, 3, S>);
    if (hipError_t e = sk::allow_full_lds(reinterpret_cast<const void*>(kernel)); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kWave * kWavesPerWG), lds, st, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_matrix(const BwdArgs& a, int S, long grid, hipStream_t st)
{
    return S == 1 ? launch_matrix_q<D, 1>(a, grid, st) : launch_matrix_q<D, 2>(a, grid, st);
}

}  // namespace

hipError_t launch_horner_bwd_matrix(const BwdArgs& a, int S, long grid, hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    // what the kernel assumes about the launch
    if (a.D < kMatrixMinD || a.D > 16 || a.Q < 1 || a.Q > kMatrixMaxQ || a.N != a.Q + 2 || a.Dpad < a.D || a.np < a.n || a.n < 0 ||
        a.sig_len != sig_length(a.D, a.N) || S < 1 || S > 2 || a.WP != matrix_waves(a.D, a.Q, S) || a.NW != a.B * a.WP || grid * kWavesPerWG < a.NW)
        return hipErrorInvalidValue;
    switch (a.D) {
        case 5: return launch_matrix<5>(a, S, grid, st);
        case 6: return launch_matrix<6>(a, S, grid, st);
        case 7: return launch_matrix<7>(a, S, grid, st);
        case 8: return launch_matrix<8>(a, S, grid, st);
        case 9: return launch_matrix<9>(a, S, grid, st);
        case 10: return launch_matrix<10>(a, S, grid, st);
        case 11: return launch_matrix<11>(a, S, grid, st);
        case 12: return launch_matrix<12>(a, S, grid, st);
        case 13: return launch_matrix<13>(a, S, grid, st);
        case 14: return launch_matrix<14>(a, S, grid, st);
        case 15: return launch_matrix<15>(a, S, grid, st);
        case 16: return launch_matrix<16>(a, S, grid, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sg
