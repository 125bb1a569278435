// Paths cut into pieces (gfx950): from the signatures B_0, ..., B_{P-1} of a path's pieces, the signature of the whole
// path, and for the backward pass the signature up to the end of every piece and the adjoint there.
//
// Chen's identity (Proposition 2.2): the signature of the first p + 1 pieces is L_p = L_{p-1} (x) B_p, the one of those
// after p is R_p = B_{p+1} (x) R_{p+1}, both truncated at level N.  The entry of L_p at a word depends on entries of
// L_{p-1} at that word's prefixes only, the entry of R_p on entries at its suffixes: a lane takes a word of N letters,
// keeps the N values at its prefixes (or suffixes) in registers, and walks over the pieces with N (N + 1) / 2
// multiply-adds each, one per nonempty subword; shorter words ride along in the lanes whose other letters are all zero.
// The backward pass of a piece starts from L_p and from dF/dL_p, which is linear in the upstream gradient G of the whole
// signature: dF/dL_p[u] = sum_w G[u w] R_p[w], one launch for all pieces.
//
// What bounds this is launches and their latency, not arithmetic, so the pieces go in one launch rather than in a tree of
// pairwise products and of their adjoints.  (B, L, d, N) = (32, 1024, 5, 4) with time, 8 and 16 pieces: signature_bwd with
// the tree 138.6 us, so 91; signature_fwd 38.9 and 28.0.  (8000, 500, 2, 3), forward, 8 pieces: 71.4 and 40.3.  Against
// extended precision the errors are those of the tree (gradients 0.5 to 2.3e-15 of the largest).
#include <hip/hip_runtime.h>

#include "sg_kernels.h"

namespace sg {

namespace {

__host__ __device__ constexpr int tri(int n) { return n * (n + 1) / 2; }

struct PieceArgs {
    const double* pieces;    // [B][P][sig_len]
    double* prefix;          // [B][P][sig_len] L_p, or nullptr
    double* suffix;          // [B][P - 1][sig_len] R_p, or nullptr
    void* whole;             // [B][sig_len] L_{P-1}, float or double, or nullptr
    int whole_f32;
    long B, sig_len;
    int P;
    unsigned D, words;       // D^(N - 1)
    unsigned blocks;         // of C last (first) letters
    unsigned lv[16], pw[16]; // starts of the levels, powers of D
};

// A lane's words of N letters share N - 1 of them (the first ones of a prefix, the last ones of a suffix) and differ in C
// letters from c0 on: the subwords of the shared letters are loaded once for all of them.  With one word per lane the loads
// were the bound: 128 paths of 256 points, d = 4, level 6, in 4 pieces, forward, 72.6 us, with C = 4 55.6.
template <int N, int C, bool SUFFIX>
__device__ __forceinline__ void scan(const PieceArgs& a, long b, unsigned w, unsigned c0)
{
    constexpr int K = N - 1, V = tri(K) + C * N, U = V <= 16 ? 4 : (V <= 40 ? 2 : 1);   // pieces requested at once
    // number of the shared word's first j letters
    unsigned pre[K + 1];
#pragma unroll
    for (int j = K; j >= 0; --j) pre[j] = j == K ? w : pre[j + 1] / a.D;
    // entry of its subword of letters i .. j - 1
    auto sub = [&](int i, int j) { return a.lv[j - i] + pre[j] - pre[i] * a.pw[j - i]; };
    // entry of the word of m of the shared letters beside letter c: its last m and c, or c and its first m
    auto edge = [&](int m, unsigned c) {
        return SUFFIX ? a.lv[m + 1] + c * a.pw[m] + pre[m] : a.lv[m + 1] + (pre[K] - pre[K - m] * a.pw[m]) * a.D + c;
    };
    // the entry this lane writes for length k < N: the first (last) k shared letters, if the others are all zero
    auto writes = [&](int k) { return c0 == 0 && (SUFFIX ? pre[K - k] == 0 : w == pre[k] * a.pw[K - k]); };
    auto entry = [&](int k) { return SUFFIX ? sub(K - k, K) : sub(0, k); };
    const double* src = a.pieces + b * a.P * a.sig_len;
    double S[K + 1], top[C];         // S[k]: value at the first (last) k shared letters
    S[0] = 1.0;
    auto put = [&](auto* o) {
#pragma unroll
        for (int k = 1; k <= K; ++k)
            if (writes(k)) o[entry(k)] = S[k];
#pragma unroll
        for (int c = 0; c < C; ++c) o[edge(K, c0 + c)] = top[c];
        if (w == 0 && c0 == 0) o[0] = 1;
    };
    double* dst = SUFFIX ? a.suffix : a.prefix;
    // after q + 1 pieces from the end: what follows piece P - 2 - q
    auto keep = [&](int q) {
        if (dst) put(dst + (SUFFIX ? b * (a.P - 1) + a.P - 2 - q : b * a.P + q) * a.sig_len);
    };
    {
        const double* s = src + (SUFFIX ? a.P - 1 : 0) * a.sig_len;
#pragma unroll
        for (int k = 1; k <= K; ++k) S[k] = s[entry(k)];
#pragma unroll
        for (int c = 0; c < C; ++c) top[c] = s[edge(K, c0 + c)];
        keep(0);
    }
    const int count = SUFFIX ? a.P - 1 : a.P;
    for (int q0 = 1; q0 < count; q0 += U) {
        double v[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u < count ? q0 + u : count - 1;
            const double* s = src + (SUFFIX ? a.P - 1 - q : q) * a.sig_len;
#pragma unroll
            for (int i = 0; i < K; ++i)
#pragma unroll
                for (int j = i + 1; j <= K; ++j) v[u][tri(j - 1) + i] = s[sub(i, j)];
#pragma unroll
            for (int m = 0; m <= K; ++m) {
                double e[C];
                if constexpr (SUFFIX) {
#pragma unroll
                    for (int c = 0; c < C; ++c) e[c] = s[edge(m, c0 + c)];
                } else {
                    __builtin_memcpy(e, s + edge(m, c0), sizeof(e));     // C letters lie side by side
                }
#pragma unroll
                for (int c = 0; c < C; ++c) v[u][tri(K) + c * N + m] = e[c];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u;
            if (q < count) {
                // longest words first: they read the values before the step
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int m = 0; m <= K; ++m)     // the old value at m shared letters, the piece at the others
                        top[c] = __builtin_fma(S[m], v[u][tri(K) + c * N + K - m], top[c]);
#pragma unroll
                for (int k = K; k >= 1; --k) {
#pragma unroll
                    for (int m = 0; m < k; ++m)
                        S[k] = __builtin_fma(S[m], SUFFIX ? v[u][tri(K - m - 1) + K - k] : v[u][tri(k - 1) + m], S[k]);
                }
                keep(q);
            }
        }
    }
    if (!SUFFIX && a.whole) {
        if (a.whole_f32) put(static_cast<float*>(a.whole) + b * a.sig_len);
        else put(static_cast<double*>(a.whole) + b * a.sig_len);
    }
}

template <int N, int C>
__global__ __launch_bounds__(kWave) void scan_pieces_kernel(const PieceArgs a)
{
    const unsigned lanes = a.words * a.blocks;      // of a path; a block of letters for all shared words, then the next
    const long total = a.B * (long)lanes;
    for (long t = (long)blockIdx.x * kWave + threadIdx.x; t < total; t += (long)gridDim.x * kWave) {
        const long b = t / lanes;
        const unsigned r = (unsigned)(t - b * lanes);
        if (blockIdx.y) {
            const unsigned blk = r / a.words;
            scan<N, C, true>(a, b, r - blk * a.words, min(blk * C, a.D - C));     // (blocks may overlap: the same values)
        } else {
            const unsigned w = r / a.blocks;
            scan<N, C, false>(a, b, w, min((r - w * a.blocks) * C, a.D - C));
        }
    }
}

// start, shift and slots as in adjoint_slots.  The slots of all pieces follow each other: with workgroups of their own per piece and level, two pieces each of 5000 paths of 100 points in
// two channels, level 3, took signature_bwd 73.5 us, so 63.5; in four 73.7 and 50.9.
struct AdjointArgs {
    const double* suffix;    // [B][P - 1][sig_len]
    double* adj;             // [B][P][sig_len]
    long pieces, sig_len, slots;
    int P, N;
    unsigned lv[16], pw[16], start[16], shift[16];
};

template <typename TI, typename I>
__global__ __launch_bounds__(256) void piece_adjoints_kernel(const TI* __restrict__ gout, const AdjointArgs a)
{
    const I total = (I)a.pieces * (I)a.slots;
    for (I t = (I)blockIdx.x * 256 + threadIdx.x; t < total; t += (I)gridDim.x * 256) {
        const I bp = t / (I)a.slots;
        const unsigned slot = (unsigned)(t - bp * (I)a.slots);
        if (slot >= a.start[a.N + 1]) continue;
        int k = 1;
        while (slot >= a.start[k + 1]) ++k;
        const unsigned lanes = 1u << a.shift[k], u = (slot - a.start[k]) >> a.shift[k], lane = slot & (lanes - 1);
        const I b = bp / (I)a.P;
        const TI* g = gout + (long)b * a.sig_len;
        double acc = lane == 0 ? (double)g[a.lv[k] + u] : 0.0;         // the empty word
        if (bp - b * (I)a.P != (I)a.P - 1) {
            const double* r = a.suffix + (long)(bp - b) * a.sig_len;
            for (int j = 1; j <= a.N - k; ++j) {
                const unsigned cnt = a.pw[j];
                const TI* gj = g + a.lv[k + j] + u * cnt;
                const double* rj = r + a.lv[j];
                for (unsigned o = lane; o < cnt; o += lanes) acc = __builtin_fma((double)gj[o], rj[o], acc);
            }
            for (unsigned m = 1; m < lanes; m *= 2) acc += __shfl_xor(acc, (int)m, 64);     // (all lanes of a word are here)
        }
        if (lane == 0) a.adj[(long)bp * a.sig_len + a.lv[k] + u] = acc;
    }
}

bool levels(int D, int N, unsigned (&lv)[16], unsigned (&pw)[16])
{
    if (D < 1 || N < 1 || N > kPiecesMaxN) return false;
    unsigned long o = 0, q = 1;
    for (int k = 0; k <= N + 1; ++k) {
        if (o >= (1UL << 31)) return false;
        lv[k] = (unsigned)o;
        pw[k] = (unsigned)q;
        o += q;
        q *= (unsigned long)D;
    }
    return true;
}

template <int N>
hipError_t launch_scan(PieceArgs& a, hipStream_t st)
{
    // letters per lane: what loads least for all blocks of them
    auto loads = [&](int C) { return (long)((a.D + C - 1) / C) * (tri(N - 1) + C * N); };
    int C = 1;
    for (int c = 2; c <= 4 && c <= (int)a.D; ++c)
        if (loads(c) < loads(C)) C = c;
    a.blocks = (a.D + C - 1) / C;
    long gx = (a.B * (long)a.words * a.blocks + kWave - 1) / kWave;
    if (gx > (1L << 20)) gx = 1L << 20;
    const dim3 grid((unsigned)gx, a.suffix ? 2 : 1);
    switch (C) {
    case 1: hipLaunchKernelGGL((scan_pieces_kernel<N, 1>), grid, dim3(kWave), 0, st, a); break;
    case 2: hipLaunchKernelGGL((scan_pieces_kernel<N, 2>), grid, dim3(kWave), 0, st, a); break;
    case 3: hipLaunchKernelGGL((scan_pieces_kernel<N, 3>), grid, dim3(kWave), 0, st, a); break;
    default: hipLaunchKernelGGL((scan_pieces_kernel<N, 4>), grid, dim3(kWave), 0, st, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_scans(PieceArgs& a, int D, int N, hipStream_t st)
{
    if (a.B <= 0) return hipSuccess;
    if (a.P < 2 || !levels(D, N, a.lv, a.pw) || a.sig_len != (long)a.lv[N] + a.pw[N]) return hipErrorInvalidValue;
    a.D = (unsigned)D;
    a.words = a.pw[N - 1];
    switch (N) {
    case 1: return launch_scan<1>(a, st);
    case 2: return launch_scan<2>(a, st);
    case 3: return launch_scan<3>(a, st);
    case 4: return launch_scan<4>(a, st);
    case 5: return launch_scan<5>(a, st);
    case 6: return launch_scan<6>(a, st);
    case 7: return launch_scan<7>(a, st);
    case 8: return launch_scan<8>(a, st);
    case 9: return launch_scan<9>(a, st);
    case 10: return launch_scan<10>(a, st);
    case 11: return launch_scan<11>(a, st);
    case 12: return launch_scan<12>(a, st);
    case 13: return launch_scan<13>(a, st);
    case 14: return launch_scan<14>(a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_piece_product(const double* pieces, void* out, bool out_f32, long B, int P, int D, int N, long sig_len,
                                hipStream_t st)
{
    PieceArgs a = {};
    a.pieces = pieces; a.whole = out; a.whole_f32 = out_f32;
    a.B = B; a.P = P; a.sig_len = sig_len;
    return launch_scans(a, D, N, st);
}

hipError_t launch_piece_scans(const double* pieces, double* prefix, double* suffix, long B, int P, int D, int N, long sig_len,
                              hipStream_t st)
{
    PieceArgs a = {};
    a.pieces = pieces; a.prefix = prefix; a.suffix = suffix;
    a.B = B; a.P = P; a.sig_len = sig_len;
    return launch_scans(a, D, N, st);
}

template <typename TI>
hipError_t launch_piece_adjoints(const TI* gout, const double* suffix, double* adj, long B, int P, int D, int N, long sig_len,
                                 hipStream_t st)
{
    if (B <= 0) return hipSuccess;
    AdjointArgs a = {};
    if (P < 2 || !levels(D, N, a.lv, a.pw) || sig_len != (long)a.lv[N] + a.pw[N]) return hipErrorInvalidValue;
    a.suffix = suffix; a.adj = adj; a.pieces = B * P; a.sig_len = sig_len; a.P = P; a.N = N;
    a.slots = (long)adjoint_slots(D, N, a.start, a.shift);
    const long total = a.pieces * a.slots;
    long grid = (total + 255) / 256;
    if (grid > (1L << 20)) grid = 1L << 20;
    if (total < (1L << 31))      // (a step of the loop adds at most 2^28)
        hipLaunchKernelGGL((piece_adjoints_kernel<TI, unsigned>), dim3((unsigned)grid), dim3(256), 0, st, gout, a);
    else
        hipLaunchKernelGGL((piece_adjoints_kernel<TI, unsigned long>), dim3((unsigned)grid), dim3(256), 0, st, gout, a);
    return hipGetLastError();
}

template hipError_t launch_piece_adjoints<float>(const float*, const double*, double*, long, int, int, int, long, hipStream_t);
template hipError_t launch_piece_adjoints<double>(const double*, const double*, double*, long, int, int, int, long, hipStream_t);

}  // namespace sg
