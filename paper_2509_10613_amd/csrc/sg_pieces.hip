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
// the tree 138.6 us, so 98.9; signature_fwd 38.9 and 29.4.  (8000, 500, 2, 3), forward, 8 pieces: 71.4 and 40.3.  Against
// extended precision the errors are those of the tree (gradients 0.5 to 2.3e-15 of the largest).
#include <hip/hip_runtime.h>

#include "sg_kernels.h"

namespace sg {

namespace {

__host__ __device__ constexpr int tri(int n) { return n * (n + 1) / 2; }

struct PieceArgs {
    const double* pieces;    // [B][P][sig_len]
    double* prefix;          // [B][P][sig_len] L_p, or nullptr
    double* suffix;          // [B][P][sig_len] R_p, p < P - 1, or nullptr
    void* whole;             // [B][sig_len] L_{P-1}, float or double, or nullptr
    int whole_f32;
    long B, sig_len;
    int P;
    unsigned D, words;       // D^N
    unsigned lv[16], pw[16]; // starts of the levels, powers of D
};

template <int N, bool SUFFIX>
__device__ __forceinline__ void scan(const PieceArgs& a, long b, unsigned w)
{
    constexpr int U = pieces_batch(N);     // requested before the arithmetic that reads them
    // number of the word's first j letters
    unsigned pre[N + 1];
#pragma unroll
    for (int j = N; j >= 0; --j) pre[j] = j == N ? w : pre[j + 1] / a.D;
    // entry of the subword of letters i .. j - 1
    auto sub = [&](int i, int j) { return a.lv[j - i] + pre[j] - pre[i] * a.pw[j - i]; };
    // the entry this lane writes for length k: its first (last) k letters, if the others are all zero
    auto entry = [&](int k) { return SUFFIX ? sub(N - k, N) : sub(0, k); };
    auto writes = [&](int k) { return SUFFIX ? pre[N - k] == 0 : w == pre[k] * a.pw[N - k]; };
    const double* src = a.pieces + b * a.P * a.sig_len;
    double S[N + 1];         // S[k]: value at the first (last) k letters
    S[0] = 1.0;
#pragma unroll
    for (int k = 1; k <= N; ++k) S[k] = 0.0;
    const int count = SUFFIX ? a.P - 1 : a.P;
    for (int q0 = 0; q0 < count; q0 += U) {
        double v[U][tri(N)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u < count ? q0 + u : count - 1;
            const double* s = src + (SUFFIX ? a.P - 1 - q : q) * a.sig_len;
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int j = i + 1; j <= N; ++j) v[u][tri(j - 1) + i] = s[sub(i, j)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u;
            if (q < count) {
                // longest words first: they read the values before the step
#pragma unroll
                for (int k = N; k >= 1; --k) {
#pragma unroll
                    for (int m = 0; m < k; ++m)      // m letters of the old value, k - m of the piece
                        S[k] = __builtin_fma(S[m], SUFFIX ? v[u][tri(N - m - 1) + N - k] : v[u][tri(k - 1) + m], S[k]);
                }
                double* dst = SUFFIX ? a.suffix : a.prefix;
                if (dst) {
                    // after q + 1 pieces from the end: what follows piece P - 2 - q
                    double* o = dst + (b * a.P + (SUFFIX ? a.P - 2 - q : q)) * a.sig_len;
#pragma unroll
                    for (int k = 1; k <= N; ++k)
                        if (writes(k)) o[entry(k)] = S[k];
                    if (w == 0) o[0] = 1.0;
                }
            }
        }
    }
    if (!SUFFIX && a.whole) {
        auto put = [&](auto* o) {
#pragma unroll
            for (int k = 1; k <= N; ++k)
                if (writes(k)) o[entry(k)] = S[k];
            if (w == 0) o[0] = 1;
        };
        if (a.whole_f32) put(static_cast<float*>(a.whole) + b * a.sig_len);
        else put(static_cast<double*>(a.whole) + b * a.sig_len);
    }
}

template <int N>
__global__ __launch_bounds__(kWave) void scan_pieces_kernel(const PieceArgs a)
{
    const long total = a.B * (long)a.words;
    for (long t = (long)blockIdx.x * kWave + threadIdx.x; t < total; t += (long)gridDim.x * kWave) {
        const long b = t / a.words;
        const unsigned w = (unsigned)(t - b * a.words);
        if (blockIdx.y) scan<N, true>(a, b, w);
        else scan<N, false>(a, b, w);
    }
}

// Words of k letters sum over 1 + D + ... + D^(N - k) terms: one lane, eight lanes or a wave per word (shift[k] = 0, 3, 6),
// in workgroups from block[k] on.
struct AdjointArgs {
    const double* suffix;    // [B][P][sig_len]
    double* adj;             // [B][P][sig_len]
    long pieces, sig_len;
    int P, N;
    unsigned lv[16], pw[16], block[16], shift[16];
};

template <typename TI>
__global__ __launch_bounds__(256) void piece_adjoints_kernel(const TI* __restrict__ gout, const AdjointArgs a)
{
    int k = 1;
    while (blockIdx.x >= a.block[k + 1]) ++k;
    const unsigned lanes = 1u << a.shift[k];
    const unsigned slot = (blockIdx.x - a.block[k]) * 256 + threadIdx.x;
    const unsigned u = slot >> a.shift[k], lane = slot & (lanes - 1);
    if (u >= a.pw[k]) return;                              // (all lanes of a word together)
    for (long bp = blockIdx.y; bp < a.pieces; bp += gridDim.y) {
        const long b = bp / a.P;
        const TI* g = gout + b * a.sig_len;
        double acc = 0.0;
        if (bp - b * a.P == a.P - 1) {
            acc = (double)g[a.lv[k] + u];
        } else {
            const double* r = a.suffix + bp * a.sig_len;
            if (lane == 0) acc = (double)g[a.lv[k] + u];   // the empty word
            for (int j = 1; j <= a.N - k; ++j) {
                const unsigned cnt = a.pw[j];
                const TI* gj = g + a.lv[k + j] + u * cnt;
                const double* rj = r + a.lv[j];
                for (unsigned o = lane; o < cnt; o += lanes) acc = __builtin_fma((double)gj[o], rj[o], acc);
            }
            for (unsigned m = 1; m < lanes; m *= 2) acc += __shfl_xor(acc, (int)m, 64);
        }
        if (lane == 0) a.adj[bp * a.sig_len + a.lv[k] + u] = acc;
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
hipError_t launch_scan(const PieceArgs& a, dim3 grid, hipStream_t st)
{
    hipLaunchKernelGGL(scan_pieces_kernel<N>, grid, dim3(kWave), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_scans(PieceArgs& a, int D, int N, hipStream_t st)
{
    if (a.B <= 0) return hipSuccess;
    if (a.P < 2 || !levels(D, N, a.lv, a.pw) || a.sig_len != (long)a.lv[N] + a.pw[N]) return hipErrorInvalidValue;
    a.D = (unsigned)D;
    a.words = a.pw[N];
    long gx = (a.B * (long)a.words + kWave - 1) / kWave;
    if (gx > (1L << 20)) gx = 1L << 20;
    const dim3 grid((unsigned)gx, a.suffix ? 2 : 1);
    switch (N) {
    case 1: return launch_scan<1>(a, grid, st);
    case 2: return launch_scan<2>(a, grid, st);
    case 3: return launch_scan<3>(a, grid, st);
    case 4: return launch_scan<4>(a, grid, st);
    case 5: return launch_scan<5>(a, grid, st);
    case 6: return launch_scan<6>(a, grid, st);
    case 7: return launch_scan<7>(a, grid, st);
    case 8: return launch_scan<8>(a, grid, st);
    case 9: return launch_scan<9>(a, grid, st);
    case 10: return launch_scan<10>(a, grid, st);
    case 11: return launch_scan<11>(a, grid, st);
    case 12: return launch_scan<12>(a, grid, st);
    case 13: return launch_scan<13>(a, grid, st);
    case 14: return launch_scan<14>(a, grid, st);
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
    unsigned long blocks = 0;
    for (int k = 1; k <= N; ++k) {
        const unsigned terms = a.lv[N - k] + a.pw[N - k];
        a.shift[k] = terms <= 8 ? 0 : (terms <= 64 ? 3 : 6);
        a.block[k] = (unsigned)blocks;
        blocks += (((unsigned long)a.pw[k] << a.shift[k]) + 255) / 256;
    }
    a.block[N + 1] = (unsigned)blocks;
    if (blocks > 0x7fffffffUL) return hipErrorInvalidValue;
    const unsigned gy = (unsigned)(a.pieces < 65535 ? a.pieces : 65535);
    hipLaunchKernelGGL(piece_adjoints_kernel<TI>, dim3((unsigned)blocks, gy), dim3(256), 0, st, gout, a);
    return hipGetLastError();
}

template hipError_t launch_piece_adjoints<float>(const float*, const double*, double*, long, int, int, int, long, hipStream_t);
template hipError_t launch_piece_adjoints<double>(const double*, const double*, double*, long, int, int, int, long, hipStream_t);

}  // namespace sg
