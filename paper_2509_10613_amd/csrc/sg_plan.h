// Host-side launch plan for batched truncated signatures by Horner's scheme (paper Section 2.3): pure arithmetic,
// no HIP calls, so that the workspace query, the description and the launch agree by construction.
//
// How the update of Section 2.3 is spread over lanes.  One step of Horner's algorithm updates every level k by
//     A_k[w c] += G_k[w] z[c],   G_k[v c'] = G_k[v] z[c'] / (k - |v|) + A_{|v|+1}[v c'],   G_k[empty] = 1,
// for words w of length k - 1 (the nesting of Section 2.3 read word by word: G_k[w] = B_k[w] + A_{k-1}[w]).  The value
// at a word depends only on values at its prefixes, so the entries of the signature whose words start with a given
// prefix u form a closed system.  A lane owns a prefix u of Q letters, a block of S consecutive next letters, and
// every word that continues them up to M further letters: S (D^(M+1) - 1)/(D - 1) numbers, kept in registers for all
// steps of the path; it also carries the Q entries at the prefixes of u (every lane under the same prefix carries the
// same copies).  A step needs no communication between lanes.  Lanes of one wave belong to one path, so the
// increment z of a step is the same for the whole wave and is fetched by scalar loads.
#pragma once
#include <cstddef>
#include <cstdint>

namespace sg {

constexpr int kWave = 64;
constexpr int kWavesPerWG = 4;
constexpr int kXcds = 8;
constexpr int kQMax = 8;            // longest carried prefix
constexpr int kQExact = 4;          // prefix lengths with code of their own
constexpr int kLongPrefixMaxD = 9;   // channel counts whose variants also exist for prefixes longer than kQExact
constexpr int64_t kSimds = 1024;       // 256 compute units of 4 SIMDs
constexpr int kMinPiece = 12;          // fewest segments a piece of a path is cut down to
constexpr int kMaxPieces = 1024;
constexpr int kPiecesMaxN = 14;        // deepest level with a kernel that multiplies pieces: kQMax letters, one, and five owned
constexpr int kSharedMaxQ = 2;         // waves that hold several paths: longest prefix and most channels with such kernels
constexpr int kSharedMaxD = 9;

// (channels, owned depth M, letter block S), per channel count in order of falling register use.
#define SG_VARIANTS(X)                                                                                     \
    X(2, 5, 1) X(2, 4, 1) X(2, 3, 1) X(2, 2, 1) X(2, 1, 1)                                                 \
    X(3, 3, 1) X(3, 2, 1) X(3, 1, 1)                                                                       \
    X(4, 3, 1) X(4, 2, 1) X(4, 1, 1)                                                                       \
    X(5, 2, 1) X(5, 1, 1) X(6, 2, 1) X(6, 1, 1) X(7, 2, 1) X(7, 1, 1) X(8, 2, 1) X(8, 1, 1) X(9, 2, 1) X(9, 1, 1) \
    X(10, 1, 5) X(11, 1, 4) X(12, 1, 4) X(13, 1, 4) X(14, 1, 4) X(15, 1, 4) X(16, 1, 4) X(17, 1, 4)

// Variants of the backward kernels: a lane also holds the adjoints of its entries, so the subtrees are smaller.
#define SG_BWD_VARIANTS(X)                                                                                 \
    X(2, 4, 1) X(2, 3, 1) X(2, 2, 1) X(2, 1, 1)                                                            \
    X(3, 3, 1) X(3, 2, 1) X(3, 1, 1)                                                                       \
    X(4, 2, 2) X(4, 2, 1) X(4, 1, 1)                                                                       \
    X(5, 2, 1) X(5, 1, 1) X(6, 2, 1) X(6, 1, 3) X(6, 1, 1) X(7, 1, 4) X(7, 1, 1) X(8, 1, 4) X(8, 1, 1)     \
    X(9, 1, 3) X(9, 1, 1)                                                                                  \
    X(10, 1, 2) X(11, 1, 2) X(12, 1, 2) X(13, 1, 2) X(14, 1, 2) X(15, 1, 2) X(16, 1, 2) X(17, 1, 2)
constexpr int kBwdLongPrefixMaxD = 5;   // as kLongPrefixMaxD, for the backward variants
constexpr int kBwdMaxRuntimeD = 1024;   // run-time channel count kernel, backward: per-channel sums of a wave live in LDS

struct Variant { int D, M, S; };
#define SG_ROW(D, M, S) {D, M, S},
constexpr Variant kVariants[] = {SG_VARIANTS(SG_ROW)};
constexpr Variant kBwdVariants[] = {SG_BWD_VARIANTS(SG_ROW)};
#undef SG_ROW

// Backward with the top level's sum over words on the matrix cores (sg_horner_bwd_matrix.hip): lanes of one or two words of
// N - 1 letters, the last letter over 4, 8 or 16 lanes, sixteen segments at a time.
constexpr int kMatrixMinD = 5, kMatrixMaxQ = 3, kMatrixSteps = 16, kMatrixFlush = 4;
constexpr int matrix_lanes(int D, int S)                           // per prefix, S last letters each
{
    int l = kMatrixFlush;
    while (l * S < D) l *= 2;
    return l;
}
constexpr int matrix_lds_doubles(int S) { return kMatrixSteps * 16 + kMatrixFlush * kWave + S * kMatrixSteps * kWave; }   // per wave
inline int64_t matrix_waves(int64_t D, int Q, int S)               // per path
{
    int64_t prefixes = 1;
    for (int i = 0; i < Q; ++i) prefixes *= D;
    const int64_t per_wave = kWave / matrix_lanes((int)D, S);
    return (prefixes + per_wave - 1) / per_wave;
}
// Two words per lane once one word each gives more than a wavefront per SIMD: they share the arithmetic of their prefix, but
// are half as many wavefronts.  signature_bwd, one and two words (B, L, D, N): (128, 512, 8, 4) 200 and 249 us, (128, 512,
// 16, 3) 191 and 199; (128, 512, 12, 4) 529 and 489, (128, 1024, 16, 4) 1832 and 1476.
inline int matrix_words(int64_t VB, int64_t D, int Q) { return VB * matrix_waves(D, Q, 1) > kSimds ? 2 : 1; }
// Where the matrix kernel is taken.  From eleven channels and words of at most three letters on always: (1000, 65, 11, 4)
// 357 us by the other kernel, 322 by this one, (1000, 65, 14, 4) 848 and 555, (4000, 65, 12, 3) 254 and 176, (8000, 17, 16,
// 3) 206 and 184.  Below, the matrix instruction's sixteen columns are half empty, and four letters leave most of the time
// in the chains over the prefix, which the other kernel spreads over more words of a lane: there only while the chip is not
// full and a segment's latency counts, up to two wavefronts per SIMD: (500, 65, 8, 4) 67 and 60, (128, 256, 7, 4) 203 and
// 109, (128, 256, 5, 5) 220 and 197; but (2000, 65, 8, 4) 164 and 195, (4000, 65, 5, 3) 99 and 138, (128, 512, 8, 5) 552 and
// 741.  Lead-lag paths, where the other kernel leaves out the half that stands still (L points, twice the segments): (128,
// 512, 8, 4) 1904 and 1398, (128, 256, 4, 4) 280 and 199, (500, 65, 3, 4) 115 and 89, (16, 300, 5, 5) 638 and 462; only with
// eight channels and five levels, where its waves come out even, it stays ahead of more than one wavefront per SIMD: (28,
// 300, 4, 5) 451 and 290, (37, 300, 4, 5) 436 and 456, (64, 300, 4, 5) 437 and 458.
inline bool matrix_pays(int64_t VB, int64_t D, int N, int64_t segments, bool lead_lag)
{
    if (D < kMatrixMinD || D > 16 || N < 3 || N - 2 > kMatrixMaxQ || segments < kMatrixSteps) return false;
    if (D >= 11 && N <= 4) return true;
    const int64_t most = lead_lag && D == 8 && N == 5 ? kSimds : 2 * kSimds;
    return VB * matrix_waves(D, N - 2, matrix_words(VB, D, N - 2)) <= most;
}
// Pieces of long paths for the matrix kernel (make_plan): segments from which a path is long, the least of a piece, and the
// entries of a signature up to which more pieces are worth their products.  With more of the matrix kernel's waves than half
// of the chip's SIMDs such paths go by the other kernel's: (B, L, D, N) = (128, 1024, 5, 4), 1 and 4 pieces, 350 and 171 us.
constexpr int64_t kMatrixCut = 160;    // fewest segments of a path that is cut for the matrix kernel
constexpr int pieces_batch(int N) { return N <= 3 ? 4 : (N <= 5 ? 2 : 1); }   // pieces a lane of the product asks for at once
// Forward, estimated us: a segment's latency, the launch of the product, and in it the latency of a batch and a piece's word
constexpr int kSharedPiece = 40;
constexpr double kSegmentBwd = 0.75, kSegmentMatrix = 0.35, kPieceWordBwd = 2.8e-5;   // backward, forward part included
constexpr double kSegment = 0.2, kProduct = 4.0, kPieceLatency = 0.6, kPieceWord = 0.9e-5;
constexpr int64_t kMatrixLong = 768, kMatrixPiece = 120, kMatrixPieceEntries = 100000;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// LDS of a wave that holds PW paths (forward): their points in chunks, `stride` doubles per path (odd: the paths of a wave
// then start in different banks), and in their place, if it fits, the finished signatures.  At most kSharedLds doubles and
// the few past the end that the last point's missing channels are read from: five workgroups per compute unit.  Signatures
// are worth twice that, two workgroups: 300000 paths of 5 points in 2 channels to level 5, double, 64.6 us stored word by
// word, 38.8 through LDS.
constexpr int kSharedLds = 1024, kSharedStage = 2048;
struct SharedLds { int points, stride, doubles; bool staged; };
#ifdef __HIP__
__host__ __device__
#endif
inline SharedLds shared_lds(int PW, int d, int L, int64_t sig_len)
{
    SharedLds s;
    int points = (kSharedLds / PW - 1) / d;       // (at least 15: a path has at least d lanes)
    s.points = points < L ? points : L;
    s.stride = (s.points * d) | 1;
    s.staged = sig_len <= kSharedStage / PW;
    const int pts = PW * s.stride + kSharedMaxD, sig = s.staged ? PW * (int)sig_len : 0;
    s.doubles = pts > sig ? pts : sig;
    return s;
}

// Adjoints of the pieces: words of k letters sum over 1 + D + ... + D^(N - k) terms, with a wave, eight lanes or one lane per
// word (shift[k] = 6, 3, 0, falling with k), slots start[k] .. start[k + 1] - 1.  Returns the slots of a piece, a multiple of the
// largest group and fewer than 2^31: so many words have fewer lanes each.  (Signatures of fewer than 2^31 entries.)
inline uint64_t adjoint_slots(int D, int N, unsigned (&start)[16], unsigned (&shift)[16])
{
    for (unsigned most = 6;; most -= 3) {
        uint64_t slots = 0, words = 1, terms[16], t = 0, pw = 1;
        for (int j = 0; j < N; ++j, pw *= (uint64_t)D) terms[N - j] = t += pw;
        for (int k = 1; k <= N; ++k) {
            const unsigned lanes = terms[k] <= 8 ? 0 : (terms[k] <= 64 ? 3 : 6);
            shift[k] = lanes < most ? lanes : most;
            start[k] = (unsigned)slots;
            words *= (uint64_t)D;
            slots += words << shift[k];
        }
        start[N + 1] = (unsigned)slots;
        slots = align_up(slots, (size_t)1 << shift[1]);
        if (slots < ((uint64_t)1 << 31) || most == 0) return slots;
    }
}

// Backward, kernels for a channel count and a prefix length: whether a path's lanes are one wave's.
constexpr bool lone_wave(int D, int S, int Q)
{
    if (Q > kQExact) return false;
    int lanes = (D + S - 1) / S;
    for (int i = 0; i < Q; ++i) lanes *= D;
    return lanes <= kWave;
}

struct Plan {
    bool valid = false;
    const char* why = "";
    int64_t B = 0, L = 0;
    int d = 0;            // channels of the caller's paths
    int D = 0;            // channels after the transformations
    int N = 0;
    int64_t n = 0;        // segments after the transformations
    int64_t np = 0;       // increment rows stored per piece: its segments, then zero rows up to an odd count
    int P = 1;            // pieces per path (forward only): the signatures of the pieces are multiplied afterwards
    int64_t Lc = 0;       // segments per piece
    int64_t VB = 0;       // pieces in the batch: B * P, each one a path of its own to the Horner kernel
    int DT = 0;           // kernel template channel count (0: run-time channel count, M = 0, S = 1)
    int M = 0, S = 1, Q = 0, NB = 1;
    int64_t LP = 0;       // lanes per path: D^Q * NB
    int64_t WP = 0;       // waves per path
    int PW = 1;           // paths per wave (forward): short paths side by side in one wave
    int64_t waves = 0;
    int64_t grid = 0;
    int Dpad = 0;         // doubles per stored increment row
    int64_t sig_len = 0;  // entries per path, level 0 included
    int io_elem = 8;
    size_t off_dz = 0, total = 0;
    size_t off_t0 = 0;    // signatures of the pieces (P > 1); backward: then the adjoints at their ends
    size_t off_t1 = 0;    // backward: signatures of the pieces up to each one and after it
    // backward
    bool backward = false;
    size_t lds_wave = 0;      // doubles of LDS per wave
    size_t lds_bytes = 0;
    size_t off_gz = 0, off_sig = 0;
    bool matrix = false;             // the top level on the matrix cores; launch shape of that kernel:
    int matrix_Q = 0, matrix_S = 1;
    int64_t matrix_WP = 0, matrix_waves = 0, matrix_grid = 0;
};

// entries of levels 0..N over D channels; 0 if that does not fit in 2^40
inline int64_t sig_length(int64_t D, int N)
{
    if (D < 1 || N < 0) return 0;
    const int64_t lim = (int64_t)1 << 40;
    int64_t tot = 0, p = 1;
    for (int k = 0; k <= N; ++k) {
        tot += p;
        if (tot > lim) return 0;
        if (k < N) {
            if (p > lim / D) return 0;
            p *= D;
        }
    }
    return tot;
}

// force_M >= 0 / force_S > 0 pick the variant with that owned depth / letter block (diagnostics and tests);
// -1 / 0 = the estimate below decides
// backward: the plan of signature_bwd (have_sig: the caller passes the signatures, else they are computed into the
// workspace first, with the forward plan for the same arguments)
inline Plan make_plan(int64_t B, int64_t L, int64_t d, int N, bool time_aug, bool lead_lag, bool io_double,
                      int force_M = -1, bool backward = false, bool have_sig = false, int force_S = 0,
                      int force_P = 0,   // force_P: 0 = the plan decides, else the number of pieces (a power of two)
                      int force_W = 0)   // force_W: 1 = a wave never holds more than one path
{
    Plan p;
    p.backward = backward;
    p.B = B; p.L = L; p.d = (int)d; p.N = N;
    p.io_elem = io_double ? 8 : 4;
    const int64_t D = (lead_lag ? 2 * d : d) + (time_aug ? 1 : 0);
    p.D = (int)D;
    p.n = L < 1 ? 0 : (lead_lag ? 2 * (L - 1) : L - 1);
    p.Lc = p.n;
    p.np = p.n == 0 ? 0 : (p.n | 1);
    p.VB = B;
    p.sig_len = sig_length(D, N);
    if (p.sig_len == 0) { p.why = "the signature has more than 2^40 entries per path"; return p; }
    if (B > 0 && p.sig_len > ((int64_t)1 << 46) / B) { p.why = "the batch of signatures has more than 2^46 entries"; return p; }
    if (B > 0 && p.np * (D + 1) > ((int64_t)1 << 44) / B) { p.why = "the batch of increments has more than 2^44 entries"; return p; }

    auto lanes = [&](int M, int S, int64_t& LP, int& Q, int& NB) -> bool {
        Q = N - M - 1;
        if (Q < 0 || Q > kQMax) return false;
        if (Q > kQExact && M > 0 && D > (backward ? kBwdLongPrefixMaxD : kLongPrefixMaxD)) return false;
        NB = (int)((D + S - 1) / S);
        LP = NB;
        for (int i = 0; i < Q; ++i) {
            if (LP > ((int64_t)1 << 40) / D) return false;
            LP *= D;
        }
        return true;
    };
    double step_cycles = 0.0;     // estimate for a step of all paths, by choose
    auto choose = [&](int64_t Bsel) -> bool {
        // The variant with the least estimated time.  A lane executes about `instr` vector instructions per step: the
        // multiply-adds of its owned levels and their chains, the chains over the carried prefix for each owned level,
        // the updates of the carried entries, and a fixed part for loads and loop control.  A SIMD issues one such
        // instruction per 4 clocks when it has several waves and per about 5 clocks when it has a single one, and the
        // waves of the launch are spread over kSimds SIMDs.
        bool have = false;
        double best = 0.0;       // (0 without a variant: the run-time channel count)
        const Variant* list = backward ? kBwdVariants : kVariants;
        const size_t nlist = backward ? sizeof(kBwdVariants) / sizeof(Variant) : sizeof(kVariants) / sizeof(Variant);
        for (size_t vi = 0; vi < nlist; ++vi) {
            const Variant& v = list[vi];
            if (v.D != D || (force_M >= 0 && v.M != force_M) || (force_S > 0 && v.S != force_S)) continue;
            int64_t LP; int Q, NB;
            if (!lanes(v.M, v.S, LP, Q, NB)) continue;
            // lane groups of at most half a wave can share a wave (forward kernels for few channels and letters)
            const int pw = (LP <= kWave / 2 && Q <= kSharedMaxQ && D <= kSharedMaxD && force_W != 1) ? (int)(kWave / LP) : 1;
            const int64_t waves = pw > 1 ? (Bsel + pw - 1) / pw : Bsel * ((LP + kWave - 1) / kWave);
            double owned = 0.0, lvl = v.S, sum = 0.0;
            for (int m = 0; m <= v.M; ++m) {
                sum += lvl;        // nodes of levels 0..m
                owned += sum;      // the update of owned level m touches all of them once
                lvl *= (double)D;
            }
            // several paths per wave: the increments are loaded per lane; backward, a lane per path and channel reads the
            // LDS rows of its path
            const double instr = owned + (v.M + 1) * (2.0 * Q + 1.0) + (double)Q * Q + 12.0 + (pw > 1 ? (double)D : 0.0) +
                                 (pw > 1 && backward ? (double)LP : 0.0);
            const double rounds = (double)((waves + kSimds - 1) / kSimds);
            const double cost = rounds * instr * (waves <= kSimds ? 5.0 : 4.0);
            if (!have || cost < best) {
                best = cost;
                p.DT = v.D; p.M = v.M; p.S = v.S; p.Q = Q; p.NB = NB; p.LP = LP; p.PW = pw;
                have = true;
            }
        }
        if (!have && force_M > 0) { p.why = "no kernel with the requested subtree depth for this number of channels and level"; return false; }
        if (!have) {
            int64_t LP; int Q, NB;
            if (!lanes(0, 1, LP, Q, NB)) { p.why = "truncation level too high for this number of channels (a lane carries at most 8 prefix letters)"; return false; }
            p.DT = 0; p.M = 0; p.S = 1; p.Q = Q; p.NB = NB; p.LP = LP;
            p.PW = (!backward && LP <= kWave / 2 && Q <= kSharedMaxQ && force_W != 1) ? (int)(kWave / LP) : 1;
        }
        p.WP = (p.LP + kWave - 1) / kWave;
        step_cycles = best;
        return true;
    };
    if (!choose(B)) return p;
    const bool may_matrix = backward && force_M < 0 && force_S == 0 && force_W == 0;   // (no kernel of the others asked for)
    // Few long paths leave most SIMDs without a wave: cut every path into P pieces of Lc segments, let the Horner
    // kernel treat the pieces as paths, and multiply the signatures of the pieces afterwards (Chen's identity,
    // Proposition 2.2).  Backward: the products up to and after every piece give the signature and the adjoint that the
    // backward kernel starts a piece from.
    if (p.n > 0) {
        int P = 1;
        if (force_P > 0) {
            P = force_P;
        } else if (B > 0 && p.sig_len < ((int64_t)1 << 31) && !backward) {
            // The number with the least estimated time: a segment takes kSegment us, that long after the one before it
            // has asked for its increments, or what all waves of a SIMD issue; a piece costs its latency and the
            // multiply-adds of its words in the product, and the product a launch.  1, 2, 4, ... pieces, in us, (B, L, d, N)
            // = (40, 2048, 7, 5): 565, 298, 174; (16, 1024, 16, 4), from 4: 110, 122, 173; (200, 100, 3, 3): 19.9, 14.2,
            // 10.4, 8.8; (4, 1024, 8, 3), from 8: 30.9, 21.1, 16.7, 18.4; (128, 1024, 5, 4), from 4: 57.6, 42.8, 36.3, 39.2.
            const double words = (double)B * ((double)(p.sig_len - 1) * (double)(D - 1) / (double)D + 1.0);
            double best = 0.0;
            for (int q = 1; q <= kMaxPieces && (q == 1 || p.n / q >= kMinPiece); q *= 2) {
                if (q == 1 && p.n < 2 * kMinPiece) break;
                if (p.sig_len > ((int64_t)1 << 44) / (B * q) || !choose(B * q)) break;
                const double issue = step_cycles / 2400.0;
                const double t = (double)p.n / q * (issue > kSegment ? issue : kSegment) +
                                 (q > 1 ? kProduct + q * (kPieceLatency / pieces_batch(N) + words * kPieceWord) : 0.0);
                if (q == 1 || t < best) {
                    best = t;
                    P = q;
                }
            }
            if (!choose(B)) return p;
        } else if (B > 0 && p.sig_len < ((int64_t)1 << 31)) {
            // Backward: cut while that leaves at most four waves per SIMD, from less than half a wave per SIMD.  The matrix
            // kernel has more waves for the same words and takes a third of the time of the other per segment, so it cuts
            // later.  Waves of many paths have sums of as many paths per segment, and stop at one wave per SIMD, two with long pieces: (8000, 500, 2, 3),
            // from 1: 285, 271, 221, 251; (3000, 200, 3, 2): 103, 101, 80, 82.  The others: 1, 2, 4, ... pieces, in us, (B, L, d, N) = (100, 200, 4, 3), from 2: 115, 69, 44, 34; (200, 100, 3, 3): 71,
            // 58, 38, 30; (500, 500, 3, 4), from 4: 156, 113, 109, 131; matrix kernel: (64, 1024, 6, 4), from 2: 283, 165, 139,
            // 128; (4, 1024, 8, 3), from 8: 72, 47, 36, 38; (64, 128, 12, 3): 44, 57, 46, 52.
            // No further than twice as many save segments' time over what the words of their products take: (128, 256, 4, 6),
            // whole and in 8 pieces, 170 and 274.
            const double words = (double)B * ((double)(p.sig_len - 1) * (double)(D - 1) / (double)D + 1.0);
            auto pieces = [&](int64_t w1, int64_t want, int64_t least, double segment) {
                int q = 1;
                if (w1 < kSimds / 2)
                    while (q < kMaxPieces && w1 * 2 * q <= want && p.n / (2 * q) >= least &&
                           (double)p.n / (2 * q) * segment > q * words * kPieceWordBwd) q *= 2;
                return q;
            };
            const int64_t w1 = p.PW > 1 ? (B + p.PW - 1) / p.PW : B * p.WP;
            if (may_matrix && matrix_pays(B, D, N, p.n, lead_lag)) {
                if (p.n >= kMatrixCut) P = pieces(B * matrix_waves(D, N - 2, 1), 3 * kSimds, kMatrixSteps, kSegmentMatrix);
                const int q = p.n >= kMatrixLong && p.sig_len < kMatrixPieceEntries ? pieces(w1, 2 * kSimds - 1, kMatrixPiece, kSegmentMatrix) : 1;
                if (q > P) P = q;
            } else if (p.n >= 4 * kMinPiece) {
                P = pieces(w1, p.PW > 4 ? kSimds : 4 * kSimds, kMinPiece, kSegmentBwd);
                if (p.PW > 4) {
                    const int q = pieces(w1, 2 * kSimds, kSharedPiece, kSegmentBwd);
                    if (q > P) P = q;
                }
            }
        }
        if (P > 1) {
            if ((P & (P - 1)) != 0 || P > kMaxPieces) { p.why = "the number of pieces must be a power of two up to 1024"; return p; }
            if (p.sig_len >= ((int64_t)1 << 31)) { p.why = "paths are cut into pieces only for signatures of fewer than 2^31 entries"; return p; }
            if (B > 0 && (p.sig_len > ((int64_t)1 << 44) / (B * P))) { p.why = "too many pieces for this signature size"; return p; }
            p.P = P;
            p.Lc = (p.n + P - 1) / P;
            if (lead_lag) p.Lc += p.Lc & 1;      // a piece starts with a move of the lead half
            p.np = p.Lc | 1;
            p.VB = B * P;
            if (!choose(p.VB)) return p;
        }
    }
    // Forward, fewer paths than fill the chip: fewer in a wave, on more of its SIMDs, so that a wave copies less in a row.
    // Waves full and spread: (B, L, d, N) = (1000, 100, 6, 2) 23.9 and 14.5 us, (20, 2000, 2, 2) 38.4 and 23.5,
    // (5000, 64, 4, 3) with time 27.2 and 19.1.
    if (!backward && p.PW > 2 && p.VB < (int64_t)p.PW * kSimds) {
        const int64_t even = (p.VB + kSimds - 1) / kSimds;
        p.PW = even > 2 ? (int)even : 2;
    }
    p.waves = p.PW > 1 ? (p.VB + p.PW - 1) / p.PW : p.VB * p.WP;
    p.grid = (p.waves + kWavesPerWG - 1) / kWavesPerWG;
    if (p.grid > 0x7fffffffLL) { p.why = "too many workgroups"; return p; }
    p.Dpad = (int)align_up((size_t)D, 2);
    size_t off = 0;
    p.off_dz = off;      // (kernels that hold several paths per wave read the points; the backward ones read increments always)
    if (backward || p.PW == 1) off = align_up(off + (size_t)p.VB * (size_t)p.np * p.Dpad * sizeof(double), 256);
    if (!backward) {
        if (p.P > 1) {
            p.off_t0 = off;
            off = align_up(off + (size_t)p.VB * (size_t)p.sig_len * sizeof(double), 256);
        }
    } else {
        if (p.DT == 0 && D > kBwdMaxRuntimeD) { p.why = "backward: more than 1024 channels"; return p; }
        if (may_matrix && matrix_pays(p.VB, D, N, p.Lc, lead_lag)) {
            p.matrix_Q = N - 2;
            p.matrix_S = matrix_words(p.VB, D, p.matrix_Q);
            p.matrix_WP = matrix_waves(D, p.matrix_Q, p.matrix_S);
            p.matrix_waves = p.VB * p.matrix_WP;
            p.matrix_grid = (p.matrix_waves + kWavesPerWG - 1) / kWavesPerWG;
            p.matrix = p.matrix_grid <= 0x7fffffffLL;
        }
        const bool uniform = p.DT > 0 && p.M > 0;
        p.lds_wave = (size_t)p.Dpad + (uniform ? (size_t)kWave * (size_t)(D | 1) : 0);
        p.lds_bytes = (size_t)kWavesPerWG * p.lds_wave * sizeof(double);
        p.off_gz = off;      // dF/dz, one row per stored increment row
        off = align_up(off + (size_t)p.VB * (size_t)p.np * p.Dpad * sizeof(double), 256);
        p.off_sig = off;     // signatures in double, if the caller has none
        if (p.P == 1 && !have_sig) off = align_up(off + (size_t)B * (size_t)p.sig_len * sizeof(double), 256);
        if (p.P > 1) {
            const size_t pieces = (size_t)p.VB * (size_t)p.sig_len * sizeof(double);
            p.off_t0 = off;
            off = align_up(off + pieces, 256);
            p.off_t1 = off;      // (nothing follows a path's last piece)
            off = align_up(off + 2 * pieces - (size_t)B * (size_t)p.sig_len * sizeof(double), 256);
        }
    }
    p.total = off < 256 ? 256 : off;
    p.valid = true;
    return p;
}

}  // namespace sg
