// Kernel arguments and launchers of the truncated-signature path (Section 2.3), shared by the entry points and the
// kernel file.
#pragma once
#include <hip/hip_runtime.h>

#include "sg_plan.h"

namespace sg {

struct Args {
    const double* dz;   // [B][np][Dpad] increments of the transformed paths, rows n..np-1 zero (not read if PW > 1)
    void* out;          // [B][sig_len], float if out_f32, else double
    int out_f32;
    long B;
    long n;             // segments per path
    long np;            // stored rows per path: n rounded up to an odd number (0 if n = 0)
    int D, Dpad, N, Q, NB;
    long LP, WP;        // lanes and waves per path
    long sig_len;
    int PW;             // paths per wave (1, or several short paths side by side in a wave: then WP = 1)
    long NW;            // waves of the launch
    int leadlag;        // rows alternate between moves of the lead and of the lag half of the channels (n is even)
    // several paths per wave: the kernel reads the points themselves
    const void* x;      // [B / P][L][d], float if x_f32, else double
    int x_f32;
    long L;
    int d, time;        // channels of the points, 1 if the time channel follows
    long total;         // segments of a whole path; piece p of its P pieces holds those from p n on
    int P;              // a power of two
};

struct BwdArgs {
    const double* dz;    // [B][np][Dpad] increments of the transformed paths
    double* gz;          // [B][np][Dpad] dF/dz: zero on entry and accumulated by atomics, unless a path is one wave's
    const void* sig;     // [B][sig_len] signatures of the whole paths, float if sig_f32, else double
    const void* gout;    // [B][sig_len] upstream gradient, likewise
    int sig_f32, gout_f32;
    long B;
    long n, np;
    int D, Dpad, N, Q, NB;
    long LP, WP;
    long sig_len;
    size_t lds_wave;     // doubles of LDS per wave
    int PW;              // paths per wave (several short paths side by side: then WP = 1)
    long NW;             // waves of the launch
    int leadlag;         // rows alternate between moves of the lead and of the lag half of the channels (n is even)
};

hipError_t launch_horner(int DT, int M, int S, const Args& a, long grid, hipStream_t st);
hipError_t launch_horner_bwd(int DT, int M, int S, const BwdArgs& a, long grid, size_t lds_bytes, hipStream_t st);
// a.Q = N - 2, a.WP and a.NW in wavefronts of this kernel; a.NB, a.LP, a.PW, a.lds_wave and a.leadlag are not read
hipError_t launch_horner_bwd_matrix(const BwdArgs& a, int S, long grid, hipStream_t st);

template <typename TO>
hipError_t launch_point_gradients(const double* gz, TO* gx, long B, long L, int d, int Dpad, int P, long Lc, long np,
                                  int lead_lag, hipStream_t st);

// zero: as many doubles to clear on the way, or nullptr
template <typename TI>
hipError_t launch_increments(const TI* x, double* dz, double* zero, long B, long L, int d, int D, int Dpad, long n, int P, long Lc,
                             long np, int time_aug, int lead_lag, hipStream_t st);

// Signatures of P pieces per path, sig_len entries each (levels 0..N over D channels): their product, float or double;
// or the products of the first p + 1 pieces and of the pieces after p (p < P - 1), for every p; and the adjoint of the
// former from the upstream gradient of the whole (levels 1..N).
hipError_t launch_piece_product(const double* pieces, void* out, bool out_f32, long B, int P, int D, int N, long sig_len,
                                hipStream_t st);
hipError_t launch_piece_scans(const double* pieces, double* prefix, double* suffix, long B, int P, int D, int N, long sig_len,
                              hipStream_t st);
template <typename TI>
hipError_t launch_piece_adjoints(const TI* gout, const double* suffix, double* adj, long B, int P, int D, int N, long sig_len,
                                 hipStream_t st);

}  // namespace sg
