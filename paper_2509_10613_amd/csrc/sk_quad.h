// Shared by the kernels that work on four path pairs per wavefront, 16 lanes each (sk_quad.hip forward,
// sk_four.hip backward): lane exchange inside a row of 16 lanes, and the sequence of quads a launch works through.
#pragma once
#include <hip/hip_runtime.h>

#include "sk_dev.h"
#include "sk_kernels.h"

namespace sk {

// lane i of a row of 16 lanes receives v of lane i - 1; the row's first lane receives edge (its own lane's value)
__device__ __forceinline__ real row_from_above_or(real v, real edge)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    int elo = __double2loint(edge), ehi = __double2hiint(edge);
    lo = __builtin_amdgcn_update_dpp(elo, lo, 0x111, 0xf, 0xf, false);
    hi = __builtin_amdgcn_update_dpp(ehi, hi, 0x111, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// lane i of a row of 16 lanes receives v of lane i + 1; the row's last lane receives edge (its own lane's value)
__device__ __forceinline__ real row_from_below_or(real v, real edge)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    int elo = __double2loint(edge), ehi = __double2hiint(edge);
    lo = __builtin_amdgcn_update_dpp(elo, lo, 0x101, 0xf, 0xf, false);
    hi = __builtin_amdgcn_update_dpp(ehi, hi, 0x101, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
// the same; the row's last lane receives zero
__device__ __forceinline__ real row_from_below(real v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_update_dpp(0, lo, 0x101, 0xf, 0xf, true);
    hi = __builtin_amdgcn_update_dpp(0, hi, 0x101, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Quad q of the sequence a launch works through: row yi of the Gram matrix in groups of four x paths, rows in
// ascending order.  A row has N pairs, or, for a symmetric Gram matrix K(X, X), the yi + 1 pairs n <= yi.
struct QuadCursor {
    long yi, xi0, npr;
    __device__ __forceinline__ void locate(const SweepArgs& a, long u)
    {
        if (!a.tri) {
            const long per_row = (a.gramN + kQuadPairs - 1) / kQuadPairs;
            yi = u / per_row;
            xi0 = (u - yi * per_row) * kQuadPairs;
            npr = a.gramN;
        } else {
            // rows 4 j .. 4 j + 3 hold j + 1 quads each: 2 j (j + 1) quads lie before row 4 j
            long j = (long)((sqrt(2.0 * (double)u + 1.0) - 1.0) * 0.5);
            while (2 * (j + 1) * (j + 2) <= u) ++j;
            while (2 * j * (j + 1) > u) --j;
            const long rest = u - 2 * j * (j + 1);
            yi = 4 * j + rest / (j + 1);
            xi0 = (rest % (j + 1)) * kQuadPairs;
            npr = yi + 1;
        }
    }
    __device__ __forceinline__ void next(const SweepArgs& a)
    {
        xi0 += kQuadPairs;
        if (xi0 >= npr) {
            xi0 = 0;
            ++yi;
            if (a.tri) npr = yi + 1;
        }
    }
};

// The quads a wavefront works through: an equal share of the first qd_even of them, then, until the sequence ends, one
// at a time from the launch's counter (zero at launch).  Two wavefronts on a SIMD do not share it evenly (the older one
// goes first): with equal shares of everything the favoured one is done early and leaves the other alone at two thirds of
// the SIMD's rate (Gram 256 x 256 backward, L = 128, order 1, d = 3: 4.1 -> 3.6 ms).  A grab is a round trip to one
// address for all wavefronts (20 ns each there), so short launches have equal shares only.
struct QuadQueue {
    QuadCursor cur;
    long u, u1;
    __device__ __forceinline__ QuadQueue(const SweepArgs& a, long slot, long nslots)
    {
        u = slot * a.qd_even / nslots;
        u1 = (slot + 1) * a.qd_even / nslots;
        if (u < u1) cur.locate(a, u);
        else grab(a);
    }
    __device__ __forceinline__ void grab(const SweepArgs& a)
    {
        u1 = u = a.qd_nquads;
        if (a.qd_even >= a.qd_nquads) return;
        int at = 0;
        if ((threadIdx.x & 63) == 0) at = atomicAdd(a.bd_flags, 1);
        const long got = a.qd_even + __builtin_amdgcn_readfirstlane(at);
        if (got >= a.qd_nquads) return;
        u = got;
        u1 = u + 1;
        cur.locate(a, u);
    }
    __device__ __forceinline__ bool more() const { return u < u1; }
    __device__ __forceinline__ void next(const SweepArgs& a)
    {
        if (++u < u1) cur.next(a);
        else grab(a);
    }
};

}  // namespace sk
