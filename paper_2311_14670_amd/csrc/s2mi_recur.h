// s2mi_recur.h -- device helpers of the descending-m Wigner recursion shared by
// the fused FP64 sweeps (s2mi_sweep.hip) and the d-tile generator of the
// matrix-core path (s2mi_mfma.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace s2mi {

constexpr int RT = 700;   // realise once the scale exponent is above -RT (a multiple of 4)
constexpr int SG = 8;     // degrees (or rings) per register chunk
// Renormalisation period of the recursion (orders; a power of two).  The state grows
// by at most |kappa lambda| + 1 < 2^20 per order for L <= 4096 (|lambda| sin theta <=
// |n| + m + 1 with kappa (|n| + m + 1) <= 181 over every degree below 4096, and
// sin theta >= 1.9e-4 on every grid's swept rings), so between passes a pair left at or
// below 2^-600 stays below 2^-280: far from overflow, and its unscaled contribution
// negligible (see renorm).
constexpr int RN = 16;

__device__ __forceinline__ int ufl(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Tile order of the matrix-core contractions.  Workgroups are dispatched round-robin
// over the 8 XCDs (workgroup i to XCD i mod 8), each with its own L2.  With xcd set, a
// 1-D grid of ceil(gx gy gz / 8) * 8 workgroups is remapped so that every XCD takes one
// contiguous run of the tiles, ordered z fastest, then x, then y: tiles that share an
// operand along x (and every z) then read it through one L2, while each XCD still
// gets tiles of every z.  Without xcd, workgroup i is tile i in x-fastest order.
// Returns false for the padding of the grid.
constexpr int NXCD = 8;
__device__ __forceinline__ bool xcd_tile(int gx, int gy, int gz, int &bx, int &by, int &bz, bool xcd = true)
{
    const int T = gx * gy * gz;
    const int i = (int)blockIdx.x;
    if (!xcd) {
        if (i >= T) return false;
        bx = i % gx;
        const int r = i / gx;
        by = r % gy;
        bz = r / gy;
        return true;
    }
    const int per = (T + NXCD - 1) / NXCD;
    const int j = (i % NXCD) * per + i / NXCD;
    if (j >= T) return false;
    bz = j % gz;
    const int r = j / gz;
    bx = r % gx;
    by = r / gx;
    return true;
}

// State of one recursion slot: the pair (e, ep) and an int E, the slot's values
// being e 2^E and ep 2^E.  Realised (E = 0): e is the value itself.  Not yet realised:
// E < 0 and the pair is kept scaled to at most 2^-600 at each pass, so a sweep can use
// e unscaled in its contraction -- such a slot then contributes at most 2^-280 times its
// record (the growth between two passes of the sweeps is below 2^320) instead of its
// exact (equally negligible) value, and no exponent scaling is needed per step.  So
// records 2^220 times those that matter at a ring are still below rounding there; with
// both bounds 2^100 higher, at the same cost, 2^120 times them was the limit.  A slot
// that has not started holds zeros with E = 0.

// Exact power-of-two renormalisation of the pair (e, ep) carrying exponent E
// (running renormalisation, Sec. 3.4).  Nothing is due while the pair is below 2^-600
// (its value then is below that too): the 2^100 between that and the scale it is brought
// back to spares most passes the rescaling.  Above, a pair whose value is below 2^-RT is
// rescaled so its larger entry is in [2^-RT, 2^(4-RT)), E absorbing the change, and one
// whose value is at least 2^-RT is realised (E = 0, unscaled from then on).  Every
// scaling is by a power of two, so the values themselves never change; every E is a
// multiple of 4 (the sweeps store E / 4 in 16 bits: log2 of a start value is at least
// 2 l log2 sin(theta / 2) > -2^17 for L <= 4096 on every grid's swept rings).
__device__ __forceinline__ void renorm(double &e, double &ep, int &E)
{
    const double mx = fmax(fabs(e), fabs(ep));
    if (E < 0 && mx > 0x1p-600) {
        // floor(log2 mx) = frexp exponent - 1 (mx is finite: the state grows by a bounded
        // factor between passes)
        const int k = __builtin_amdgcn_frexp_exp(mx) - 1;
        const bool real = (E + k >= -RT);               // the value's exponent is E + k
        const int k4 = k & ~3;
        const int sh = real ? E : -k4 - RT;
        e = ldexp(e, sh);
        ep = ldexp(ep, sh);
        E = real ? 0 : E + k4 + RT;                      // < 0: E + k < -RT
    }
}

// A run's values at the rings and orders that the other run supplies (below) are rounding
// errors grown like the second solution of the recursion, without bound: at more than 51
// orders of up to 2^20 each they could overflow, and an infinity times the zeros that stand
// for those rings in the forward sums is NaN.  Runs of |n| > DROP_AN therefore drop a pair
// beyond 2^400 every RN orders below |n| (a value that is used is at most 1, e within
// some 2^10 of it), so nothing passes 2^720.
constexpr int DROP_AN = 32;
__device__ __forceinline__ void drop_unstable(double &e, double &ep)
{
    if (fmax(fabs(e), fabs(ep)) > 0x1p400) e = ep = 0.0;
}

// Stable-direction switch for runs with n != 0.  At a ring the descending
// recursion of d^l_{m,n} grows (is stable) down to about m = n cos(theta); for
// the run with n cos(theta) > 0 the orders m < ms = ceil(|n cos(theta)|) are
// taken instead from the run -n (which is stable down to m = -ms) via
// d^l_{m,n} = (-1)^{m-n} d^l_{-m,-n}.  ring_good: this run is the one with
// n cos(theta) < 0 (ties: n < 0) at the ring; switch_order: ms in [0, |n|].
__device__ __forceinline__ bool ring_good(int n, double ct)
{
    return n != 0 && ((double)n * ct < 0.0 || (ct == 0.0 && n < 0));
}

__device__ __forceinline__ int switch_order(int n, double ct, double cs)
{
    const int an = n < 0 ? -n : n;
    if (an == 0) return 0;
    const int ms = (int)ceil(fabs((double)n * ct / cs) - 1e-9);   // |n cos(theta)|, cos = cot / csc
    return ms < 0 ? 0 : (ms > an ? an : ms);
}

}  // namespace s2mi
