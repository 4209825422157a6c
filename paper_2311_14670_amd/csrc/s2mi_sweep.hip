// s2mi_sweep.hip -- the FP64 Wigner sweeps: the descending-m recursion of
// d^l_{m,n}(theta) (Eqs. 25-27, running renormalisation of Sec. 3.4) fused with
// the l-contraction of Eq. 33 (inverse) and the theta-contraction of Eq. 30
// (forward) on the FP64 matrix instruction.
//
// Paper: Price & McEwen, arXiv 2311.14670.
//
// Recursion in rescaled form.  With alpha_k = sqrt((l+k)(l-k+1)) and
// d_m = e_m g_m (g from the plan tables), Eq. 25 becomes
//     e_{m-1} = kappa_m lambda_m e_m - e_{m+1},  lambda_m = (n - m cos th)/sin th,
// two FP64 operations per step.  Each (ring, l) carries (e_m, e_{m+1}, E) with
// d = e g 2^E; see s2mi_recur.h for the renormalisation.
//
// Contraction.  v_mfma_f64_4x4x4 multiplies four independent 4x4 blocks: lane
// i + 4 b + 16 k supplies A_b[i][k], lane j + 4 b + 16 k supplies B_b[k][j], and lane
// j + 4 b + 16 i receives D_b[i][j] (i, j, k, b in 0..3).  Both sweeps keep the
// recursion state in that A layout, so a step's values are the matrix operand as
// they stand: 16 rows (rings in the inverse, degrees in the forward) in lanes 0..15,
// the 4 terms of the sum (degrees resp. rings) in the four groups of 16 lanes, and
// the 4 columns {Re A, Im A, Re B, Im B} from the coefficient or spectra operand, one
// double per lane and the same in the four blocks.  A wave holds 32 such slots, 4 row
// groups x 8 terms.
//
// What bounds it.  The matrix instruction takes 16 cycles for 64 d values x 4
// columns, the recursion 2 FP64 operations (8 cycles); the two share the FP64
// pipeline, so a slot costs 24 cycles at best.  (Measured in a loop of nothing else, two
// waves per SIMD: 22.7 for the product and one of the two operations, 27 with both;
// the product and one operation as five vector operations 29.1: the product needs neither
// four accumulators nor dependent adds close together.)  The contraction's other operand
// and kappa are vector loads that the next order's step has in flight while this one
// computes (a lane's registers are reloaded as soon as they are used), where the vector
// form waited for scalar loads, and one wave holds 4 x 16 rows, so the sums that cross the
// waves of a workgroup are 1/32 of the d values.
//
// A third of the vector instructions were not FP64 at first: addresses, the sums over
// the waves, the renormalisation.  So the operands and kappa are buffer loads and the
// partial sums buffer stores at scalar offsets (the lane's part of an address is fixed
// for a piece), one half of the waves reduces an iteration's orders after the first of
// the next iteration and the other half after the third (the matrix unit of a SIMD is
// left to the other wave meanwhile), and only values beyond 2^-600 lose exponent.
//
// Measured on MI355X (one map, spin 0, MW L = 2048): inverse sweep 2.58 -> 1.65 ms,
// forward 2.70 -> 1.93 ms against the vector form with scalar record loads, 1.56 and 1.75
// ms with scalar offsets and the two halves apart, and 1.45 and 1.76 ms with consecutive
// pieces run as one; HEALPix nside 1024, L = 2048, real signal 2.68 -> 1.82 and 2.73 ->
// 1.83 ms; MW L = 4096 19.3 -> 10.5 and 19.0 -> 12.2 ms; L = 512, 16 maps in one launch
// instead of 16 in turn 2.95 -> 0.54 and 3.50 -> 0.50 ms.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "s2mi_internal.h"
#include "s2mi_kernels.h"
#include "s2mi_recur.h"

namespace s2mi {

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ double mfma4(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Sides of a run present in a call: 0 both, 1 the A side (orders +m of slice sliceA),
// 2 the B side (orders -m of slice sliceB).  half (real signals): the A side only.
__device__ __forceinline__ int run_side(const SweepRun &r, int half)
{
    return half ? 1 : (r.sliceA >= 0 && r.sliceB >= 0) ? 0 : (r.sliceA >= 0 ? 1 : 2);
}

// rows of an 8-degree chunk's records: orders -nx .. 8 q + 7, stored after those of
// the chunks below it
__device__ __forceinline__ size_t rec_row(int q, int m, int nx)
{
    return (size_t)q * nx + 4 * (size_t)q * (q + 1) + (size_t)(m + nx);
}

// doubles of a chunk's record row: kappa and four columns, or two for a one-sided run
// (mirror rings: those two and their copies signed (-1)^l)
constexpr int rec_doubles(bool one, bool pair) { return one && !pair ? 24 : 40; }

// ------------------------------------------------------------------ inverse pack
// Records of the inverse sweep, one row per (8-degree chunk q, order m <= 8 q + 7):
//   {kappa[k][h], coef[k][j][h]}, degree l = 8 q + 2 k + h (k < 4, h < 2),
//   kappa_{m+1}^l, coef columns j: wA_l g_m^l flmA[l][m] (re, im),
//   wB_l g_m^l (-1)^{m-n} flmB[l][-m] (re, im); a one-sided run holds its side's two
//   (PAIR: then these times (-1)^l).
// Zero where the run does not reach (l < max(m, |n|), l >= L).  The B column is used
// at m > 0 and, for n != 0, at m <= 0 by the continuation of the run below m = 0
// (orders m <= 0 then feed the B slice at -m >= 0 and the A slice at m < 0).
// A workgroup packs 32 orders of one chunk: coefficients are read with lanes along the
// orders (contiguous in flm) and written through LDS as whole rows.
template <bool ONE, bool PAIR>
__global__ __launch_bounds__(256) void k_pack_inv(InvArgs a, const double2 *__restrict__ flm, long long fstride,
                                                  const double *__restrict__ wl, const double *__restrict__ kap,
                                                  const double *__restrict__ gtab)
{
    constexpr int RS = rec_doubles(ONE, PAIR);
    constexpr int LS = RS + 1;
    __shared__ double sh[32 * LS];
    const int q = blockIdx.y, L = a.L, nx = a.nx;
    const int m0 = 32 * (int)blockIdx.x - nx;
    const int mtop = 8 * q + 7;
    if (m0 > mtop) return;
    const int map = blockIdx.z / a.nrun, ri = blockIdx.z % a.nrun;
    const SweepRun r = a.runs[ri];
    const int n = r.n, an = n < 0 ? -n : n, side = run_side(r, a.half);
    const int M = 2 * L - 1;
    const double2 *fm = flm + (size_t)map * fstride;
    {
        const int t = threadIdx.x, e = t >> 5, mi = t & 31;
        const int m = m0 + mi, l = 8 * q + e, k = e >> 1, h = e & 1;
        double kp = 0.0, c[4] = {0.0, 0.0, 0.0, 0.0};
        if (l < L && l >= m && l >= an && m < L) {
            const double g = gtab[(ptrdiff_t)m * L + l];
            if (l > m) kp = kap[(ptrdiff_t)m * L + l];
            if (side != 2) {
                const double2 v = fm[(size_t)r.sliceA * L * M + (size_t)l * M + (L - 1) + m];
                const double s = wl[(size_t)r.sliceA * L + l] * g;
                c[0] = s * v.x;
                c[1] = s * v.y;
            }
            if (side != 1 && (m > 0 || an > 0)) {
                const double2 v = fm[(size_t)r.sliceB * L * M + (size_t)l * M + (L - 1) - m];
                double s = wl[(size_t)r.sliceB * L + l] * g;
                if ((m - n) & 1) s = -s;
                c[2] = s * v.x;
                c[3] = s * v.y;
            }
        }
        double *o = sh + mi * LS;
        o[2 * k + h] = kp;
        if constexpr (ONE && PAIR) {
#pragma unroll
            for (int j = 0; j < 4; ++j) o[8 + 8 * k + 2 * j + h] = j >= 2 && h ? -c[j & 1] : c[j & 1];
        } else if constexpr (ONE) {
            o[8 + 4 * k + h] = side == 2 ? c[2] : c[0];
            o[8 + 4 * k + 2 + h] = side == 2 ? c[3] : c[1];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) o[8 + 8 * k + 2 * j + h] = c[j];
        }
    }
    __syncthreads();
    const int rows = min(32, mtop - m0 + 1);
    double *dst = a.C + (size_t)map * a.wsd + (size_t)ri * a.nC + rec_row(q, m0, nx) * RS;
    for (int i = threadIdx.x; i < rows * RS; i += 256) dst[i] = sh[(i / RS) * LS + i % RS];
}

// ------------------------------------------------------------------ states at the cuts
// State of the recursion after order c (e_c, e_{c+1}, E) at every cut of a sweep's
// work table: the value sequence of the sweeps (kappa lambda, then one fma,
// renormalising every RN orders by exact powers of two at the same orders), so a
// piece that starts from it holds exactly the state of the uninterrupted sweep.
// Degrees not started by order c and rings past nreg hold zeros.
// Inverse (FWD = false): block b holds degrees b D + i, state ck[cut][i][3][ring];
// lanes along the rings.  Forward: group b holds degrees b 64 + i or, for a mirror-ring
// sweep (par), 128 (b / 2) + 2 i + b % 2, state ck[cut][3][ring][i]; lanes along i.
// What bounds it: kappa.  All lanes of a wave are at the same order (a row of kappa is read
// at once; degrees below it wait), the rows up to the next renormalisation are loaded
// together, once every lane has started the steps have no conditions, and forward a wave
// takes several rings with a row.  (MI355X, one run of MW L = 2048, ms, inverse / forward:
// each lane at its own order, a row at a time 1.04 / 7.4; one order, rows together - / 3.05;
// no conditions 0.58 / 2.9; four rings, forward 1.0, with conditions 5.4.)
constexpr int CUT_RINGS = 4;
template <bool FWD>
__global__ __launch_bounds__(64) void k_cut_state(int L, int nreg, int rp, int D, int par,
                                                  const SweepRun *__restrict__ runs,
                                                  const double *__restrict__ cot, const double *__restrict__ csc,
                                                  const double *__restrict__ kap, const int *__restrict__ cfirst,
                                                  const int2 *__restrict__ cuts)
{
    const SweepRun run = runs[blockIdx.z];
    const int n = run.n;
    const double2 *init = run.init;
    double *ck = const_cast<double *>(FWD ? run.ckF : run.ckI);
    constexpr int NR = FWD ? CUT_RINGS : 1;              // rings r0 .. of a lane
    int r0, b, i, l;
    if constexpr (FWD) {
        i = threadIdx.x;
        b = blockIdx.x;
        r0 = NR * (int)blockIdx.y;
        l = par ? 128 * (b >> 1) + 2 * i + (b & 1) : 64 * b + i;
    } else {
        r0 = (int)(blockIdx.x * blockDim.x + threadIdx.x);
        l = blockIdx.y;
        b = l / D;
        i = l - b * D;
    }
    const int c0 = cfirst[b], c1 = cfirst[b + 1];
    const int an = n < 0 ? -n : n;
    const int low = FWD ? (par ? l - 2 * i : l - i) : l;     // first and last degree of the lanes
    const int top = min(FWD ? low + (par ? 126 : 63) : l, L - 1);
    double cur[NR], prev[NR], ct[NR], ncs[NR];              // e_m, e_{m+1}
    double2 start[NR];
    int E[NR], m = top + 1;
    const bool deg = l >= an && l < L;
#pragma unroll
    for (int k = 0; k < NR; ++k) {                           // (a ring or degree that is not there holds zeros)
        cur[k] = prev[k] = ct[k] = ncs[k] = 0.0;
        E[k] = 0;
        start[k] = make_double2(0.0, 0.0);
        if (deg && r0 + k < nreg) {
            ct[k] = cot[r0 + k];
            ncs[k] = (double)n * csc[r0 + k];
            start[k] = init[(size_t)(r0 + k) * L + l];
        }
    }
    const double *kl = kap + min(l, L - 1);
    auto step = [&](int k, int mm, double kq) {
        const double lam = fma(-(double)(mm + 1), ct[k], ncs[k]);
        const double p = kq * lam;
        const double nw = fma(p, cur[k], -prev[k]);
        prev[k] = cur[k];
        cur[k] = nw;
    };
    for (int q = c0; q < c1; ++q) {                          // cuts of the block, orders descending
        const int c = cuts[q].x;
        while (m > c) {                                      // down to the next renormalisation
            const int hi = m - 1, lo = max(c, hi & ~(RN - 1));
            double kq[RN];
#pragma unroll
            for (int j = 0; j < RN; ++j) kq[j] = kl[(ptrdiff_t)max(hi - j, lo) * L];
            if (hi - lo == RN - 1 && hi < low) {             // every lane has started
#pragma unroll
                for (int j = 0; j < RN; ++j)
#pragma unroll
                    for (int k = 0; k < NR; ++k) step(k, hi - j, kq[j]);
            } else {
#pragma unroll
                for (int j = 0; j < RN; ++j) {
                    const int mm = hi - j;
                    if (mm < lo || mm > l) continue;
#pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        if (mm == l) {
                            cur[k] = start[k].x;
                            E[k] = (int)start[k].y;
                        } else {
                            step(k, mm, kq[j]);
                        }
                    }
                }
            }
            if (lo < l && (lo & (RN - 1)) == 0)
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    renorm(cur[k], prev[k], E[k]);
                    if (FWD && an > DROP_AN && lo < an) drop_unstable(cur[k], prev[k]);
                }
            m = lo;
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            if (r0 + k >= rp) continue;
            const bool have = deg && r0 + k < nreg && c <= l;
            double *o;
            size_t st;
            if constexpr (FWD) {
                o = ck + ((size_t)cuts[q].y * 3 * rp + r0 + k) * 64 + i;
                st = (size_t)rp * 64;
            } else {
                o = ck + ((size_t)cuts[q].y * D + i) * 3 * rp + r0;
                st = rp;
            }
            o[0] = have ? cur[k] : 0.0;
            o[st] = have ? prev[k] : 0.0;
            o[2 * st] = have ? (double)E[k] : 0.0;
        }
    }
}

// ------------------------------------------------------------------ work of a workgroup
// A sweep's work is cut into pieces {block, top order, bottom order, cut}, a block
// being a set of degrees that a workgroup sweeps together from its top order down.
// The pieces of all blocks, in order, are dealt to `nslot` slots of equal length (a
// long block continues in the next slot, from the state stored at the cut), and a
// workgroup runs `merge` consecutive slots: one for a single map, more when several
// runs or maps share the launch and fill the device.  Every (block, order) sum is
// computed the same way in any of these splits.

// ------------------------------------------------------------------ inverse sweep
// Workgroup: 64 rings (4 groups of 16 lanes) x a block of up to 256 degrees; its 8
// waves take the block's 8-degree chunks in turn (wave w: chunks w, w + 8, ..), each
// chunk as two steps of four degrees of one parity, l = 8 q + 2 k + h in lanes 16 k ..
// 16 k + 15.  The orders run in iterations of four, m = mb .. mb - 3 with mb = 3 mod 4;
// the two state registers alternate roles by the parity of m (odd orders land in Y).
//
// A degree l starts at order m = l.  Its slot holds zero until then and its records at
// orders m >= l have kappa = 0, coefficients 0 for m > l, so a step leaves the slot's
// other register 0 and flips the sign of the one that receives the order: writing -+e0
// (minus for the iteration's first two orders, plus for the last two, whose register is
// flipped once before) ahead of the iteration gives e_l = e0 at order l.  All starts of an
// iteration are set there, and the steps have one form.
//
// Per order the waves' sums (64 rings x 4 columns each) go to LDS; after DORD orders one
// barrier, then all threads add them over the waves and write partA /
// partB[blk][ring][m][4] (whole 128-byte lines: four orders of a ring), while the next
// orders fill the other half of the buffers.  The scale exponents E, needed only by the
// renormalisation every RN orders, are held in LDS too, a quarter of them as 16-bit
// integers (they are multiples of 4 above -2^17: see renorm): 32 registers less.
//
// PAIR (spin 0, N/S-symmetric sampling): the northern rings (nsw of nreg) also give
// the mirror ring nreg-1-r, using d^l_{m,0}(pi - theta) = (-1)^{l+m} d^l_{m,0}(theta):
// with E and O the sums over the even and odd degrees (the two steps of a chunk),
// ring r gets E + O and its mirror (-1)^m (E - O).
// ONE: one side only (columns 2, 3 repeat columns 0, 1); with PAIR the repeated columns
// take (-1)^l times the coefficient, so columns 0, 1 are E + O and 2, 3 are E - O.
// NCH: chunks of a wave at most (4, or 1 for small L: see the launcher).
constexpr int RED_DOUBLES = 8 * SW_WAVES * 256;          // reduction buffers: 8 orders (PAIR: 4) x 8 waves
constexpr int EXP_SHORTS = SW_WAVES * 32 * 64;           // exponents of every slot and lane

struct InvLane {
    double ct[4], ncs[4];       // rings of the four groups
    int ks;                     // lane / 16: which of the chunk's degree pairs
    unsigned okap, ocoef;       // byte offsets of the lane's values in a record row
};

// (buffer loads: the row is a scalar offset, so a load needs no vector address arithmetic)
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ double2 buf_load2(__amdgpu_buffer_rsrc_t rs, unsigned lane_off, unsigned row_off)
{
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rs, lane_off, row_off, 0));
}

__device__ __forceinline__ double buf_load1(__amdgpu_buffer_rsrc_t rs, unsigned lane_off, unsigned row_off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, lane_off, row_off, 0));
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t rs, unsigned lane_off, unsigned row_off, double v)
{
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), rs, lane_off, row_off, 0);
}

template <int RS>
__device__ __forceinline__ void inv_load(__amdgpu_buffer_rsrc_t rs, unsigned Cq, int m, const InvLane &ln, double2 &kq,
                                         double2 &cq)
{
    const unsigned row = Cq + (unsigned)(m * (RS * 8));
    kq = buf_load2(rs, ln.okap, row);
    cq = buf_load2(rs, ln.ocoef, row);
}

// One order of the started chunks (bits of act): recursion, products, and the load of
// the next order's records.  (One form with a branch per chunk: variants by the number
// of started chunks made the compiler keep the state in scratch memory where they meet.
// The loads stand outside the branch, at a row that exists for chunks not started, so
// that the compiler can count the loads in flight: behind a branch it would wait for all
// of them at every chunk.)
template <int PAR, bool ONE, bool PAIR, int NCH>
__device__ __forceinline__ void inv_step(int m, uint32_t act, int nx, const int (&cb)[NCH], __amdgpu_buffer_rsrc_t rsrc,
                                         const unsigned (&Cq)[NCH], const InvLane &ln,
                                         double (&X)[NCH][2][4], double (&Y)[NCH][2][4], double2 (&kq)[NCH],
                                         double2 (&cq)[NCH], double *rb)
{
    constexpr int RS = rec_doubles(ONE, PAIR);
    constexpr bool EO = PAIR && !ONE;                    // even and odd degrees summed apart
    constexpr int NA = EO ? 8 : 4;
    const double mm = -(double)(m + 1);
    double lam[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)                          // lambda_{m+1}: produces order m (PAIR: n = 0)
        lam[g] = PAIR ? mm * ln.ct[g] : fma(mm, ln.ct[g], ln.ncs[g]);
    double acc[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = 0.0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if ((act >> c) & 1u) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double kp = h ? kq[c].y : kq[c].x;
            const double cf = h ? cq[c].y : cq[c].x;
            double p[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) p[g] = kp * lam[g];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                double &nw = PAR == 0 ? Y[c][h][g] : X[c][h][g];       // receives order m
                const double od = PAR == 0 ? X[c][h][g] : Y[c][h][g];  // holds order m + 1
                nw = fma(p[g], od, -nw);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                double &a = acc[(EO ? 4 * h : 0) + g];
                a = mfma4(PAR == 0 ? Y[c][h][g] : X[c][h][g], cf, a);
            }
        }
        }
        inv_load<RS>(rsrc, Cq[c], max(min(m - 1, cb[c] + 7), -nx), ln, kq[c], cq[c]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) rb[i * 64] = acc[i];
}

// The last order of piece e, taken on through the next pieces of the workgroup where they
// continue its block (their first state is then at hand); e: the last piece taken.
__device__ __forceinline__ int piece_end(const int4 *__restrict__ seg, int4 sg, int &e, int e1, int mend)
{
    int bot = sg.z;
    while (e + 1 < e1 && seg[e + 1].x == sg.x) bot = seg[++e].z;
    return bot == 0 ? mend : bot;
}

// One buffer descriptor for the main sums of both sides: from the lower of the two
// slices (the same one, one of them null, or two of an SO(3) run) to the end of the
// higher one, a side's slice as an offset of the lane.  base null: beyond the 4 GiB of a
// descriptor, stores by pointer.  The descriptor has to be the same in every lane (a
// store through one that differs becomes a loop over the lanes' values), so nothing of a
// lane enters here: the lane's offset is offA or offB.
struct OutSpan {
    double *base;
    unsigned offA, offB, bytes;
};
__device__ inline OutSpan out_span(double *A, double *B, size_t bytes)
{
    double *lo = !A ? B : !B || A <= B ? A : B;
    const ptrdiff_t da = A ? (A - lo) * 8 : 0, db = B ? (B - lo) * 8 : 0;
    const size_t all = (size_t)(da > db ? da : db) + bytes;
    return {all < (1ull << 32) ? lo : nullptr, (unsigned)da, (unsigned)db, (unsigned)all};
}

template <bool ONE, bool PAIR, int NCH>
__global__ __launch_bounds__(64 * SW_WAVES) void k_sweep_inv(InvArgs a, const double *__restrict__ cot,
                                                             const double *__restrict__ csc)
{
    constexpr bool EO = PAIR && !ONE;
    constexpr int NA = EO ? 8 : 4;                       // accumulators of a wave and order
    constexpr int DORD = EO ? 2 : 4;                     // orders per barrier
    constexpr int RS = rec_doubles(ONE, PAIR);
    constexpr int OB = SW_WAVES * NA * 64;               // an order's buffer
    __shared__ double red[RED_DOUBLES];
    __shared__ short expo[EXP_SHORTS];
    const int lane = threadIdx.x & 63, w = ufl(threadIdx.x >> 6);
    const int L = a.L, nx = a.nx;
    // workgroup -> (work slot, ring tile, map and run); slots fastest, so that with 8
    // of them the ring tiles that read the same records share an XCD's L2
    const int nt = (a.nslot + a.merge - 1) / a.merge;
    const int t = blockIdx.x % nt, rest = blockIdx.x / nt;
    const int ring0 = (rest % a.rt) * 64, item = rest / a.rt;
    const int map = item / a.nrun, ri = item % a.nrun;
    const SweepRun r = a.runs[ri];
    const int n = r.n, an = n < 0 ? -n : n, side = run_side(r, a.half);
    const int mend = an > 1 ? -(an - 1) : 0;             // continuation below m = 0
    double *PA = side != 2 ? a.P + (size_t)map * a.wsd + (size_t)r.sliceA * a.nP : nullptr;
    double *PB = side != 1 ? a.P + (size_t)map * a.wsd + (size_t)r.sliceB * a.nP : nullptr;
    InvLane ln;
    ln.ks = lane >> 4;
    ln.okap = 16 * ln.ks;
    ln.ocoef = RS == 24 ? 64 + 16 * (2 * ln.ks + (lane & 1)) : 64 + 16 * (4 * ln.ks + (lane & 3));
    auto ring_of = [&](int g) { return min(ring0 + 16 * g + (lane & 15), a.nsw - 1); };
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        ln.ct[g] = cot[ring_of(g)];
        ln.ncs[g] = (double)n * csc[ring_of(g)];
    }
    // reducer thread: output column, order of the iteration, rows row0 (and row0 + 32)
    constexpr int NC = ONE ? 2 : 4;
    const int tid = threadIdx.x;
    const int rc = tid & (NC - 1), rq = (tid / NC) & (DORD - 1), row0 = tid / (NC * DORD);
    constexpr int ROWS = 64 * SW_WAVES / (NC * DORD);    // rows covered at once: 32 or 64
    constexpr int NR = 64 / ROWS;
    const int comp = rc + (ONE && side == 2 ? 2 : 0);
    int msg[NR];                                         // switch order of the ring, ~ms where this run is
#pragma unroll                                           // the stable one
    for (int i = 0; i < NR; ++i) {
        const int rr = min(ring0 + row0 + ROWS * i, a.nsw - 1);
        const int ms = switch_order(n, cot[rr], csc[rr]);
        msg[i] = ring_good(n, cot[rr]) ? ~ms : ms;
    }
    // its place in an order's buffer (the wave and the second row are fixed offsets), and
    // its byte offset in a block's partial sums for order mb - DORD + 1
    const int r16 = row0 & 15;
    const int rpos = (row0 >> 4) * 64 + 16 * (r16 & 3) + 4 * (r16 >> 2) + rc;
    const OutSpan po = out_span(PA, PB, (size_t)a.nreg * L * 32);
    const unsigned soff = comp * 8 + (comp < 2 ? po.offA : po.offB);
    const unsigned ooff = ((unsigned)(ring0 + row0) * L + (DORD - 1 - rq)) * 32 + soff;
    const unsigned moff = ((unsigned)(a.nreg - 1 - ring0 - row0) * L + (DORD - 1 - rq)) * 32 + soff;   // mirror
    // Every thread is a reducer.  The branch around the sums stays: without it the compiler
    // mixes them into the steps, and the one-sided forms get slower (MI355X, us, with /
    // without: MW L = 2048 spin 2 2620 / 2862, real signal 1340 / 1495, GL L = 301 108 / 114).
    const bool reducer = row0 < 64;
    short *ex = expo + (size_t)w * 32 * 64 + lane;       // exponent of slot (c, h, g) at 64 (8 c + 4 h + g)
    double X[NCH][2][4], Y[NCH][2][4];
    double2 kq[NCH], cq[NCH];
    int cb[NCH];
    unsigned Cq[NCH];                                    // byte offset of a chunk's row of order 0
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        a.C + (size_t)map * a.wsd + (size_t)ri * a.nC, 0, (int)(a.nC * 8), 0x00027000);
    uint32_t fast = 0;
    int it = 0;
    // Adds the waves' sums of the orders m1 .. m1 - DORD + 1 (buffer half `hf`) and stores
    // them to block blk's partial sums.
    auto reduce = [&](int blk, int hf, int m1, int mhi, int bot) {
        if (!reducer) return;
        const double *rb0 = red + (size_t)(hf * DORD + rq) * OB + (rpos & ~63) + ((rpos + 4 * ((m1 & 2 ? 0 : 2) * EO + rq)) & 63);
        double s[NR], s2[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const double *rb = rb0 + i * ROWS / 16 * 64;
            s[i] = 0.0;
            s2[i] = 0.0;
            if constexpr (PAIR && ONE) {                    // columns 2, 3: two doubles on
#pragma unroll
                for (int ww = 0; ww < SW_WAVES; ++ww) {
                    s[i] += rb[ww * NA * 64];
                    s2[i] += rb[ww * NA * 64 + 2];
                }
                s2[i] = ((m1 - rq) & 1) ? -s2[i] : s2[i];
            } else if constexpr (PAIR) {
                double se = 0.0, so = 0.0;
#pragma unroll
                for (int ww = 0; ww < SW_WAVES; ++ww) {
                    se += rb[ww * NA * 64];
                    so += rb[(ww * NA + 4) * 64];
                }
                s[i] = se + so;                             // ring ring0 + row
                s2[i] = ((m1 - rq) & 1) ? so - se : se - so;   // its mirror
            } else {
#pragma unroll
                for (int ww = 0; ww < SW_WAVES; ++ww) s[i] += rb[ww * NA * 64];
            }
        }
        const size_t bo = (size_t)blk * a.nreg * L * 4;
        const int m3 = m1 - (DORD - 1);
        if (po.base && m1 <= mhi && m3 >= bot && m3 >= (an > 1 ? an : 1)) {
            // main orders: every ring's own sides, at scalar offsets (no vector addresses)
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(po.base + bo, 0, (int)po.bytes, 0x00027000);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                if (ring0 + row0 + ROWS * i >= a.nsw) continue;
                buf_store(rs, ooff, m3 * 32 + i * ROWS * L * 32, s[i]);
                if (PAIR && a.nreg - 1 != 2 * (ring0 + row0 + ROWS * i))
                    buf_store(rs, moff - i * ROWS * L * 32, m3 * 32, s2[i]);
            }
            return;
        }
        const int m = m1 - rq;
        if (m > mhi || m < bot) return;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            // Orders below the ring's switch order ms come from the run that is
            // stable there (n cos(theta) < 0): it writes its own sides at m >= 0
            // and, from its continuation to m > -ms, the A slice at order m < 0
            // (components 2,3 at |m|) and the B slice at order -m >= 0 (components
            // 0,1 at |m|).  The other run writes nothing below ms.
            const bool good = msg[i] < 0;
            const int ms = good ? ~msg[i] : msg[i];
            double *dst = nullptr;
            int mo = m, co = comp;
            const bool ext = good && m <= 0 && -m < ms;
            if (comp < 2) {
                if (m >= 0 && (good || m >= ms)) dst = PA;
                else if (m < 0 && ext) { dst = PA; mo = -m; co = comp + 2; }
            } else {
                if (m > 0 && (good || m >= ms)) dst = PB;
                else if (ext) { dst = PB; mo = -m; co = comp - 2; }
            }
            const int rr = ring0 + row0 + ROWS * i;
            if (dst && rr < a.nsw) {
                dst[bo + ((size_t)rr * L + mo) * 4 + co] = s[i];
                if (PAIR && a.nreg - 1 - rr != rr) dst[bo + ((size_t)(a.nreg - 1 - rr) * L + mo) * 4 + co] = s2[i];
            }
        }
    };
    const int e1 = a.first[min((t + 1) * a.merge, a.nslot)];
#pragma unroll 1
    for (int e = a.first[t * a.merge]; e < e1; ++e) {
        const int4 sg = a.seg[e];
        const int blk = sg.x, mhi = sg.y, bot = piece_end(a.seg, sg, e, e1, mend);
        {
            fast = 0;
            const int q0 = blk * a.cb, nq = min(a.cb, (L + 7) / 8 - q0);   // chunks of the block
            const int nv = nq > w ? (nq - w + 7) / 8 : 0;                    // and of this wave
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                // the wave's chunks ascend to the last c; absent ones come first and are never active
                const int j = c - (NCH - nv), q = q0 + w + 8 * j;
                const bool ok = j >= 0;
                cb[c] = ok ? 8 * q : -(1 << 20);
                Cq[c] = (unsigned)rec_row(ok ? q : 0, 0, nx) * (RS * 8);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        double cur = 0.0, prev = 0.0, E = 0.0;
                        if (sg.w >= 0 && ok && 8 * q + 2 * ln.ks + h < L) {   // state after order mhi + 1
                            const int i = 8 * (w + 8 * j) + 2 * ln.ks + h;
                            const double *st = r.ckI + ((size_t)sg.w * 8 * a.cb + i) * 3 * a.rp + ring_of(g);
                            cur = st[0];
                            prev = st[a.rp];
                            E = st[2 * a.rp];
                        }
                        X[c][h][g] = cur;                 // mhi is odd (3 mod 4) below the top: X holds
                        Y[c][h][g] = prev;                // order mhi + 1, Y receives mhi
                        ex[64 * (8 * c + 4 * h + g)] = (short)((int)E >> 2);
                    }
                inv_load<RS>(rsrc, Cq[c], max(min(mhi | 3, cb[c] + 7), -nx), ln, kq[c], cq[c]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll 1
        for (int mb = mhi | 3; mb >= bot; mb -= 4) {
            // starts: the degrees mb .. mb - 3 belong to one chunk of one wave, in the lane
            // groups k0, k0 + 1 (k0 = 2 where the chunk itself starts, at mb = 8 q + 7)
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if (cb[c] != (mb & ~7)) continue;
                if (mb & 4) inv_load<RS>(rsrc, Cq[c], mb, ln, kq[c], cq[c]);
                fast &= ~(1u << c);
                const int l0 = cb[c] + 2 * ln.ks;
                const double sgn = (ln.ks & 1) ? -1.0 : 1.0;
                if ((ln.ks >> 1) == ((mb >> 2) & 1)) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (l0 + h >= an && l0 + h < L) {
#pragma unroll
                            for (int g = 0; g < 4; ++g) {
                                const double2 v = r.init[(size_t)ring_of(g) * L + l0 + h];
                                (h ? Y : X)[c][h][g] = sgn * v.x;
                                ex[64 * (8 * c + 4 * h + g)] = (short)((int)v.y >> 2);
                            }
                        }
                }
            }
            // chunks below the orders of this iteration are left out
            const int m3 = mb - 3;
            uint32_t act = 0;
#pragma unroll
            for (int c = 0; c < NCH; ++c) act |= (m3 <= cb[c] + 7 ? 1u : 0u) << c;
            auto step = [&](auto Q) {                    // order mb - Q
                constexpr int q = decltype(Q)::value;
                double *wb = red + (size_t)(EO ? (it & 1) * 2 + (q & 1) : (it & 1) * 4 + q) * OB + w * NA * 64 +
                             ((lane + 4 * q) & 63);
                inv_step<q & 1, ONE, PAIR, NCH>(mb - q, act, nx, cb, rsrc, Cq, ln, X, Y, kq, cq, wb);
            };
            // The sums of the last iteration (EO: half iteration) are added in this one, by
            // half of the waves after its first order and by the others, which share their
            // SIMDs, after its third (EO: second): while one wave of a SIMD adds, the other
            // has products to issue.  After the next barrier that half is free again.
            step(std::integral_constant<int, 0>());
            if (w < SW_WAVES / 2 && mb + DORD <= (mhi | 3)) reduce(blk, (it & 1) ^ 1, mb + DORD, mhi, bot);
            step(std::integral_constant<int, 1>());
            if constexpr (EO) {
                if (w >= SW_WAVES / 2 && mb + DORD <= (mhi | 3)) reduce(blk, (it & 1) ^ 1, mb + DORD, mhi, bot);
                __syncthreads();
                ++it;
            }
            step(std::integral_constant<int, 2>());
            if (EO ? w < SW_WAVES / 2 : w >= SW_WAVES / 2 && mb + DORD <= (mhi | 3))
                reduce(blk, (it & 1) ^ 1, EO ? mb : mb + DORD, mhi, bot);
            step(std::integral_constant<int, 3>());
            if (EO && w >= SW_WAVES / 2) reduce(blk, (it & 1) ^ 1, mb, mhi, bot);
            // renormalisation every RN orders of the started chunks not yet realised
            if ((m3 & (RN - 1)) == 0) {
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    if (m3 > cb[c] + 7 || ((fast >> c) & 1u)) continue;
                    bool z = true;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            short *q = ex + 64 * (8 * c + 4 * h + g);
                            int E = 4 * (int)*q;
                            renorm(X[c][h][g], Y[c][h][g], E);
                            *q = (short)(E >> 2);
                            z = z && E == 0;
                        }
                    if (__all(z) && m3 <= cb[c]) fast |= 1u << c;
                }
            }
            __syncthreads();
            ++it;
        }
        // the last iteration's sums (the next piece writes the other half first)
        reduce(blk, (it & 1) ^ 1, ((bot + 4096) & ~3) - 4096 + DORD - 1, mhi, bot);
    }
}

// ------------------------------------------------------------------ forward sweep
// Workgroup: a group of 64 degrees (4 x 16 lanes) x a block of rings; wave w takes the
// 4 nk consecutive rings from w 4 nk (nk <= 8 steps of four rings, in lanes 16 k ..
// 16 k + 15; rings past the last swept one are inert: zero state, zero spectra).  At
// order m acc(l) = sum over rings of e * H[m][ring], reduced over the waves as in the
// inverse and written to QA / QB[blk][l][m] (without g_m^l: the finish multiplies by
// it).  Iterations, register roles, starts and exponents as in the inverse (a degree's
// sums above its start are not written, so its operand need not be zero there).
// PAIRF (run n = 0, N/S-symmetric sampling): the slots are the northern rings and
// a group holds degrees of one parity (l = 128 (G/2) + 2 i + G%2); with
// d^l_{m,0}(pi - theta) = (-1)^{l+m} d^l_{m,0}(theta) a ring contributes d (H(ring) +
// (-1)^{l+m} H(mirror)): order m reads the sums S or the differences D of the two
// rings' spectra by the parity of m + G.
// KS: steps of a wave at most (8, or 2 for few rings: see the launcher).

// The operand row of order m: lane's column of {A re, A im, B re, B im} at its first
// ring.  Orders below |n| read copies in which the rings where this run is unstable are
// zero (the other run covers them); the continuation (m <= 0) reads the A slice at
// order m < 0 (components 2,3) and the B slice at order -m >= 0 (components 0,1).
__device__ __forceinline__ const double *fwd_row(int m, int an, int hstride, int col, const double *HA, const double *HB,
                                                 const double *HxA, const double *HxB, int r0)
{
    const int am = m < 0 ? -m : m;
    const bool low = m < an;
    const double *pa = (low ? HxA : HA) + (m < 0 ? 2 : 0), *pb = (low ? HxB : HB) + (m > 0 ? 2 : 0);
    return (col < 2 ? pa : pb) + (col & 1) + ((size_t)am * hstride + r0) * 4;
}

// One order.  hrow, kapn: the next order's rows.
template <int PAR, int KS>
__device__ __forceinline__ void fwd_step(int m, int nk, const double (&ct)[KS], const double (&ncs)[KS],
                                         __amdgpu_buffer_rsrc_t krs, unsigned krow, const unsigned (&lc)[4],
                                         const double *__restrict__ hrow, double (&X)[KS][4], double (&Y)[KS][4],
                                         double (&kp)[4], double (&hq)[KS], double *rb)
{
    const double mm = -(double)(m + 1);
    double kn[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) kn[g] = buf_load1(krs, lc[g], krow);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        if (s < nk) {
        const double lam = fma(mm, ct[s], ncs[s]);       // lambda_{m+1}: produces order m
        double p[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) p[g] = kp[g] * lam;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            double &nw = PAR == 0 ? Y[s][g] : X[s][g];
            const double od = PAR == 0 ? X[s][g] : Y[s][g];
            nw = fma(p[g], od, -nw);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[g] = mfma4(PAR == 0 ? Y[s][g] : X[s][g], hq[s], acc[g]);
        }
        hq[s] = hrow[16 * s];                            // (unconditional: see inv_step; absent steps read
                                                         // on past the row)
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) kp[g] = kn[g];
#pragma unroll
    for (int g = 0; g < 4; ++g) rb[g * 64] = acc[g];
}

template <bool ONE, bool PAIRF, int KS>
__global__ __launch_bounds__(64 * SW_WAVES) void k_sweep_fwd(FwdArgs a, const double *__restrict__ cot,
                                                             const double *__restrict__ csc,
                                                             const double *__restrict__ kap)
{
    constexpr int DORD = 4;                              // orders per barrier
    constexpr int OB = SW_WAVES * 256;                   // an order's buffer
    __shared__ double red[RED_DOUBLES];
    __shared__ short expo[EXP_SHORTS];
    const int lane = threadIdx.x & 63, w = ufl(threadIdx.x >> 6);
    const int L = a.L, nk = a.nk;
    // workgroup -> (ring block, work slot, map and run); ring blocks fastest, so that
    // with 8 of them each XCD's L2 holds one ring block's spectra
    const int nt = (a.nslot + a.merge - 1) / a.merge;
    const int blk = blockIdx.x % a.rb, rest = blockIdx.x / a.rb;
    const int t = rest % nt, item = rest / nt;
    const int map = item / a.nrun, ri = item % a.nrun;
    const SweepRun r = a.runs[ri];
    const int n = r.n, an = n < 0 ? -n : n, side = run_side(r, a.half);
    const int mend = an > 1 ? -(an - 1) : 0;             // continuation below m = 0
    const size_t mo = (size_t)map * a.wsd;
    const double *HA, *HB, *HxA = nullptr, *HxB = nullptr;
    if constexpr (PAIRF) {
        HA = a.S + mo;
        HB = a.D + mo;
    } else {
        HA = a.F + mo + (size_t)(r.sliceA >= 0 ? r.sliceA : r.sliceB) * a.nF;
        HB = a.F + mo + (size_t)(r.sliceB >= 0 ? r.sliceB : r.sliceA) * a.nF;
        if (an > 0) {
            HxA = a.Hx + mo + (size_t)ri * 2 * a.nHx;
            HxB = HxA + a.nHx;
        }
    }
    double *QA = side != 2 ? a.Q + mo + (size_t)r.sliceA * a.nQ : nullptr;
    double *QB = side != 1 ? a.Q + mo + (size_t)r.sliceB * a.nQ : nullptr;
    double *QxA = an > 0 && r.sliceA >= 0 ? a.Qx + mo + (size_t)r.sliceA * a.nQx : nullptr;
    double *QxB = an > 0 && r.sliceB >= 0 ? a.Qx + mo + (size_t)r.sliceB * a.nQx : nullptr;
    const int rb0 = (blk * SW_WAVES + w) * 4 * nk;       // this wave's first ring
    const int col = ONE ? (lane & 1) + (side == 2 ? 2 : 0) : lane & 3;
    const int ks = lane >> 4, i16 = lane & 15;           // ring of a step, degree of a group
    const int r0 = rb0 + ks;                             // this lane's first ring (operand rows)
    double ct[KS], ncs[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int rr = r0 + 4 * s;
        const bool ok = s < nk && rr < a.nreg;
        ct[s] = ok ? cot[rr] : 0.0;
        ncs[s] = ok ? (double)n * csc[rr] : 0.0;
    }
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double *>(kap - (ptrdiff_t)a.nx * L), 0, (int)((unsigned)(L + a.nx) * L * 8), 0x00027000);
    constexpr int NC = ONE ? 2 : 4;
    const int tid = threadIdx.x;
    const int rc = tid & (NC - 1), rq = (tid / NC) & (DORD - 1), row0 = tid / (NC * DORD);
    constexpr int ROWS = 64 * SW_WAVES / (NC * DORD);    // 32 or 64
    constexpr int NR = 64 / ROWS;
    const int comp = rc + (ONE && side == 2 ? 2 : 0);
    constexpr int lsh = PAIRF ? 1 : 0;                   // log2 of a group's degree stride
    const int r16 = row0 & 15;
    const int rpos = (row0 >> 4) * 64 + ((16 * (r16 & 3) + 4 * (r16 >> 2) + rc + 4 * rq) & 63);
    const OutSpan qo = out_span(QA, QB, (size_t)L * L * 32);
    const unsigned ooff =
        ((unsigned)(row0 << lsh) * L + (DORD - 1 - rq)) * 32 + comp * 8 + (comp < 2 ? qo.offA : qo.offB);
    // Adds the waves' sums of the orders m1 .. m1 - 3 of group lmin (buffer half `hf`)
    // and stores them to the block's partial sums.
    auto reduce = [&](int lmin, int hf, int m1, int mhi, int bot) {
        const double *rb0 = red + (size_t)(hf * DORD + rq) * OB + rpos;
        double s[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            s[i] = 0.0;
#pragma unroll
            for (int ww = 0; ww < SW_WAVES; ++ww) s[i] += rb0[ww * 256 + i * ROWS / 16 * 64];
        }
        const size_t bo = (size_t)blk * L * L * 4;
        const int m3 = m1 - (DORD - 1);
        if (qo.base && m1 <= mhi && m1 <= lmin && m3 >= bot && m3 >= (an > 1 ? an : 1)) {
            // main orders below the group's degrees, at scalar offsets
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(qo.base + bo, 0, (int)qo.bytes, 0x00027000);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                if (lmin + ((row0 + ROWS * i) << lsh) >= L) continue;
                buf_store(rs, ooff, (unsigned)((lmin + ((ROWS * i) << lsh)) * L + m3) * 32, s[i]);
            }
            return;
        }
        const int m = m1 - rq;
        if (m > mhi || m < bot) return;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int lo = lmin + ((row0 + ROWS * i) << lsh);
            if (lo >= L || lo < m) continue;
            const int am = m < 0 ? -m : m;
            // continuation orders: the A slice at order m < 0 (the sign cancels the
            // one the finish applies there) and the B slice at order -m >= 0,
            // d^l_{-m,-n} = (-1)^{m-n} d^l_{m,n}
            const double sx = ((am + n) & 1) ? -s[i] : s[i];
            if (comp < 2) {
                if (m >= 0) {
                    if (QA) QA[bo + ((size_t)lo * L + m) * 4 + comp] = s[i];
                } else if (QxA) {
                    QxA[(((size_t)blk * L + lo) * a.nxp + am) * 4 + comp + 2] = sx;
                }
            } else if (m > 0) {
                if (QB) QB[bo + ((size_t)lo * L + m) * 4 + comp] = s[i];
            } else if (an > 0 && QxB) {
                QxB[(((size_t)blk * L + lo) * a.nxp + am) * 4 + comp - 2] = sx;
            }
        }
    };
    short *ex = expo + (size_t)w * 32 * 64 + lane;       // exponent of slot (s, g) at 64 (4 s + g)
    double X[KS][4], Y[KS][4];
    double hq[KS], kp[4];
    unsigned lc[4];                                      // byte offsets of the lane's degrees (clamped into the table)
    uint32_t fast = 0;
    int it = 0;
    // operand row of order m (pair: sums or differences by the parity of m + group)
    auto row_of = [&](int m, int G) -> const double * {
        if constexpr (PAIRF) {
            const double *h = ((m + G) & 1) ? HB : HA;
            return h + ((size_t)m * a.hstride + r0) * 4 + col;
        } else {
            return fwd_row(m, an, a.hstride, col, HA, HB, HxA, HxB, r0);
        }
    };
    const int e1 = a.first[min((t + 1) * a.merge, a.nslot)];
#pragma unroll 1
    for (int e = a.first[t * a.merge]; e < e1; ++e) {
        const int4 sg = a.seg[e];
        const int G = sg.x, mhi = sg.y, bot = piece_end(a.seg, sg, e, e1, mend);
        const int lmin = PAIRF ? 128 * (G >> 1) + (G & 1) : 64 * G;
        {
#pragma unroll
            for (int g = 0; g < 4; ++g) lc[g] = 8 * min(lmin + ((16 * g + i16) << lsh), L - 1);
            fast = 0;
            const double *h = row_of(min(mhi | 3, L - 1), G);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int rr = r0 + 4 * s;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    double cur = 0.0, prev = 0.0, E = 0.0;
                    if (sg.w >= 0 && s < nk && rr < a.nreg) {   // state after order mhi + 1
                        const double *q = r.ckF + ((size_t)sg.w * 3 * a.rp + rr) * 64 + 16 * g + i16;
                        cur = q[0];
                        prev = q[(size_t)a.rp * 64];
                        E = q[2 * (size_t)a.rp * 64];
                    }
                    X[s][g] = cur;                        // mhi is odd (3 mod 4) below the top
                    Y[s][g] = prev;
                    ex[64 * (4 * s + g)] = (short)((int)E >> 2);
                }
                hq[s] = h[16 * s];
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) kp[g] = buf_load1(krs, lc[g], (unsigned)((min(mhi | 3, L - 1) + a.nx) * L) * 8);
        }
#pragma unroll 1
        for (int mb = mhi | 3; mb >= bot; mb -= 4) {
            if (mb >= lmin) {                             // degrees mb .. mb - 3 of the group start
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if (lmin + ((16 * g) << lsh) > mb || lmin + ((16 * g + 15) << lsh) < mb - 3) continue;
                    const int l = lmin + ((16 * g + i16) << lsh), q = mb - l;
                    if (q >= 0 && q < 4 && l >= an && l < L) {
                        const double sgn = q < 2 ? -1.0 : 1.0;
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            const int rr = r0 + 4 * s;
                            if (s < nk && rr < a.nreg) {
                                const double2 v = r.init[(size_t)rr * L + l];
                                if (l & 1) Y[s][g] = sgn * v.x;
                                else X[s][g] = sgn * v.x;
                                ex[64 * (4 * s + g)] = (short)((int)v.y >> 2);
                            }
                        }
                    }
                }
            }
            double *wb = red + (size_t)(it & 1) * DORD * OB + w * 256;
            // rows of the next order: within the tables (the orders above the top and
            // below the last one give nothing that is written)
#define S2_FWD_STEP(Q)                                                                                                \
    {                                                                                                                 \
        const int mn = max(min(mb - (Q) - 1, L - 1), mend);                                                           \
        fwd_step<(Q) & 1, KS>(mb - (Q), nk, ct, ncs, krs, (unsigned)((mn + a.nx) * L) * 8, lc, row_of(mn, G), X, Y, \
                          kp, hq,                                                                                     \
                                wb + (Q) * OB + ((lane + 4 * (Q)) & 63));                                             \
    }
            // (the last iteration's sums are added in this one, in turn by the two waves of
            // a SIMD: see the inverse)
            S2_FWD_STEP(0)
            if (w < SW_WAVES / 2 && mb + 4 <= (mhi | 3)) reduce(lmin, (it & 1) ^ 1, mb + 4, mhi, bot);
            S2_FWD_STEP(1) S2_FWD_STEP(2)
            if (w >= SW_WAVES / 2 && mb + 4 <= (mhi | 3)) reduce(lmin, (it & 1) ^ 1, mb + 4, mhi, bot);
            S2_FWD_STEP(3)
#undef S2_FWD_STEP
            const int ml = mb - (DORD - 1);
            if ((ml & (RN - 1)) == 0) {                   // renormalisation of the steps not yet realised
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    if (s >= nk || ((fast >> s) & 1u)) continue;
                    bool z = true;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        short *q = ex + 64 * (4 * s + g);
                        int E = 4 * (int)*q;
                        renorm(X[s][g], Y[s][g], E);
                        *q = (short)(E >> 2);
                        z = z && E == 0;
                    }
                    if (__all(z) && ml <= lmin) fast |= 1u << s;
                }
                if constexpr (ONE && !PAIRF)              // (two-sided runs: |n| < 8)
                    if (an > DROP_AN && ml < an) {
#pragma unroll
                        for (int s = 0; s < KS; ++s)
#pragma unroll
                            for (int g = 0; g < 4; ++g) drop_unstable(X[s][g], Y[s][g]);
                    }
            }
            __syncthreads();
            ++it;
        }
        reduce(lmin, (it & 1) ^ 1, ((bot + 4096) & ~3) - 4096 + DORD - 1, mhi, bot);
    }
}

// ------------------------------------------------------------------ launchers
#define S2_LAUNCH_CHECK() do { hipError_t _e = hipGetLastError(); if (_e != hipSuccess) return _e; } while (0)

hipError_t launch_pack_inv(hipStream_t st, const InvArgs &a, int nmap, bool one, const double2 *flm, long long fstride,
                           const double *wl, const double *kap, const double *gtab)
{
    const int nq = (a.L + 7) / 8;
    const dim3 grid((unsigned)((8 * nq + a.nx + 31) / 32), (unsigned)nq, (unsigned)(nmap * a.nrun));
    if (one && a.nsw < a.nreg)
        hipLaunchKernelGGL((k_pack_inv<true, true>), grid, dim3(256), 0, st, a, flm, fstride, wl, kap, gtab);
    else if (one) hipLaunchKernelGGL((k_pack_inv<true, false>), grid, dim3(256), 0, st, a, flm, fstride, wl, kap, gtab);
    else hipLaunchKernelGGL((k_pack_inv<false, false>), grid, dim3(256), 0, st, a, flm, fstride, wl, kap, gtab);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_cut_state(hipStream_t st, bool fwd, int L, int nreg, int rp, int D, int nblk, int par, int nrun,
                            const SweepRun *runs, const double *cot, const double *csc, const double *kap,
                            const int *cfirst, const int2 *cuts)
{
    if (rp < nreg || D < 1 || (fwd && D != FWD_L)) return hipErrorInvalidValue;
    if (fwd)
        hipLaunchKernelGGL(k_cut_state<true>, dim3(nblk, (rp + CUT_RINGS - 1) / CUT_RINGS, nrun), dim3(64), 0, st, L,
                           nreg, rp, D, par, runs, cot, csc, kap, cfirst, cuts);
    else
        hipLaunchKernelGGL(k_cut_state<false>, dim3((rp + 63) / 64, nblk * D, nrun), dim3(64), 0, st, L, nreg, rp, D, par,
                           runs, cot, csc, kap, cfirst, cuts);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_sweep_inv(hipStream_t st, const InvArgs &a, int nmap, bool one, const double *cot, const double *csc)
{
    const bool pair = a.nsw < a.nreg;                    // mirror rings from the northern sweep
    if (a.nsw < 1 || a.nsw > a.nreg || (pair && 2 * a.nsw < a.nreg)) return hipErrorInvalidValue;
    if (a.cb < 1 || a.cb > INV_BLK / 8 || a.merge < 1 || a.nslot < 1 || a.rt * 64 < a.nsw) return hipErrorInvalidValue;
    const long long nt = (a.nslot + a.merge - 1) / a.merge, wg = nt * a.rt * nmap * a.nrun;
    if (wg > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wg), block(64 * SW_WAVES);
    auto go = [&](auto *k) { hipLaunchKernelGGL(k, grid, block, 0, st, a, cot, csc); };
    auto form = [&](auto nch) {
        constexpr int N = decltype(nch)::value;
        if (pair && one) go(k_sweep_inv<true, true, N>);
        else if (pair) go(k_sweep_inv<false, true, N>);
        else if (one) go(k_sweep_inv<true, false, N>);
        else go(k_sweep_inv<false, false, N>);
    };
    // Blocks of at most one chunk per wave (L <= 64) take the form for that: the same sums in
    // half the code, without scratch.  A short block runs that code little more than once, from
    // top to bottom (sweep, us, MI355X, form of four / one: MW L = 2 12.1 / 5.4, L = 5 15.0 /
    // 7.2, L = 16 14.2 / 7.6, L = 64 spin 2 14.4 / 12.0).
    if (a.cb <= SW_WAVES) form(std::integral_constant<int, 1>());
    else form(std::integral_constant<int, INV_BLK / (8 * SW_WAVES)>());
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_sweep_fwd(hipStream_t st, const FwdArgs &a, int nmap, bool one, const double *cot, const double *csc,
                            const double *kap)
{
    const bool pair = a.S != nullptr;
    if (a.nk < 1 || a.nk > FWD_KS || a.merge < 1 || a.nslot < 1 || a.rb * SW_WAVES * 4 * a.nk < a.nreg ||
        a.hstride < a.rb * SW_WAVES * 4 * a.nk || (pair && !a.D))
        return hipErrorInvalidValue;
    const long long nt = (a.nslot + a.merge - 1) / a.merge, wg = nt * a.rb * nmap * a.nrun;
    if (wg > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wg), block(64 * SW_WAVES);
    auto go = [&](auto *k) { hipLaunchKernelGGL(k, grid, block, 0, st, a, cot, csc, kap); };
    auto form = [&](auto ks) {
        constexpr int N = decltype(ks)::value;
        if (pair && one) go(k_sweep_fwd<true, true, N>);
        else if (pair) go(k_sweep_fwd<false, true, N>);
        else if (one) go(k_sweep_fwd<true, false, N>);
        else go(k_sweep_fwd<false, false, N>);
    };
    // At most 64 rings (per block: 32 a step over the waves) take the form for two steps, as in
    // the inverse (us, form of eight steps / two: MW L = 2 13.1 / 5.8, L = 5 16.3 / 7.8, L = 16
    // 14.9 / 6.4, L = 64 spin 2 19.8 / 11.5).
    if (a.nk <= FWD_KS_FEW) form(std::integral_constant<int, FWD_KS_FEW>());
    else form(std::integral_constant<int, FWD_KS>());
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

}  // namespace s2mi
