// s2mi_kernels.hip -- gfx950 kernels of the spin SHT / Wigner transforms outside
// the Wigner sweeps (s2mi_sweep.hip).
//
// Paper: Price & McEwen, arXiv 2311.14670.
//   start     d^l_{l,n} of Eq. 27 in log space, once per plan.
//   phi-DFT   Eqs. 31-32 per isolatitude ring; HEALPix rings repeat / fold the
//             Fourier line (Sec. 4.2, HEALPix).
//   MW theta  the exact MW theta integral (Sec. 4.2, MW): torus extension,
//             band-limited sin(theta) weight, evaluated on the L rings.
//   finish    block sums, weights and layout of the forward; glue of the adjoints.
//
// Transforms of several maps and slices share one launch: blockIdx.y is the item
// item0 + y = map * nslice + slice, and every buffer has a stride per map and one per
// slice (Items).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "s2mi_conv.h"
#include "s2mi_internal.h"
#include "s2mi_kernels.h"
#include "s2mi_recur.h"

namespace s2mi {

// ------------------------------------------------------------------ helpers
struct DD {
    double hi, lo;
};

__device__ __forceinline__ DD dd_from(const double *p) { return DD{p[0], p[1]}; }

__device__ __forceinline__ DD two_sum(double a, double b)
{
    const double s = a + b;
    const double bb = s - a;
    const double e = (a - (s - bb)) + (b - bb);
    return DD{s, e};
}

__device__ __forceinline__ DD dd_add(DD a, DD b)
{
    DD s = two_sum(a.hi, b.hi);
    s.lo += a.lo + b.lo;
    return two_sum(s.hi, s.lo);
}

__device__ __forceinline__ DD dd_mul_d(DD a, double k)   // k an exact small integer
{
    const double p = a.hi * k;
    const double e = fma(a.hi, k, -p);
    return two_sum(p, e + a.lo * k);
}

// d^l_{l,n}(theta) of Eq. 27 as a recursion slot state (e, E): log2|d| =
// lbin + (l-n) log2 sin(th/2) + (l+n) log2 cos(th/2) in double-double, sign (-1)^{l-n}.
// Realised (E = 0) directly when the value is not tiny; otherwise e = v 2^-RT with
// v in [1, 2) and the value is e 2^E, E < 0 (see renorm).
__device__ __forceinline__ void d_init(int l, int n, DD lbin, DD ls, DD lc, double &e, int &E)
{
    DD x = dd_add(lbin, dd_add(dd_mul_d(ls, (double)(l - n)), dd_mul_d(lc, (double)(l + n))));
    double fl = floor(x.hi);
    double f = (x.hi - fl) + x.lo;
    if (f < 0.0) { f += 1.0; fl -= 1.0; }
    if (f >= 1.0) { f -= 1.0; fl += 1.0; }
    double v = exp2(f);
    if ((l - n) & 1) v = -v;
    int ex = (int)fl;
    if (ex >= -RT) { v = ldexp(v, ex); ex = 0; }
    else {
        v = ldexp(v, -RT);
        ex += RT;
        v = ldexp(v, ex & 3);                            // multiples of 4 (see renorm)
        ex &= ~3;
    }
    e = v;
    E = ex;
}

// ------------------------------------------------------------------ start values
// init[r][l] = {mantissa, exponent} of d^l_{l,n}(theta_r) (Eq. 27) for every
// swept ring and l >= |n| (zeros below): computed once per plan so the sweeps
// only load them when a degree starts.
__global__ void k_init_table(int L, int nreg, int n, const double *__restrict__ lsin, const double *__restrict__ lcos,
                             const double *__restrict__ lbin, double2 *__restrict__ init)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)nreg * L) return;
    const int r = (int)(i / L), l = (int)(i % L);
    const int an = n < 0 ? -n : n;
    double e = 0.0;
    int E = 0;
    if (l >= an) d_init(l, n, dd_from(lbin + 2 * l), dd_from(lsin + 2 * r), dd_from(lcos + 2 * r), e, E);
    init[i] = make_double2(e, (double)E);
}

// Sums and differences of the spectra of a ring and its mirror for the paired
// forward sweep: S[m][i] = H[m][i] + H[m][nreg-1-i], D[m][i] = H[m][i] -
// H[m][nreg-1-i] over whole 32-byte records (both sides); a ring that is its own
// mirror (the equator) enters once: S = D = H.  Pairs past nsw are zero padding.
__global__ void k_pair_spectra(int L, int nreg, int nsw, int hstride, int pstride, const double *__restrict__ H,
                               double *__restrict__ S, double *__restrict__ D, long long wsd)
{
    H += blockIdx.y * wsd;
    S += blockIdx.y * wsd;
    D += blockIdx.y * wsd;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)L * pstride) return;
    const int m = (int)(i / pstride), r = (int)(i % pstride);
    double4 a = make_double4(0.0, 0.0, 0.0, 0.0), b = a;
    if (r < nsw) {
        a = *reinterpret_cast<const double4 *>(H + ((size_t)m * hstride + r) * 4);
        const int rm = nreg - 1 - r;
        if (rm != r) {
            const double4 c = *reinterpret_cast<const double4 *>(H + ((size_t)m * hstride + rm) * 4);
            b = make_double4(a.x - c.x, a.y - c.y, a.z - c.z, a.w - c.w);
            a = make_double4(a.x + c.x, a.y + c.y, a.z + c.z, a.w + c.w);
        } else {
            b = a;
        }
    }
    *reinterpret_cast<double4 *>(S + ((size_t)m * pstride + r) * 4) = a;
    *reinterpret_cast<double4 *>(D + ((size_t)m * pstride + r) * 4) = b;
}

// Copies of the two sides' ring spectra at orders mu < |n| for the forward sweep
// of run n, restricted to the rings whose values this run supplies (switch
// order ms of the ring): the own orders (A components 0,1 at mu >= 0, B
// components 2,3 at mu > 0) where the run is stable or mu >= ms, and the
// continuation orders (A components 2,3 = A slice at -mu, B components 0,1 = B
// slice at +mu) where the run is the stable one and mu < ms.  Other entries 0.  Clears
// the map's nz continuation sums Qx too (a launch of its own took 5 us).
__global__ void k_mask_low(int nrun, const SweepRun *__restrict__ runs, int nreg, int hstride,
                           const double *__restrict__ cot, const double *__restrict__ csc,
                           const double *__restrict__ F, double *__restrict__ Hx, long long wsd, long long nF,
                           long long nHx, double *__restrict__ Qx, long long nz)
{
    const int map = blockIdx.y / nrun, ri = blockIdx.y % nrun;
    for (long long j = ((long long)ri * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; j < nz;
         j += (long long)nrun * gridDim.x * blockDim.x)
        Qx[map * wsd + j] = 0.0;
    const SweepRun run = runs[ri];
    const int n = run.n, an_run = n < 0 ? -n : n;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)an_run * hstride) return;
    const double *FA = F + map * wsd + (size_t)(run.sliceA >= 0 ? run.sliceA : run.sliceB) * nF;
    const double *FB = F + map * wsd + (size_t)(run.sliceB >= 0 ? run.sliceB : run.sliceA) * nF;
    double *HxA = Hx + map * wsd + (size_t)ri * 2 * nHx;
    double *HxB = HxA + nHx;
    const int r = (int)(i % hstride), mu = (int)(i / hstride);
    bool own = false, ext = false;
    if (r < nreg) {
        const double ct = cot[r];
        const bool good = ring_good(n, ct);
        const int ms = switch_order(n, ct, csc[r]);
        own = good || mu >= ms;
        ext = good && mu < ms;
    }
    HxA[i * 4 + 0] = own ? FA[i * 4 + 0] : 0.0;
    HxA[i * 4 + 1] = own ? FA[i * 4 + 1] : 0.0;
    HxA[i * 4 + 2] = ext ? FA[i * 4 + 2] : 0.0;
    HxA[i * 4 + 3] = ext ? FA[i * 4 + 3] : 0.0;
    HxB[i * 4 + 0] = ext ? FB[i * 4 + 0] : 0.0;
    HxB[i * 4 + 1] = ext ? FB[i * 4 + 1] : 0.0;
    HxB[i * 4 + 2] = own ? FB[i * 4 + 2] : 0.0;
    HxB[i * 4 + 3] = own ? FB[i * 4 + 3] : 0.0;
}

// ------------------------------------------------------------------ phi-DFT: inverse
// One workgroup per (map, ring).  X_k = ftilde at orders m == k mod nphi
// (summed over the d-stage blocks), times the ring's half-pixel phase, then an
// inverse DFT of length nphi.  MW rings: nphi = 2L-1 and the order line maps
// one-to-one onto the bins.  The MW south pole (ring == nreg) has the closed
// form d^l_{m,-s}(pi) = (-1)^{l+m} delta_{m,s} (Eq. 29).
template <class E>
__global__ __launch_bounds__(E::MAXT, E::WPE) void k_phi_inv(
    int L, int nreg, int nblk, Items it, Strides sp, Strides sf, Strides sm, const double *__restrict__ part,
    const int *__restrict__ mtop, const double2 *__restrict__ flm, const double *__restrict__ wl, const int *__restrict__ ring_nphi, const long long *__restrict__ ring_start,
    const int *__restrict__ ring_shift, const int *__restrict__ ring_fft, const FftArgs *__restrict__ ffts,
    double2 *__restrict__ map, double2 *__restrict__ fscr)
{
    extern __shared__ double2 buf[];
    __shared__ double2 red[E::MAXT];
    const int r = blockIdx.x;
    const int T = blockDim.x, tid = threadIdx.x;
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    const int spin = it.spin[slice];
    part += map_i * sp.map + slice * sp.slice;
    flm += map_i * sf.map + slice * sf.slice;
    map += map_i * sm.map + slice * sm.slice;
    wl += (size_t)slice * L;
    const int nphi = ring_nphi[r];
    const FftArgs *f = ffts + ring_fft[r];
    const int shift = ring_shift[r];
    const int M = 2 * L - 1;
    if (r < nreg && nphi >= M) {
        // at most one order per bin (MW, and rings of nphi >= 2L - 1 samples: HEALPix
        // belt, DH, MWSS): a thread per |m| reads whole 32-byte records (order +|m| in
        // components 0,1, order -|m| in 2,3) and fills bins |m| and nphi - |m|; the bins
        // L .. nphi - L that no order reaches are zero
        for (int k = L + tid; k <= nphi - L; k += T) buf[E::slot(f, k)] = make_double2(0.0, 0.0);
        const double *pr = part + (size_t)r * L * 4;
        const size_t bstride = (size_t)nreg * L * 4;
        for (int am = tid; am < L; am += T) {
            double2 va = make_double2(0.0, 0.0), vb = make_double2(0.0, 0.0);
            for (int b = 0; b < nblk; ++b) {
                if (am > mtop[b]) continue;                  // that block's sweep never reached order am
                const double2 *pp = reinterpret_cast<const double2 *>(pr + b * bstride + am * 4);
                va = cadd(va, pp[0]);
                vb = cadd(vb, pp[1]);
            }
            if (shift) {
                double s, c;   // e^{+- i pi am / nphi}
                sincospi((double)(am % (2 * nphi)) / (double)nphi, &s, &c);
                va = cmul(va, make_double2(c, s));
                vb = cmul(vb, make_double2(c, -s));
            }
            buf[E::slot(f, am)] = va;
            if (am > 0) buf[E::slot(f, nphi - am)] = vb;
        }
    } else if (r < nreg) {
        // Bin k sums the orders m = k + q nphi within [-(L-1), L-1].  A short ring (nphi
        // below the thread count, HEALPix caps) spreads each bin's orders over `per`
        // threads, j-th taking every per-th order, and adds their sums in a fixed order.
        const double *pr = part + (size_t)r * L * 4;
        const size_t bstride = (size_t)nreg * L * 4;
        const int per = nphi >= T ? 1 : T / nphi;
        auto bin_sum = [&](int k, int j) {
            double2 acc = make_double2(0.0, 0.0);
            for (int m = k - ((k + L - 1) / nphi) * nphi + j * nphi; m <= L - 1; m += per * nphi) {
                const int am = m < 0 ? -m : m;
                const int off = am * 4 + (m < 0 ? 2 : 0);
                double2 v = make_double2(0.0, 0.0);
                for (int b = 0; b < nblk; ++b) {
                    if (am > mtop[b]) continue;              // that block's sweep never reached order m
                    const double *pp = pr + b * bstride + off;
                    v.x += pp[0];
                    v.y += pp[1];
                }
                if (shift) {
                    double s, c;   // e^{i pi m / nphi}
                    sincospi((double)(((long long)m % (2 * nphi) + 2 * nphi) % (2 * nphi)) / (double)nphi, &s, &c);
                    v = cmul(v, make_double2(c, s));
                }
                acc = cadd(acc, v);
            }
            return acc;
        };
        if (per == 1) {
            for (int k = tid; k < nphi; k += T) buf[E::slot(f, k)] = bin_sum(k, 0);
        } else {                                               // uniform over the workgroup
            if (tid < per * nphi) red[tid] = bin_sum(tid % nphi, tid / nphi);
            __syncthreads();
            for (int k = tid; k < nphi; k += T) {
                double2 acc = red[k];
                for (int j = 1; j < per; ++j) acc = cadd(acc, red[k + j * nphi]);
                buf[E::slot(f, k)] = acc;
            }
        }
    } else {
        // south pole (ring nreg): only m = s contributes, value sum_l (-1)^{l+s} w_l flm[l][s];
        // north pole (ring nreg + 1, MWSS): only m = -s, value sum_l w_l flm[l][-s]  (Eq. 29)
        const bool north = r > nreg;
        const int mp = north ? -spin : spin;
        double2 acc = make_double2(0.0, 0.0);
        const int as = spin < 0 ? -spin : spin;
        for (int l = as + tid; l < L; l += T) {
            double2 v = flm[(size_t)l * M + (L - 1) + mp];
            const double c = (!north && ((l + spin) & 1)) ? -wl[l] : wl[l];
            acc.x += c * v.x;
            acc.y += c * v.y;
        }
        red[tid] = acc;
        __syncthreads();
        int p2 = 1;
        while (p2 < T) p2 <<= 1;
        for (int s = p2 / 2; s > 0; s >>= 1) {   // T need not be a power of two
            if (tid < s && tid + s < T) red[tid] = cadd(red[tid], red[tid + s]);
            __syncthreads();
        }
        for (int k = tid; k < nphi; k += T) buf[E::slot(f, k)] = make_double2(0.0, 0.0);
        __syncthreads();
        if (tid == 0) buf[E::slot(f, ((mp % nphi) + nphi) % nphi)] = red[0];
    }
    __syncthreads();
    double2 *out = map + ring_start[r];
    E::template dft<+1, false>(
        buf, f, fscr ? fscr + (size_t)blockIdx.x * FFT_SCRATCH : nullptr, FftNone(),
        [&](int k, double2 v) { out[k] = v; });
}

// ------------------------------------------------------------------ phi-DFT: forward
// One workgroup per (map, ring): X = DFT_nphi(ring); ftilde_m = q e^{-i pi m s_r/nphi} X[m mod nphi]
// for |m| < L (the periodic repeat of Sec. 4.2 for short HEALPix rings), written
// to F[m][ring] = {ftilde_m, ftilde_-m}.
template <class E>
__global__ __launch_bounds__(E::MAXT, E::WPE) void k_phi_fwd(
    int L, int nring, int hstride, double q, Items it, Strides sm, Strides sF, const double2 *__restrict__ map, const int *__restrict__ ring_nphi,
    const long long *__restrict__ ring_start, const int *__restrict__ ring_shift,
    const int *__restrict__ ring_fft, const FftArgs *__restrict__ ffts, const double *__restrict__ ringq,
    double *__restrict__ F, double2 *__restrict__ fscr)
{
    extern __shared__ double2 buf[];
    // a row of F holds a ring's 32-byte record per order: four rings share a 128-byte line,
    // so they go to one XCD (workgroup i to XCD i mod 8), whose L2 joins their stores
    const int bi = blockIdx.x, b32 = bi & ~31;
    const int r = b32 + 32 <= (int)gridDim.x ? b32 + (bi & 7) * 4 + ((bi >> 3) & 3) : bi;
    const int T = blockDim.x, tid = threadIdx.x;
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    map += map_i * sm.map + slice * sm.slice;
    F += map_i * sF.map + slice * sF.slice;
    if (r >= nring) {                       // padding rings of the forward sweep: zeros
        for (int m = tid; m < L; m += T) {
            double *o = F + ((size_t)m * hstride + r) * 4;
            *reinterpret_cast<double2 *>(o) = make_double2(0.0, 0.0);
            *reinterpret_cast<double2 *>(o + 2) = make_double2(0.0, 0.0);
        }
        return;
    }
    const int nphi = ring_nphi[r];
    const FftArgs *f = ffts + ring_fft[r];
    const int shift = ring_shift[r];
    if (ringq) q = ringq[r];                     // per-ring quadrature weight (DH, GL)
    const double2 *in = map + ring_start[r];
    E::template dft<-1, false>(
        buf, f, fscr ? fscr + (size_t)blockIdx.x * FFT_SCRATCH : nullptr, [&](int k) { return in[k]; },
        FftNone());
    for (int m = tid; m < L; m += T) {
        double2 a = buf[E::slot(f, m % nphi)];
        double2 b = buf[E::slot(f, (nphi - (m % nphi)) % nphi)];
        if (shift) {
            double s, c;   // e^{-i pi m / nphi}
            sincospi((double)(m % (2 * nphi)) / (double)nphi, &s, &c);
            a = cmul(a, make_double2(c, -s));
            b = cmul(b, make_double2(c, s));
        }
        double *o = F + ((size_t)m * hstride + r) * 4;
        *reinterpret_cast<double2 *>(o) = make_double2(q * a.x, q * a.y);
        *reinterpret_cast<double2 *>(o + 2) = make_double2(q * b.x, q * b.y);
    }
}

// ------------------------------------------------------------------ phi-DFTs of real signals
// Spin 0.  The spectrum of a real ring is Hermitian (X[-k] = conj X[k], X[0]
// real), so two rings of equal length and phase offset share one complex DFT:
// ring r1 in the real and ring r2 in the imaginary part of z = x1 + i x2, with
// Z = X1 + i X2.  One workgroup per pair (r2 < 0: r1 alone); the pairs are
// built on the host.
//
// Inverse: the order-m spectrum of a swept ring is the sweep's side A (summed
// over its blocks) for m >= 0 and its conjugate for m < 0; the poles (MW south
// ring nreg, MWSS north ring nreg + 1) hold only order 0, sum_l (+-1)^l w_l
// Re flm[l][0] (Eq. 29).  Order 0 enters with its real part: the result is the
// real part of the complex transform of the Hermitian completion of the orders
// m >= 0.  Rings of 2L-1 samples without offset map orders one-to-one onto
// bins; other rings sum the orders of each bin (HEALPix repeat) with the
// half-pixel phase.
template <class E>
__global__ __launch_bounds__(E::MAXT, E::WPE) void k_phi_inv_real(
    int L, int nreg, int nblk, int item0, long long sp, long long sf, long long sm, const int *__restrict__ pairs, const double *__restrict__ part,
    const int *__restrict__ mtop, const double2 *__restrict__ flm, const double *__restrict__ wl,
    const int *__restrict__ ring_nphi, const long long *__restrict__ ring_start, const int *__restrict__ ring_shift,
    const int *__restrict__ ring_fft, const FftArgs *__restrict__ ffts, double *__restrict__ map,
    double2 *__restrict__ fscr)
{
    extern __shared__ double2 buf[];
    __shared__ double2 red[E::MAXT];
    const int map_i = item0 + blockIdx.y;
    part += map_i * sp;
    flm += map_i * sf;
    map += map_i * sm;
    const int r1 = pairs[2 * blockIdx.x], r2 = pairs[2 * blockIdx.x + 1];
    const int T = blockDim.x, tid = threadIdx.x;
    const int M = 2 * L - 1;
    const int nphi = ring_nphi[r1];
    const FftArgs *f = ffts + ring_fft[r1];
    const int shift = ring_shift[r1];
    double2 pole = make_double2(0.0, 0.0);                 // (south, north) order-0 values
    if (r1 >= nreg || r2 >= nreg) {                        // uniform over the workgroup
        double2 acc = make_double2(0.0, 0.0);
        for (int l = tid; l < L; l += T) {
            const double v = wl[l] * flm[(size_t)l * M + (L - 1)].x;
            acc.x += (l & 1) ? -v : v;
            acc.y += v;
        }
        red[tid] = acc;
        __syncthreads();
        int p2 = 1;
        while (p2 < T) p2 <<= 1;
        for (int h = p2 / 2; h > 0; h >>= 1) {           // T need not be a power of two
            if (tid < h && tid + h < T) red[tid] = cadd(red[tid], red[tid + h]);
            __syncthreads();
        }
        pole = red[0];
    }
    const size_t bstride = (size_t)nreg * L * 4;
    auto spec = [&](int r, int am) {                       // order +am of ring r (real part only at am = 0)
        double2 v = make_double2(0.0, 0.0);
        if (r < 0) return v;
        if (r < nreg) {
            const double *pr = part + ((size_t)r * L + am) * 4;
            for (int b = 0; b < nblk; ++b) {
                if (am > mtop[b]) continue;                  // that block's sweep never reached order am
                v = cadd(v, *reinterpret_cast<const double2 *>(pr + b * bstride));
            }
        } else if (am == 0) {
            v.x = r == nreg ? pole.x : pole.y;
        }
        if (am == 0) v.y = 0.0;
        return v;
    };
    if (nphi == M && !shift) {
        for (int am = tid; am < L; am += T) {
            const double2 x1 = spec(r1, am), x2 = spec(r2, am);
            buf[E::slot(f, am)] = make_double2(x1.x - x2.y, x1.y + x2.x);                      // X1 + i X2
            if (am > 0) buf[E::slot(f, M - am)] = make_double2(x1.x + x2.y, x2.x - x1.y);     // conj X1 + i conj X2
        }
    } else {
        // bins sum the orders = k mod nphi; short rings spread a bin over `per` threads
        // (fixed-order combination, as in the complex inverse)
        const int per = nphi >= T ? 1 : T / nphi;
        auto bin_sum = [&](int k, int j) {
            double2 z = make_double2(0.0, 0.0);
            for (int m = k - ((k + L - 1) / nphi) * nphi + j * nphi; m <= L - 1; m += per * nphi) {
                const int am = m < 0 ? -m : m;
                double2 x1 = spec(r1, am), x2 = spec(r2, am);
                if (m < 0) { x1 = cconj(x1); x2 = cconj(x2); }
                if (shift) {
                    double sn, cs;   // e^{i pi m / nphi}
                    sincospi((double)(((long long)m % (2 * nphi) + 2 * nphi) % (2 * nphi)) / (double)nphi, &sn, &cs);
                    x1 = cmul(x1, make_double2(cs, sn));
                    x2 = cmul(x2, make_double2(cs, sn));
                }
                z.x += x1.x - x2.y;
                z.y += x1.y + x2.x;
            }
            return z;
        };
        if (per == 1) {
            for (int k = tid; k < nphi; k += T) buf[E::slot(f, k)] = bin_sum(k, 0);
        } else {
            __syncthreads();                                   // red may still hold the pole sums
            if (tid < per * nphi) red[tid] = bin_sum(tid % nphi, tid / nphi);
            __syncthreads();
            for (int k = tid; k < nphi; k += T) {
                double2 z = red[k];
                for (int j = 1; j < per; ++j) z = cadd(z, red[k + j * nphi]);
                buf[E::slot(f, k)] = z;
            }
        }
    }
    __syncthreads();
    double *o1 = map + ring_start[r1];
    double *o2 = r2 >= 0 ? map + ring_start[r2] : nullptr;
    E::template dft<+1, false>(
        buf, f, fscr ? fscr + (size_t)blockIdx.x * FFT_SCRATCH : nullptr, FftNone(),
        [&](int k, double2 v) {
            o1[k] = v.x;
            if (o2) o2[k] = v.y;
        });
}

// Forward: Z = DFT(x1 + i x2), X1[k] = (Z[k] + conj Z[-k]) / 2, X2[k] = (Z[k] -
// conj Z[-k]) / 2i; order m >= 0 of a ring is q e^{-i pi m s/nphi} X[m mod nphi]
// (q per ring for DH / GL), written as F[m][ring] = {X_m, conj X_m} (the layout
// of the complex phi-DFT).  Workgroups past the pairs zero the sweep's padding
// rings nring .. hstride-1, two per workgroup.
template <class E>
__global__ __launch_bounds__(E::MAXT, E::WPE) void k_phi_fwd_real(
    int L, int nring, int hstride, int npair, double q, int item0, long long sm, long long sF,
    const int *__restrict__ pairs, const double *__restrict__ map,
    const int *__restrict__ ring_nphi, const long long *__restrict__ ring_start, const int *__restrict__ ring_shift,
    const int *__restrict__ ring_fft, const FftArgs *__restrict__ ffts, const double *__restrict__ ringq,
    double *__restrict__ F, double2 *__restrict__ fscr)
{
    extern __shared__ double2 buf[];
    const int T = blockDim.x, tid = threadIdx.x;
    map += (item0 + (int)blockIdx.y) * sm;
    F += (item0 + (int)blockIdx.y) * sF;
    if ((int)blockIdx.x >= npair) {
        const int r0 = nring + 2 * ((int)blockIdx.x - npair);
        for (int m = tid; m < L; m += T)
            for (int r = r0; r < r0 + 2 && r < hstride; ++r) {
                double2 *o = reinterpret_cast<double2 *>(F + ((size_t)m * hstride + r) * 4);
                o[0] = make_double2(0.0, 0.0);
                o[1] = make_double2(0.0, 0.0);
            }
        return;
    }
    const int r1 = pairs[2 * blockIdx.x], r2 = pairs[2 * blockIdx.x + 1];
    const int nphi = ring_nphi[r1];
    const FftArgs *f = ffts + ring_fft[r1];
    const int shift = ring_shift[r1];
    const double q1 = 0.5 * (ringq ? ringq[r1] : q);
    const double q2 = 0.5 * (ringq && r2 >= 0 ? ringq[r2] : q);
    const double *x1 = map + ring_start[r1];
    const double *x2 = r2 >= 0 ? map + ring_start[r2] : nullptr;
    E::template dft<-1, false>(
        buf, f, fscr ? fscr + (size_t)blockIdx.x * FFT_SCRATCH : nullptr,
        [&](int k) { return make_double2(x1[k], x2 ? x2[k] : 0.0); }, FftNone());
    for (int m = tid; m < L; m += T) {
        const int b = m % nphi;
        const double2 z = buf[E::slot(f, b)];
        const double2 zc = cconj(buf[E::slot(f, b == 0 ? 0 : nphi - b)]);
        double2 a = make_double2(q1 * (z.x + zc.x), q1 * (z.y + zc.y));     // q X1[m]
        double2 c = make_double2(q2 * (z.y - zc.y), -q2 * (z.x - zc.x));    // q X2[m]
        if (shift) {
            double sn, cs;   // e^{-i pi m / nphi}
            sincospi((double)(m % (2 * nphi)) / (double)nphi, &sn, &cs);
            a = cmul(a, make_double2(cs, -sn));
            c = cmul(c, make_double2(cs, -sn));
        }
        double2 *o1 = reinterpret_cast<double2 *>(F + ((size_t)m * hstride + r1) * 4);
        o1[0] = a;
        o1[1] = cconj(a);
        if (r2 >= 0) {
            double2 *o2 = reinterpret_cast<double2 *>(F + ((size_t)m * hstride + r2) * 4);
            o2[0] = c;
            o2[1] = cconj(c);
        }
    }
}

// ------------------------------------------------------------------ MW / MWSS theta filter
// For g = the torus extension of ftilde_{+-m} (g(2pi - th) = (-1)^{m+s} g(th)), on the
// N torus points
// (MW: N = 2L-1, theta_t = (2t+1) pi/N; MWSS: N = 2L, theta_t = 2 pi t/N)
//   h = P_{L-1}[g w'],   w' = P_{2L-2}[sin(theta) 1_[0,pi]],
// folded onto the rings: h~(theta_t) = (2pi/N) [h(theta_t) + (-1)^{m+s} h(mirror t)]
// (MW mirror N-1-t, MWSS N-t), unfolded at the poles, so that
// sum_t h~(theta_t) d(theta_t) = int_0^pi g d sin(theta) exactly.  On the doubled
// grid {theta_t} u {mu_t = theta_t + pi/N}:
//   h = (g w'_theta + S-[w'_mu S+ g]) / 2,
// S+-: band-limited half-sample shifts (DFT, phase e^{+-i k pi/N}/N, inverse DFT).
// MWSS: g is the torus interpolant without the Nyquist frequency L (it vanishes
// for band-limited samples); its value at theta_t is g_t - ghat_L (-1)^t.
// Torus point t <-> ring: MW t < L: ring t (t = L-1: south pole), MWSS t = 0:
// north pole (ring L), 0 < t < L: ring t-1, t = L: south pole (ring L-1).  In
// place: F[m][ring] -> H[m][ring] for the swept rings; the pole values go to
// hpole[(L-1) +- m] (south) and hpoleN (north, MWSS).
//
// Two orders per workgroup.  Of the weight only the even part |sin| / 2 of
// sin 1_[0,pi] = (|sin| + sin) / 2 reaches the fold of an extension (which has the fold's
// own parity), and with it the filter commutes with the mirror map; consecutive orders
// have extensions of opposite parity.  So one pass over the sum z of the extensions of
// orders 2j and 2j + 1 gives both, h~_m = sc (h(t) + (-1)^{m+s} h(mirror t)) keeping each
// order's own part.  (Half the transforms of one order at a time: MW L = 2048
// 0.50 -> 0.28 ms, L = 4096 5.2 -> 2.8 ms, L = 64 0.036 -> 0.022 ms; with the transforms
// of s2mi_fft.h and s2mi_conv.h as they are now 0.22, 1.5 and 0.011 ms;
// both orders come from, or go into, the same ring DFTs, so their rounding is relative to
// one another anyway.)  The one thing an extension of odd parity holds beyond that is its
// sample at a fixed point of the mirror (a pole): it is even, and the odd part sin / 2 of
// the weight carries it to the rings: P_{L-1}[sin / 2 times the interpolant of a unit
// sample] = (-1)^L sin((L-1) theta) / (2N) (without (-1)^L for the north pole), since all
// other frequencies cancel.  So an odd order's pole sample is left out of z and added as
// vs[t] g_pole, and the adjoint (adj) gives its pole the sum of vs[t] g(t); the values at
// odd poles that nothing reads (the finish uses |m| = |s|, even) are 0.  The sides +m and
// -m are workgroups of their own, on one XCD (their values interleave in 32-byte
// records).  half (real signals):
// only the side of order +m is filtered, the filter being real and the side
// of order -m the conjugate.
// adj (MWSS): the Hermitian adjoint of the filter.  With the Nyquist projector
// P (real, symmetric) and (S+)^H = S-, the filter is sc E^T [(W P + S- W' S+) / 2] E,
// whose adjoint differs only in the first term: P W instead of W P, i.e. the
// Nyquist component is removed from g w'_theta rather than from g.  (MW has no
// Nyquist bin: its filter is Hermitian and adj changes nothing.)
__device__ __forceinline__ int torus_ring(int t, int L, int N, int ss, bool *mirrored)
{
    *mirrored = ss ? t > L : t >= L;
    const int u = *mirrored ? (ss ? N - t : N - 1 - t) : t;     // sample on [0, pi]
    if (!ss) return u;
    return u == 0 ? L : u - 1;
}

// Sum of v over the lanes of a wave, in every lane.  (A workgroup of a small convolution
// engine is 16 or 32 threads, fewer than a wave; the others are multiples of 64.)
template <class E>
__device__ __forceinline__ double2 wave_sum(double2 v)
{
    for (int o = (E::MAXT < 64 ? E::MAXT : 64) / 2; o > 0; o >>= 1) {
        v.x += __shfl_xor(v.x, o, 64);
        v.y += __shfl_xor(v.y, o, 64);
    }
    return v;
}

template <class E, bool ss>
__global__ __launch_bounds__(E::MAXT, E::WPE) void k_mw_filter(int L, int hstride, Items it, Strides sF, Strides sh,
                                                    const FftArgs *__restrict__ fN, const double *__restrict__ wq,
                                                    const double *__restrict__ ph, double *__restrict__ F,
                                                    double2 *__restrict__ hpole, double2 *__restrict__ hpoleN,
                                                    double2 *__restrict__ fscr, int half, int adj)
{
    extern __shared__ double2 buf[];
    __shared__ double2 nyq;
    __shared__ double2 wpart[16];                          // per-wave partial sums (<= 1024 threads)
    // workgroup -> (pair of orders, side): both sides of a pair at distance 8
    const int bx = blockIdx.x;
    const int side = half ? 0 : (bx >> 3) & 1;
    const int pair = half ? bx : ((bx >> 4) << 3) + (bx & 7);
    const int m0 = 2 * pair, m1 = m0 + 1;
    if (m0 >= L) return;
    const bool has0 = side == 0 || m0 > 0, has1 = m1 < L;    // (side -m exists for m > 0)
    if (!has0 && !has1) return;
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    const int spin = it.spin[slice];
    F += map_i * sF.map + slice * sF.slice;
    hpole += map_i * sh.map + slice * sh.slice;
    if (hpoleN) hpoleN += map_i * sh.map + slice * sh.slice;
    const int N = ss ? 2 * L : 2 * L - 1;
    const int T = blockDim.x, tid = threadIdx.x;
    const double par = ((m0 + spin) & 1) ? -1.0 : 1.0;       // parity of m0; m1 has the other
    const double2 *phc = reinterpret_cast<const double2 *>(ph);
    double2 *scr = fscr ? fscr + (size_t)blockIdx.x * FFT_SCRATCH : nullptr;
    const double *F0 = F + (size_t)m0 * hstride * 4 + 2 * side;
    const double *F1 = F + (size_t)m1 * hstride * 4 + 2 * side;
    // z(t): the two orders' extensions; their values at ring r
    auto rings = [&](int r, bool pole, double2 &a, double2 &b) {
        a = b = make_double2(0.0, 0.0);
        if (has0 && !(pole && par < 0.0)) a = *reinterpret_cast<const double2 *>(F0 + (size_t)r * 4);
        if (has1 && !(pole && par > 0.0)) b = *reinterpret_cast<const double2 *>(F1 + (size_t)r * 4);
    };
    auto sample = [&](int t) {
        bool mir;
        const int r = torus_ring(t, L, N, ss, &mir);
        double2 a, b;
        rings(r, ss ? (t == 0 || t == L) : t == L - 1, a, b);
        const double s = mir ? par : 1.0, q = mir ? -par : 1.0;
        return make_double2(fma(s, a.x, q * b.x), fma(s, a.y, q * b.y));
    };
    // the odd-parity order: its pole samples (south, plus the north one signed for MWSS)
    // reach the rings through vs; adj: the rings reach its poles (sums of vs g)
    const double *vs = wq + 2 * (size_t)N;
    const bool hasO = par < 0.0 ? has0 : has1;
    const double *FO = par < 0.0 ? F0 : F1;
    const double sgN = (L & 1) ? -1.0 : 1.0;                 // vs of the north pole: (-1)^L vs
    double2 gpo = make_double2(0.0, 0.0);
    if (hasO) {
        gpo = *reinterpret_cast<const double2 *>(FO + (size_t)(L - 1) * 4);
        if (ss) {
            const double2 gn = *reinterpret_cast<const double2 *>(FO + (size_t)L * 4);
            gpo = make_double2(fma(sgN, gn.x, gpo.x), fma(sgN, gn.y, gpo.y));
        }
    }
    constexpr bool conv = E::CONV && !ss;                  // see below
    {
        // torus samples
        double2 acc = make_double2(0.0, 0.0);                // adj: sum_t (-1)^t w'_theta z
        for (int t = tid; ((E::CONV && ss) || (ss && adj)) && t < N; t += T) {
            const double2 g = sample(t);
            if (E::CONV) buf[t] = g;
            if (ss && adj) {
                const double sw = (t & 1) ? -wq[t] : wq[t];
                acc.x = fma(sw, g.x, acc.x);
                acc.y = fma(sw, g.y, acc.y);
            }
        }
        if (ss && adj) {                                    // uniform over the workgroup
            acc = wave_sum<E>(acc);
            if ((tid & 63) == 0) wpart[tid >> 6] = acc;
            __syncthreads();
            if (tid == 0) {
                double2 tot = make_double2(0.0, 0.0);
                for (int w = 0; w < (T + 63) / 64; ++w) tot = cadd(tot, wpart[w]);
                nyq = make_double2(tot.x / N, tot.y / N);   // Nyquist component of z w'_theta
            }
        }
        double2 po = make_double2(0.0, 0.0);                // adj: the odd order's pole value
        if (adj && hasO) {                                  // uniform over the workgroup
            for (int r = tid; r < L - 1; r += T) {
                const double2 g = *reinterpret_cast<const double2 *>(FO + (size_t)r * 4);
                const double v = vs[ss ? r + 1 : r];
                po.x = fma(v, g.x, po.x);
                po.y = fma(v, g.y, po.y);
            }
            po = wave_sum<E>(po);
            __syncthreads();                                // wpart is free again
            if ((tid & 63) == 0) wpart[tid >> 6] = po;
            __syncthreads();
            po = make_double2(0.0, 0.0);
            for (int w = 0; w < (T + 63) / 64; ++w) po = cadd(po, wpart[w]);
        }
        // the midpoint samples S g times the weights w'', moved back: S^{-1} (w'' S g)
        if constexpr (conv) {
            // MW, N not 13-smooth: each shift is a circular convolution of length N with a fixed
            // kernel (fN + 1 and fN + 2: the two shifts' FftArgs), and the whole filter
            // stays in registers.
            double2 v[E::V];
            int t0 = E::first_point();
#pragma unroll
            for (int i = 0; i < E::V; ++i) {
                const int t = t0 + E::T * i;
                v[i] = t < N ? sample(t) : make_double2(0.0, 0.0);
                E::few_loads(i);
            }
#pragma unroll 1
            for (int pass = 0; pass < 2; ++pass) {
                E::convolve(v, reinterpret_cast<double *>(buf), fN + 1 + pass);
                if (pass == 0) {
                    t0 = E::first_point();
#pragma unroll
                    for (int i = 0; i < E::V; ++i) {
                        const int t = t0 + E::T * i;
                        const double wv = t < N ? wq[N + t] : 0.0;
                        v[i] = make_double2(v[i].x * wv, v[i].y * wv);
                        E::few_loads(i);
                    }
                }
            }
            __syncthreads();
            t0 = E::first_point();
#pragma unroll
            for (int i = 0; i < E::V; ++i)
                if (t0 + E::T * i < N) buf[t0 + E::T * i] = v[i];
        } else {
            // forward, shift, inverse: midpoints; weights; forward, shift back, inverse
            auto shift = [&](int pass, double2 v, double2 w) { return pass ? cmulc(v, w) : cmul(v, w); };
            auto weigh = [&](int t, double2 v) { return make_double2(v.x * wq[N + t], v.y * wq[N + t]); };
            __syncthreads();
            if constexpr (E::CONV) {
                // MWSS, 2L not 13-smooth: four DFTs of the samples in LDS
#pragma unroll 1
                for (int pass = 0; pass < 2; ++pass) {
                    E::template dft<-1, true>(buf, fN, scr, [&](int k) { return buf[k]; }, FftNone());
                    for (int k = tid; k < N; k += T) {
                        if (ss && !adj && pass == 0 && k == L) nyq = make_double2(buf[k].x / N, buf[k].y / N);   // ghat_L
                        buf[k] = shift(pass, buf[k], phc[k]);
                    }
                    __syncthreads();
                    E::template dft<+1, true>(
                        buf, fN, scr, FftNone(),
                        [&](int t, double2 v) { buf[t] = pass ? v : weigh(t, v); });
                }
            } else {
                // one pass over LDS per stage; the shifts (phc in the order of the positions)
                // between the two innermost stages, the weights between the last inverse and
                // the first forward stage
                const int nst = fN->nst, last = nst - 1;
                const int pL = ss ? fft_pos(fN, L) : -1;
                auto get = [&](int i) { return buf[fft_place(fN, i)]; };
                auto put = [&](int i, double2 v) { buf[fft_place(fN, i)] = v; };
                if (last) {
                    fft_stage<FFT_FWD>(fN, 0, sample, FftNone(), put);
                } else {                                         // one stage alone: from LDS
                    for (int t = tid; t < N; t += T) put(t, sample(t));
                    __syncthreads();
                }
#pragma unroll 1
                for (int pass = 0; pass < 2; ++pass) {
                    fft_forward(buf, fN, 1, last);
                    fft_inner(
                        fN, last, get,
                        [&](int p, double2 v) {
                            if (ss && !adj && pass == 0 && p == pL) nyq = make_double2(v.x / N, v.y / N);   // ghat_L
                            return shift(pass, v, phc[p]);
                        },
                        put);
                    fft_inverse(buf, fN, 1, last);
                    if (pass) break;
                    if (last) {
                        fft_turn(fN, get, weigh, put);
                    } else {                                     // one stage alone
                        for (int t = tid; t < N; t += T) put(t, weigh(t, get(t)));
                        __syncthreads();
                    }
                }
                if (last) fft_stage<FFT_INV>(fN, 0, get, FftNone(), put);
            }
        }
        __syncthreads();
        const double sc = 2.0 * M_PI / (double)N;
        // + z w'_theta, folded onto the rings: z at a ring and at its mirror are the sum and
        // the difference of the same two values
        auto fold = [&](int t, double2 za, double2 zb) {
            const bool pole = ss ? (t == 0 || t == L) : t == L - 1;
            const int mt = pole ? t : ss ? N - t : N - 1 - t;
            auto value = [&](int u, double2 g) {
                const double wv = wq[u], sg = (u & 1) ? -1.0 : 1.0;
                const double2 v = buf[E::point(fN, u)];
                if (ss && !adj) {                                // P z, then times w'
                    g.x -= sg * nyq.x;
                    g.y -= sg * nyq.y;
                }
                double2 gw = make_double2(g.x * wv, g.y * wv);
                if (ss && adj) {                                 // P (z w')
                    gw.x -= sg * nyq.x;
                    gw.y -= sg * nyq.y;
                }
                return make_double2(0.5 * (gw.x + v.x), 0.5 * (gw.y + v.y));
            };
            const double2 h = value(t, cadd(za, zb));
            if (!pole) {
                const double2 d = csub(za, zb);
                const double2 hr = value(mt, make_double2(par * d.x, par * d.y));
                const size_t o = (size_t)(ss ? t - 1 : t) * 4;
                const double v = vs[t];
                const double v0 = par < 0.0 ? v : 0.0, v1 = par < 0.0 ? 0.0 : v;
                if (has0)
                    *reinterpret_cast<double2 *>(const_cast<double *>(F0) + o) =
                        make_double2(fma(v0, gpo.x, sc * fma(par, hr.x, h.x)), fma(v0, gpo.y, sc * fma(par, hr.y, h.y)));
                if (has1)
                    *reinterpret_cast<double2 *>(const_cast<double *>(F1) + o) =
                        make_double2(fma(v1, gpo.x, sc * fma(-par, hr.x, h.x)), fma(v1, gpo.y, sc * fma(-par, hr.y, h.y)));
            } else {
                double2 *hp = ss && t == 0 ? hpoleN : hpole;
                const double so = ss && t == 0 ? sgN : 1.0;
                const double2 v = make_double2(sc * h.x, sc * h.y), z = make_double2(so * po.x, so * po.y);
                if (has0) hp[side == 0 ? (L - 1) + m0 : (L - 1) - m0] = par > 0.0 ? v : z;
                if (has1) hp[side == 0 ? (L - 1) + m1 : (L - 1) - m1] = par < 0.0 ? v : z;
            }
        };
        for (int t = tid; t < (ss ? L + 1 : L); t += T) {
            double2 za, zb;
            rings(!ss ? t : t == 0 ? L : t - 1, ss ? (t == 0 || t == L) : t == L - 1, za, zb);
            fold(t, za, zb);
        }
    }
}

// ------------------------------------------------------------------ adjoint of the forward (MW)
// The MW forward is F = Finish Dfwd Theta PhiFwd with the theta filter Theta =
// sc E^H A E (torus extension E, Hermitian A, fold sc E^H): Theta is
// Hermitian, so F^H = PhiFwd^H Theta Dfwd^H Finish^H, where Dfwd^H Finish^H
// is the inverse sweep with the SHT weights on the regular rings plus the
// closed-form south pole (Eq. 29).  gather: sum the sweep's blocks (and the
// pole) into the filter's [m][ring] layout; scatter: filtered rings and pole
// -> [ring][m] partials of a single block, scaled by the phi weight q.
// MWSS (ss): the rows are the L-1 regular rings, the south pole (row L-1) and the
// north pole (row L, the forward's w_l h~_{-s}(0) at order -s), and the adjoint
// filter runs in between.
__global__ void k_fadj_gather(int L, int ss, int nblk, Items it, Strides sp, Strides sf, Strides sF, const double *__restrict__ part,
                              const int *__restrict__ mtop, const double2 *__restrict__ flm,
                              const double *__restrict__ wl, int hstride, double *__restrict__ F)
{
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    const int spin = it.spin[slice];
    part += map_i * sp.map + slice * sp.slice;
    flm += map_i * sf.map + slice * sf.slice;
    F += map_i * sF.map + slice * sF.slice;
    wl += (size_t)slice * L;
    const int nrow = L + ss;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)L * nrow) return;
    const int m = (int)(i / nrow), t = (int)(i % nrow);
    const int nreg = L - 1, M = 2 * L - 1;
    const size_t bstride = (size_t)nreg * L * 4;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (t < nreg) {
        for (int b = 0; b < nblk; ++b) {
            if (m > mtop[b]) continue;                  // that block's sweep never reached order m
            const double *pp = part + b * bstride + ((size_t)t * L + m) * 4;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] += pp[c];
        }
    } else {
        // south pole (t == nreg): only the signed order s is nonzero, sum_l (-1)^{l+s} w_l G[l][s];
        // north pole (t == nreg + 1): only the order -s, sum_l w_l G[l][-s]
        const bool north = t > nreg;
        const int mp = north ? -spin : spin;
        const int as = spin < 0 ? -spin : spin;
        if (m == as) {
            double2 acc = make_double2(0.0, 0.0);
            for (int l = as; l < L; ++l) {
                const double2 g = flm[(size_t)l * M + (L - 1) + mp];
                const double c = (!north && ((l + spin) & 1)) ? -wl[l] : wl[l];
                acc.x += c * g.x;
                acc.y += c * g.y;
            }
            const int off = (mp < 0) ? 2 : 0;
            v[off] = acc.x;
            v[off + 1] = acc.y;
        }
    }
    if (m == 0) { v[2] = 0.0; v[3] = 0.0; }
    double *dst = F + ((size_t)m * hstride + t) * 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) dst[c] = v[c];
}

__global__ void k_fadj_scatter(int L, int ss, int hstride, double q, Items it, Strides sF, Strides sh, Strides so,
                               const double *__restrict__ F,
                               const double2 *__restrict__ hpole, const double2 *__restrict__ hpoleN,
                               double *__restrict__ out)
{
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    F += map_i * sF.map + slice * sF.slice;
    hpole += map_i * sh.map + slice * sh.slice;
    if (hpoleN) hpoleN += map_i * sh.map + slice * sh.slice;
    out += map_i * so.map + slice * so.slice;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)(L + ss) * L) return;
    const int t = (int)(i / L), m = (int)(i % L);
    double v[4];
    if (t < L - 1) {
        const double *src = F + ((size_t)m * hstride + t) * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = src[c];
    } else {
        const double2 *hp = t == L - 1 ? hpole : hpoleN;   // south pole; north pole (MWSS)
        const double2 a = hp[(L - 1) + m], b = hp[(L - 1) - m];
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    }
    if (m == 0) { v[2] = 0.0; v[3] = 0.0; }
    double *dst = out + ((size_t)t * L + m) * 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) dst[c] = q * v[c];
}

// ------------------------------------------------------------------ forward finish
// flm[l][m] = w_l * (g sum_b Q[b][l][|m|].side + g' sum_b Qx[b][l][|m|].side) * ((-1)^{|m|-nB} for m < 0)
//           (g = g_{|m|}^l, g' = g_{-|m|}^l: the sweeps leave the recursion's scale to here;
//           gtab null: already applied)
//           + south pole: w_l (-1)^{l+s} h~_s(pi) at m = s  (Eq. 29)
//           + north pole (MWSS): w_l h~_{-s}(0) at m = -s.
// Zero where l < max(|m|, |spin|).  One thread per (l, |m|) reads whole 32-byte
// records (side A = order +|m| in components 0,1, side B = order -|m| in 2,3) and
// writes both orders.  half (real signals, spin 0): only side A is read, and
// half = 1: flm[l][-m] = (-1)^m conj(flm[l][m]) (Hermitian symmetry);
// half = 2 (gradient of the real-signal inverse with respect to its complex
// input, whose orders m > 0 enter twice and order 0 through its real part):
// 2 x side A at m > 0, its real part at m = 0, zero at m < 0.
__global__ void k_finish_fwd(int L, int nblk, Items it, Strides sQ, Strides sQx, Strides sh, Strides sf,
                             const double *__restrict__ gtab, const double *__restrict__ Q,
                             const double *__restrict__ Qx, int nxp, const double *__restrict__ wl,
                             const double2 *__restrict__ hpole, const double2 *__restrict__ hpoleN,
                             double2 *__restrict__ flm, int half)
{
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    const int spin = it.spin[slice], nB = spin;
    Q += map_i * sQ.map + slice * sQ.slice;
    if (Qx) Qx += map_i * sQx.map + slice * sQx.slice;
    if (hpole) hpole += map_i * sh.map + slice * sh.slice;
    if (hpoleN) hpoleN += map_i * sh.map + slice * sh.slice;
    flm += map_i * sf.map + slice * sf.slice;
    wl += (size_t)slice * L;
    const int M = 2 * L - 1;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)L * L) return;
    const int l = (int)(i / L), am = (int)(i % L);
    const int as = spin < 0 ? -spin : spin;
    double2 a = make_double2(0.0, 0.0), b = make_double2(0.0, 0.0);
    if (l >= am && l >= as) {
        for (int bb = 0; bb < nblk; ++bb) {
            const double2 *q = reinterpret_cast<const double2 *>(Q + (((size_t)bb * L + l) * L + am) * 4);
            a = cadd(a, q[0]);
            if (!half) b = cadd(b, q[1]);
        }
        if (gtab) {
            const double g = gtab[(size_t)am * L + l];
            a = make_double2(g * a.x, g * a.y);
            b = make_double2(g * b.x, g * b.y);
        }
        if (Qx && am < nxp) {                          // orders below |n| from the other run's continuation
            double2 ax = make_double2(0.0, 0.0), bx = ax;
            for (int bb = 0; bb < nblk; ++bb) {
                const double2 *qx = reinterpret_cast<const double2 *>(Qx + (((size_t)bb * L + l) * nxp + am) * 4);
                ax = cadd(ax, qx[0]);
                bx = cadd(bx, qx[1]);
            }
            const double gx = gtab ? gtab[-(ptrdiff_t)am * L + l] : 1.0;
            a = make_double2(fma(gx, ax.x, a.x), fma(gx, ax.y, a.y));
            b = make_double2(fma(gx, bx.x, b.x), fma(gx, bx.y, b.y));
        }
        const double w = wl[l];
        const double wb = ((am - nB) & 1) ? -w : w;
        a = make_double2(a.x * w, a.y * w);
        b = make_double2(b.x * wb, b.y * wb);
        if (hpole) {
            const double c = ((l + spin) & 1) ? -w : w;
            if (am == spin) {
                const double2 hp = hpole[(L - 1) + am];
                a = make_double2(fma(c, hp.x, a.x), fma(c, hp.y, a.y));
            }
            if (am > 0 && -am == spin) {
                const double2 hp = hpole[(L - 1) - am];
                b = make_double2(fma(c, hp.x, b.x), fma(c, hp.y, b.y));
            }
        }
        if (hpoleN) {                                  // MWSS north pole: w_l h~_{-s}(0) at m = -s
            if (am == -spin) {
                const double2 hp = hpoleN[(L - 1) + am];
                a = make_double2(fma(w, hp.x, a.x), fma(w, hp.y, a.y));
            }
            if (am > 0 && -am == -spin) {
                const double2 hp = hpoleN[(L - 1) - am];
                b = make_double2(fma(w, hp.x, b.x), fma(w, hp.y, b.y));
            }
        }
    }
    if (half == 1) {
        b = (am & 1) ? make_double2(-a.x, a.y) : make_double2(a.x, -a.y);
    } else if (half == 2) {
        a = am == 0 ? make_double2(a.x, 0.0) : make_double2(2.0 * a.x, 2.0 * a.y);
        b = make_double2(0.0, 0.0);
    }
    double2 *row = flm + (size_t)l * M + (L - 1);
    row[am] = a;
    if (am > 0) row[-am] = b;
}

// ------------------------------------------------------------------ ring scaling
// map[t][p] *= w[t] for rings of nphi samples each (adjoint of a ring-weighted quadrature)
__global__ void k_ring_scale(int nring, int nphi, const double *__restrict__ w, double2 *__restrict__ map,
                             long long sm)
{
    map += blockIdx.y * sm;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)nring * nphi) return;
    const double s = w[i / nphi];
    map[i] = make_double2(map[i].x * s, map[i].y * s);
}

// real maps: map[t][p] *= w[t] over rings given by their start and length
__global__ void k_ring_scale_real(int nring, const long long *__restrict__ ring_start,
                                  const int *__restrict__ ring_nphi, const double *__restrict__ w,
                                  double *__restrict__ map, long long sm)
{
    const int r = blockIdx.x;
    if (r >= nring) return;
    map += blockIdx.y * sm;
    double *row = map + ring_start[r];
    const double s = w[r];
    for (int k = threadIdx.x; k < ring_nphi[r]; k += blockDim.x) row[k] *= s;
}

// Hermitian part of a coefficient cotangent: out[l][+-m] from
// h_m = (G[l][m] + (-1)^m conj G[l][-m]) / 2 (m > 0), h_0 = Re G[l][0], with
// out[l][-m] = (-1)^m conj h_m.  For a real map x and the forward transform F,
// Re <G, F x> = <h, F x>: the real-signal adjoint of the forward sees only h.
__global__ void k_hermitian_part(int L, const double2 *__restrict__ G, double2 *__restrict__ out, long long sG,
                                 long long so)
{
    G += blockIdx.y * sG;
    out += blockIdx.y * so;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)L * L) return;
    const int l = (int)(i / L), am = (int)(i % L);
    const int M = 2 * L - 1;
    const double2 *row = G + (size_t)l * M + (L - 1);
    double2 *orow = out + (size_t)l * M + (L - 1);
    const double2 a = row[am];
    if (am == 0) {
        orow[0] = make_double2(a.x, 0.0);
        return;
    }
    const double2 b = row[-am];
    const double sg = (am & 1) ? -1.0 : 1.0;
    const double2 h = make_double2(0.5 * (a.x + sg * b.x), 0.5 * (a.y - sg * b.y));
    orow[am] = h;
    orow[-am] = make_double2(sg * h.x, -sg * h.y);
}

// ------------------------------------------------------------------ SO(3) gamma DFT
// inverse: out[k][i] = sum_n e^{i n gamma_k} in[n][i];  forward: out[n][i] = q sum_k e^{-i n gamma_k} in[k][i]
// Bound by the latency of a few loads: the 2N - 1 roots are the same for every thread and,
// with N known to the compiler, sit in scalar registers at fixed places (indexed by a
// remainder per product, the products took 21 us of L = 96, N = 4 against 6).
template <int N>
__global__ __launch_bounds__(128) void k_gamma_dft(long long nper, int sign, double q, const double *__restrict__ roots,
                                                   const double2 *__restrict__ in, double2 *__restrict__ out,
                                                   long long si, long long so)
{
    constexpr int G = 2 * N - 1;
    in += blockIdx.y * si;
    out += blockIdx.y * so;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nper) return;
    double2 v[G];
#pragma unroll
    for (int a = 0; a < G; ++a) v[a] = in[(size_t)a * nper + i];
    // sign = +1 (inverse): v is indexed by n + N - 1, the result by k; -1: the reverse
    auto sums = [&](auto inverse) {
#pragma unroll
        for (int b = 0; b < G; ++b) {
            double2 acc = make_double2(0.0, 0.0);
#pragma unroll
            for (int a = 0; a < G; ++a) {
                constexpr bool inv = decltype(inverse)::value;
                const int e = ((inv ? a : b) - (N - 1)) * (inv ? b : a);
                acc = cadd(acc, cmul(v[a], ldroot(roots, (e % G + G) % G, inv ? 1 : -1)));
            }
            out[(size_t)b * nper + i] = make_double2(q * acc.x, q * acc.y);
        }
    };
    if (sign > 0) sums(std::true_type());
    else sums(std::false_type());
}

// ------------------------------------------------------------------ debug export of d
// d^l_{m,n}(theta_r) for one (ring, l) from the same init / step / renormalisation
// as the sweeps, handed to put(m, d, cont) for m = l down to 0; where this run is the
// unstable one below the switch order ms, the run -n is then continued to order
// -(ms-1) and put(m, d^l_{m,n}, true) gives the orders m < ms again from
// d^l_{m,n} = (-1)^{m-n} d^l_{-m,-n} (those replace the first values).
template <typename Put>
__device__ __forceinline__ void d_walk(int L, int n, int r, int l, const double *__restrict__ cot,
                                       const double *__restrict__ csc, const double *__restrict__ lsin,
                                       const double *__restrict__ lcos, const double *__restrict__ lbin,
                                       const double *__restrict__ kap, const double *__restrict__ gtab, Put put)
{
    const int an = n < 0 ? -n : n;
    if (l < an) return;
    double e, ep = 0.0;
    int E;
    d_init(l, n, dd_from(lbin + 2 * l), dd_from(lsin + 2 * r), dd_from(lcos + 2 * r), e, E);
    put(l, ldexp(e * gtab[(size_t)l * L + l], E), false);
    for (int m = l - 1; m >= 0; --m) {
        const double lam = fma(-(double)(m + 1), cot[r], (double)n * csc[r]);
        const double en = fma(kap[(size_t)m * L + l] * lam, e, -ep);
        ep = e;
        e = en;
        if (E != 0) renorm(e, ep, E);
        put(m, ldexp(e * gtab[(size_t)m * L + l], E), false);
    }
    const double ct = cot[r];
    const int ms = switch_order(n, ct, csc[r]);
    if (an > 0 && !ring_good(n, ct) && ms > 0) {
        E = 0;
        ep = 0.0;
        d_init(l, -n, dd_from(lbin + 2 * l), dd_from(lsin + 2 * r), dd_from(lcos + 2 * r), e, E);
        for (int m = l - 1; m >= -(ms - 1); --m) {
            const double lam = fma(-(double)(m + 1), ct, -(double)n * csc[r]);
            const double en = fma(kap[(ptrdiff_t)m * L + l] * lam, e, -ep);
            ep = e;
            e = en;
            if (E != 0) renorm(e, ep, E);
            const int mm = -m;
            if (mm >= 0 && mm < ms) {
                const double v = ldexp(e * gtab[(ptrdiff_t)m * L + l], E);
                put(mm, ((mm - n) & 1) ? -v : v, true);
            }
        }
    }
}

// out[r][m][l] = d^l_{m,n}(theta_r), one thread per (ring, l).
__global__ void k_debug_d(int L, int nreg, int n, const double *__restrict__ cot, const double *__restrict__ csc,
                          const double *__restrict__ lsin, const double *__restrict__ lcos,
                          const double *__restrict__ lbin, const double *__restrict__ kap,
                          const double *__restrict__ gtab, double *__restrict__ out)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    const int l = blockIdx.y;
    if (r >= nreg) return;
    double *o = out + (size_t)r * L * L;
    for (int m = 0; m <= l; ++m) o[(size_t)m * L + l] = 0.0;
    d_walk(L, n, r, l, cot, csc, lsin, lcos, lbin, kap, gtab,
           [&](int m, double v, bool) { o[(size_t)m * L + l] = v; });
}

// Unitarity check (debug): for ring rsel[i] and degree l, out[i][l] = {sum over
// m >= 0 of (d^l_{m,n})^2, d^l_{0,n}} with the values the sweeps use.  d^l(theta) is
// the matrix of a rotation in the (2l+1)-dimensional representation, real and
// orthogonal, so with d^l_{-m,n} = (-1)^{m-n} d^l_{m,-n} the runs n and -n give
// sum_{|m| <= l} (d^l_{m,n})^2 = 1.
__global__ void k_unitarity(int L, int n, int nsel, const int *__restrict__ rsel, const double *__restrict__ cot,
                            const double *__restrict__ csc, const double *__restrict__ lsin,
                            const double *__restrict__ lcos, const double *__restrict__ lbin,
                            const double *__restrict__ kap, const double *__restrict__ gtab,
                            double *__restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int l = blockIdx.y;
    if (i >= nsel) return;
    const int r = rsel[i];
    const int an = n < 0 ? -n : n;
    const double ct = cot[r];
    const int ms = switch_order(n, ct, csc[r]);
    const int ovr = (an > 0 && !ring_good(n, ct) && ms > 0) ? ms : 0;   // orders the continuation replaces
    double sum = 0.0, d0 = 0.0;
    d_walk(L, n, r, l, cot, csc, lsin, lcos, lbin, kap, gtab, [&](int m, double v, bool cont) {
        if (!cont && m < ovr) return;
        sum = fma(v, v, sum);
        if (m == 0) d0 = v;
    });
    out[((size_t)i * L + l) * 2] = sum;
    out[((size_t)i * L + l) * 2 + 1] = d0;
}

// ------------------------------------------------------------------ Bluestein filters
// For every Bluestein transform: bflt = DFT_len(b) / len with b_j = c_j (j < n),
// b_{len-j} = c_j (0 < j < n), 0 elsewhere -- the circular form of the chirp.
// Split form (convolution length M = 2H, H = f.len): by decimation in
// frequency the even samples are DFT_H(b_j + b_{j+H}) and the odd ones
// DFT_H((b_j - b_{j+H}) w^j), w = e^{-2 pi i/M}; with n < H, b_j = c_j for
// j < n and b_{j+H} = c_{H-j} for j > H - n.
__global__ __launch_bounds__(1024) void k_bluestein_prep(const FftArgs *__restrict__ ffts)
{
    extern __shared__ double2 buf[];
    const FftArgs *f = ffts + blockIdx.x;
    if (!f->blue || f->conv) return;                    // the theta filter's kernels carry their own spectra
    const int n = f->n, len = f->len;
    const double2 *ch = reinterpret_cast<const double2 *>(f->chirp);
    if (f->split) {
        const double2 *wm = reinterpret_cast<const double2 *>(f->twm);
        double2 *out = reinterpret_cast<double2 *>(const_cast<double *>(f->bflt));
        const double inv = 1.0 / (2.0 * (double)len);
        for (int half = 0; half < 2; ++half) {
            for (int j = threadIdx.x; j < len; j += blockDim.x) {
                const double2 lo = j < n ? ch[j] : make_double2(0.0, 0.0);
                const double2 hi = (j > len - n) ? ch[len - j] : make_double2(0.0, 0.0);
                buf[fft_place(f, j)] = half == 0 ? cadd(lo, hi) : cmul(csub(lo, hi), wm[j]);
            }
            __syncthreads();
            fft_forward<true>(buf, f, 0, f->nst);
            for (int k = threadIdx.x; k < len; k += blockDim.x) {
                const int p = fft_pos(f, k);
                const double2 v = buf[fft_place(f, p)];
                out[half * len + (f->perm ? conv_index(len, k) : p)] = make_double2(v.x * inv, v.y * inv);
            }
            __syncthreads();
        }
        return;
    }
    for (int i = threadIdx.x; i < len; i += blockDim.x) {
        double2 v = make_double2(0.0, 0.0);
        if (i < n) v = ch[i];
        else if (i > len - n) v = ch[len - i];
        buf[fft_place(f, i)] = v;
    }
    __syncthreads();
    fft_forward<true>(buf, f, 0, f->nst);
    double2 *out = reinterpret_cast<double2 *>(const_cast<double *>(f->bflt));
    const double inv = 1.0 / (double)len;
    for (int k = threadIdx.x; k < len; k += blockDim.x) {
        const int p = fft_pos(f, k);
        const double2 v = buf[fft_place(f, p)];
        out[f->perm ? conv_index(len, k) : p] = make_double2(v.x * inv, v.y * inv);
    }
}

// pole[(L-1) + m] = F[|m|][ring].side(m): the MW south-pole ring's Fourier line
__global__ void k_pole_from_F(int L, int hstride, int ring, Items it, Strides sF, Strides sh,
                              const double *__restrict__ F, double2 *__restrict__ pole)
{
    const int item = it.item0 + blockIdx.y, map_i = item / it.nslice, slice = item % it.nslice;
    F += map_i * sF.map + slice * sF.slice;
    pole += map_i * sh.map + slice * sh.slice;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * L - 1) return;
    const int m = i - (L - 1), am = m < 0 ? -m : m;
    const double *src = F + ((size_t)am * hstride + ring) * 4 + (m < 0 ? 2 : 0);
    pole[i] = make_double2(src[0], src[1]);
}

// ------------------------------------------------------------------ launchers
#define S2_LAUNCH_CHECK() do { hipError_t _e = hipGetLastError(); if (_e != hipSuccess) return _e; } while (0)

hipError_t launch_pair_spectra(hipStream_t st, int nmap, long long wsd, int L, int nreg, int nsw, int hstride,
                               int pstride, const double *H, double *S, double *D)
{
    if (nsw > pstride || 2 * nsw < nreg || nreg > hstride) return hipErrorInvalidValue;
    const size_t tot = (size_t)L * pstride;
    hipLaunchKernelGGL(k_pair_spectra, dim3((unsigned)((tot + 255) / 256), nmap), dim3(256), 0, st, L, nreg, nsw,
                       hstride, pstride, H, S, D, wsd);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_init_table(hipStream_t st, int L, int nreg, int n, const double *lsin, const double *lcos,
                             const double *lbin, double2 *init)
{
    const size_t tot = (size_t)L * nreg;
    hipLaunchKernelGGL(k_init_table, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, L, nreg, n, lsin, lcos,
                       lbin, init);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

// The DFT kernels of a plan whose rings need global scratch (fscr) run one item per
// launch, so that the items share it.
template <typename F>
static hipError_t over_items(int nitem, bool one_by_one, F go)
{
    const int step = one_by_one ? 1 : 32768;             // grid.y limit
    for (int i = 0; i < nitem; i += step) {
        go(i, nitem - i < step ? nitem - i : step);
        S2_LAUNCH_CHECK();
    }
    return hipSuccess;
}

// DFT kernels over the engine of a plan: go(engine, threads, LDS bytes).  conv: the
// convolution length where all rings share one length that needs Bluestein's identity.
template <typename F>
static hipError_t with_engine(const DftShape &d, F go)
{
    auto conv = [&](auto e) {
        using E = decltype(e);
        return go(e, E::T, std::max(d.n * sizeof(double2), (size_t)(E::T * E::V) * sizeof(double)));
    };
    switch (d.conv) {
    case 0: return d.threads > 1024 ? hipErrorInvalidValue : go(LdsDft{}, d.threads, d.lds);
    case 64: return conv(ConvDft<64, false>{});
    case 128: return conv(ConvDft<128, false>{});
    case 256: return conv(ConvDft<256, false>{});
    case 512: return conv(ConvDft<512, false>{});
    case 1024: return conv(ConvDft<1024, false>{});
    case 2048: return conv(ConvDft<2048, false>{});
    case 4096: return conv(ConvDft<4096, false>{});
    case 8192: return conv(ConvDft<8192, false>{});
    case 16384: return conv(ConvDft<8192, true>{});
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_phi_inv(hipStream_t st, const DftShape &dft, int nring, int L, int nreg, int nblk, Items it,
                          int nitem, Strides sp, Strides sf, Strides sm, const double *part, const int *mtop,
                          const double2 *flm, const double *wl, const int *ring_nphi, const long long *ring_start,
                          const int *ring_shift, const int *ring_fft, const FftArgs *ffts, double2 *map,
                          double2 *fscr)
{
    return with_engine(dft, [&](auto e, int nt, size_t lds) {
        return over_items(nitem, fscr != nullptr, [&](int i, int ny) {
            it.item0 = i;
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_phi_inv<decltype(e)>), dim3(nring, ny), dim3(nt), lds, st, L, nreg, nblk, it, sp, sf, sm, part,
                               mtop, flm, wl, ring_nphi, ring_start, ring_shift, ring_fft, ffts, map, fscr);
        });
    });
}

hipError_t launch_phi_fwd(hipStream_t st, const DftShape &dft, int nring, int hstride, int L, double q, Items it,
                          int nitem, Strides sm, Strides sF, const double2 *map, const int *ring_nphi,
                          const long long *ring_start, const int *ring_shift, const int *ring_fft, const FftArgs *ffts,
                          const double *ringq, double *F, double2 *fscr)
{
    return with_engine(dft, [&](auto e, int nt, size_t lds) {
        return over_items(nitem, fscr != nullptr, [&](int i, int ny) {
            it.item0 = i;
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_phi_fwd<decltype(e)>), dim3(hstride, ny), dim3(nt), lds, st, L, nring, hstride, q, it, sm, sF, map,
                               ring_nphi, ring_start, ring_shift, ring_fft, ffts, ringq, F, fscr);
        });
    });
}

hipError_t launch_phi_inv_real(hipStream_t st, const DftShape &dft, int npair, int L, int nreg, int nblk, int nmap,
                               long long sp, long long sf, long long sm, const int *pairs, const double *part,
                               const int *mtop, const double2 *flm, const double *wl, const int *ring_nphi,
                               const long long *ring_start, const int *ring_shift, const int *ring_fft,
                               const FftArgs *ffts, double *map, double2 *fscr)
{
    if (npair < 1) return hipErrorInvalidValue;
    return with_engine(dft, [&](auto e, int nt, size_t lds) {
        return over_items(nmap, fscr != nullptr, [&](int i, int ny) {
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_phi_inv_real<decltype(e)>), dim3(npair, ny), dim3(nt), lds, st, L, nreg, nblk, i, sp, sf, sm,
                               pairs, part, mtop, flm, wl, ring_nphi, ring_start, ring_shift, ring_fft, ffts, map, fscr);
        });
    });
}

hipError_t launch_phi_fwd_real(hipStream_t st, const DftShape &dft, int nring, int hstride, int npair, int L,
                               double q, int nmap, long long sm, long long sF, const int *pairs, const double *map,
                               const int *ring_nphi, const long long *ring_start, const int *ring_shift,
                               const int *ring_fft, const FftArgs *ffts, const double *ringq, double *F, double2 *fscr)
{
    if (hstride < nring || npair < 1) return hipErrorInvalidValue;
    const int nblocks = npair + (hstride - nring + 1) / 2;
    return with_engine(dft, [&](auto e, int nt, size_t lds) {
        return over_items(nmap, fscr != nullptr, [&](int i, int ny) {
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_phi_fwd_real<decltype(e)>), dim3(nblocks, ny), dim3(nt), lds, st, L, nring, hstride, npair, q, i,
                               sm, sF, pairs, map, ring_nphi, ring_start, ring_shift, ring_fft, ffts, ringq, F, fscr);
        });
    });
}

hipError_t launch_mw_filter(hipStream_t st, const DftShape &dft, int L, int ss, int hstride, Items it, int nitem,
                            Strides sF, Strides sh, const FftArgs *fN, const double *wq, const double *ph, double *F,
                            double2 *hpole, double2 *hpoleN, double2 *fscr, int half, int adj)
{
    if (ss && !hpoleN) return hipErrorInvalidValue;
    return with_engine(dft, [&](auto e, int nt, size_t lds) {
        return over_items(nitem, fscr != nullptr, [&](int i, int ny) {
            it.item0 = i;
            const int np = (L + 1) / 2;                      // pairs of orders, and their two sides
            auto *k = ss ? k_mw_filter<decltype(e), true> : k_mw_filter<decltype(e), false>;
            hipLaunchKernelGGL(k, dim3(half ? np : (np + 7) / 8 * 16, ny), dim3(nt), lds, st, L, hstride, it, sF, sh,
                               fN, wq, ph, F, hpole, hpoleN, fscr, half, adj);
        });
    });
}

hipError_t launch_ring_scale_real(hipStream_t st, int nmap, long long sm, int nring, const long long *ring_start,
                                  const int *ring_nphi, const double *w, double *map)
{
    if (nring < 1) return hipSuccess;
    return over_items(nmap, false, [&](int i, int ny) {
        hipLaunchKernelGGL(k_ring_scale_real, dim3(nring, ny), dim3(256), 0, st, nring, ring_start, ring_nphi, w,
                           map + i * sm, sm);
    });
}

hipError_t launch_hermitian_part(hipStream_t st, int nmap, long long sG, long long so, int L, const double2 *G,
                                 double2 *out)
{
    const size_t tot = (size_t)L * L;
    return over_items(nmap, false, [&](int i, int ny) {
        hipLaunchKernelGGL(k_hermitian_part, dim3((unsigned)((tot + 255) / 256), ny), dim3(256), 0, st, L, G + i * sG,
                           out + i * so, sG, so);
    });
}

hipError_t launch_ring_scale(hipStream_t st, int nmap, long long sm, int nring, int nphi, const double *w, double2 *map)
{
    const size_t tot = (size_t)nring * nphi;
    if (tot == 0) return hipSuccess;
    return over_items(nmap, false, [&](int i, int ny) {
        hipLaunchKernelGGL(k_ring_scale, dim3((unsigned)((tot + 255) / 256), ny), dim3(256), 0, st, nring, nphi, w,
                           map + i * sm, sm);
    });
}

hipError_t launch_finish_fwd(hipStream_t st, int L, int nblk, Items it, int nitem, Strides sQ, Strides sQx, Strides sh,
                             Strides sf, const double *gtab, const double *Q, const double *Qx, int nxp,
                             const double *wl, const double2 *hpole, const double2 *hpoleN, double2 *flm, int half)
{
    if (half && Qx) return hipErrorInvalidValue;                  // real signals: spin 0
    const size_t tot = (size_t)L * L;
    return over_items(nitem, false, [&](int i, int ny) {
        it.item0 = i;
        hipLaunchKernelGGL(k_finish_fwd, dim3((unsigned)((tot + 255) / 256), ny), dim3(256), 0, st, L, nblk, it, sQ,
                           sQx, sh, sf, gtab, Q, Qx, nxp, wl, hpole, hpoleN, flm, half);
    });
}

hipError_t launch_gamma_dft(hipStream_t st, int nmap, long long si, long long so, int N, long long nper, int sign,
                            double q, const double *roots, const double2 *in, double2 *out)
{
    return over_items(nmap, false, [&](int i, int ny) {
        auto go = [&](auto *k) {
            hipLaunchKernelGGL(k, dim3((unsigned)((nper + 127) / 128), ny), dim3(128), 0, st, nper, sign, q, roots,
                               in + i * si, out + i * so, si, so);
        };
        switch (N) {
        case 1: return go(k_gamma_dft<1>);
        case 2: return go(k_gamma_dft<2>);
        case 3: return go(k_gamma_dft<3>);
        case 4: return go(k_gamma_dft<4>);
        case 5: return go(k_gamma_dft<5>);
        case 6: return go(k_gamma_dft<6>);
        case 7: return go(k_gamma_dft<7>);
        default: return go(k_gamma_dft<8>);
        }
    });
}

hipError_t launch_unitarity(hipStream_t st, int L, int n, int nsel, const int *rsel, const double *cot,
                           const double *csc, const double *lsin, const double *lcos, const double *lbin,
                           const double *kap, const double *gtab, double *out)
{
    if (nsel < 1) return hipSuccess;
    dim3 grid((nsel + 63) / 64, L);
    hipLaunchKernelGGL(k_unitarity, grid, dim3(64), 0, st, L, n, nsel, rsel, cot, csc, lsin, lcos, lbin, kap, gtab,
                       out);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_debug_d(hipStream_t st, int L, int nreg, int n, const double *cot, const double *csc,
                          const double *lsin, const double *lcos, const double *lbin, const double *kap,
                          const double *gtab, double *out)
{
    dim3 grid((nreg + 63) / 64, L);
    hipLaunchKernelGGL(k_debug_d, grid, dim3(64), 0, st, L, nreg, n, cot, csc, lsin, lcos, lbin, kap, gtab, out);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_bluestein_filter(hipStream_t st, int nfft, const FftArgs *ffts, int nthreads, size_t lds)
{
    hipLaunchKernelGGL(k_bluestein_prep, dim3(nfft), dim3(nthreads), lds, st, ffts);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_fadj_gather(hipStream_t st, int L, int ss, int nblk, Items it, int nitem, Strides sp, Strides sf,
                              Strides sF, const double *part, const int *mtop, const double2 *flm, const double *wl,
                              int hstride, double *F)
{
    if (hstride < L + ss) return hipErrorInvalidValue;
    const size_t tot = (size_t)L * (L + ss);
    return over_items(nitem, false, [&](int i, int ny) {
        it.item0 = i;
        hipLaunchKernelGGL(k_fadj_gather, dim3((unsigned)((tot + 255) / 256), ny), dim3(256), 0, st, L, ss, nblk, it, sp,
                           sf, sF, part, mtop, flm, wl, hstride, F);
    });
}

hipError_t launch_fadj_scatter(hipStream_t st, int L, int ss, int hstride, double q, Items it, int nitem, Strides sF,
                               Strides sh, Strides so, const double *F, const double2 *hpole, const double2 *hpoleN,
                               double *out)
{
    if (ss && !hpoleN) return hipErrorInvalidValue;
    const size_t tot = (size_t)(L + ss) * L;
    return over_items(nitem, false, [&](int i, int ny) {
        it.item0 = i;
        hipLaunchKernelGGL(k_fadj_scatter, dim3((unsigned)((tot + 255) / 256), ny), dim3(256), 0, st, L, ss, hstride, q,
                           it, sF, sh, so, F, hpole, hpoleN, out);
    });
}

hipError_t launch_mask_low(hipStream_t st, int nmap, int nrun, const SweepRun *runs, int anmax, int nreg, int hstride,
                           const double *cot, const double *csc, const double *F, double *Hx, long long wsd,
                           long long nF, long long nHx, double *Qx, long long nz)
{
    const size_t tot = (size_t)anmax * hstride;
    if (tot == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mask_low, dim3((unsigned)((tot + 255) / 256), nmap * nrun), dim3(256), 0, st, nrun, runs, nreg,
                       hstride, cot, csc, F, Hx, wsd, nF, nHx, Qx, nz);
    S2_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_pole_from_F(hipStream_t st, int L, int hstride, int ring, Items it, int nitem, Strides sF, Strides sh,
                              const double *F, double2 *pole)
{
    return over_items(nitem, false, [&](int i, int ny) {
        it.item0 = i;
        hipLaunchKernelGGL(k_pole_from_F, dim3((2 * L - 1 + 255) / 256, ny), dim3(256), 0, st, L, hstride, ring, it, sF,
                           sh, F, pole);
    });
}

// Kernels with large dynamic LDS need the per-kernel limit raised.
hipError_t set_kernel_lds_limits(const DftShape &dft)
{
    auto raise = [](const void *k, size_t lds) {
        return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    };
    const hipError_t rc = raise((const void *)k_bluestein_prep, dft.lds);
    if (rc != hipSuccess) return rc;
    return with_engine(dft, [&](auto e, int, size_t lds) {
        using E = decltype(e);
        for (const void *k : {(const void *)k_phi_inv<E>, (const void *)k_phi_fwd<E>, (const void *)k_phi_inv_real<E>,
                              (const void *)k_phi_fwd_real<E>, (const void *)k_mw_filter<E, false>,
                              (const void *)k_mw_filter<E, true>}) {
            const hipError_t rk = raise(k, lds);
            if (rk != hipSuccess) return rk;
        }
        return hipSuccess;
    });
}

}  // namespace s2mi
