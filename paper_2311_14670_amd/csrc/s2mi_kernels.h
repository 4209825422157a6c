// s2mi_kernels.h -- host launchers of the gfx950 kernels (s2mi_kernels.hip, s2mi_sweep.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "s2mi_internal.h"

namespace s2mi {

// A run as the sweeps read it (device table of the plan).
struct SweepRun {
    int n, sliceA, sliceB, pad;
    const double2 *init;      // [nreg][L] start values of Eq. 27
    const double *ckI, *ckF;  // recursion states at the cuts of the inverse / forward work
};

// Arguments of the inverse sweep and its pack, shared by every map and run of a launch.
// Maps lie wsd doubles apart in the workspace, runs nC apart in the records, slices
// nP apart in the partial sums.
struct InvArgs {
    int L, nx;                // band-limit, negative orders held in the tables
    int nreg, nsw;            // rings of the output, rings swept (nsw < nreg: mirror rings)
    int nrun, half;           // runs; real signals: A side only
    int rt;                   // 64-ring tiles
    int nslot, merge;         // work slots, slots per workgroup
    int cb;                   // 8-degree chunks per block
    int rp;                   // ring stride of a cut's state
    long long wsd, nC, nP;
    const SweepRun *runs;
    const int4 *seg;          // pieces {block, top order, bottom order (0: to the run's lowest), cut or -1}
    const int *first;         // [nslot + 1] first piece of each slot
    double *C, *P;
};

struct FwdArgs {
    int L, nxp;               // band-limit, orders of the continuation sums
    int nx;                   // negative orders held in the tables
    int nreg, hstride;        // rings swept, ring stride of the spectra rows
    int nrun, half;
    int rb, nk;               // ring blocks, four-ring steps per wave
    int nslot, merge;
    int rp;
    long long wsd, nF, nQ, nHx, nQx;
    const SweepRun *runs;
    const int4 *seg;          // pieces {degree group, top order, bottom order, cut or -1}
    const int *first;
    const double *F, *Hx;     // ring spectra [slice][m][ring][4], low-order copies [run][2][m][ring][4]
    const double *S, *D;      // mirror-ring sweep: sums and differences (else null)
    double *Q, *Qx;
};

hipError_t launch_pack_inv(hipStream_t st, const InvArgs &a, int nmap, bool one, const double2 *flm, long long fstride,
                           const double *wl, const double *kap, const double *gtab);
hipError_t launch_sweep_inv(hipStream_t st, const InvArgs &a, int nmap, bool one, const double *cot, const double *csc);
hipError_t launch_sweep_fwd(hipStream_t st, const FwdArgs &a, int nmap, bool one, const double *cot, const double *csc,
                            const double *kap);
// The recursion state at the cuts of the runs' inverse (D degrees per block) or
// forward (groups of 64 degrees) work: rings [0, rp), zero past nreg.
hipError_t launch_cut_state(hipStream_t st, bool fwd, int L, int nreg, int rp, int D, int nblk, int par, int nrun,
                            const SweepRun *runs, const double *cot, const double *csc, const double *kap,
                            const int *cfirst, const int2 *cuts);
hipError_t launch_init_table(hipStream_t st, int L, int nreg, int n, const double *lsin, const double *lcos,
                             const double *lbin, double2 *init);

// Items of a launch: map * nslice + slice, from item0; spin of every slice.
struct Items {
    int nslice, item0;
    const int *spin;
};
// Stride of a buffer per map and per slice (in elements of its type).
struct Strides {
    long long map, slice;
};

hipError_t launch_pair_spectra(hipStream_t st, int nmap, long long wsd, int L, int nreg, int nsw, int hstride,
                               int pstride, const double *H, double *S, double *D);
// weights wl: [slice][L]
// the DFT engine of a plan's rings (and of its theta filter)
struct DftShape {
    int threads;      // LDS engine: threads and LDS of a workgroup
    size_t lds;
    int conv;         // convolution length where every ring has the length n and that needs
    int n;            // Bluestein's identity (register engine); 0: LDS engine
};

hipError_t launch_phi_inv(hipStream_t st, const DftShape &dft, int nring, int L, int nreg, int nblk, Items it,
                          int nitem, Strides sp, Strides sf, Strides sm, const double *part, const int *mtop,
                          const double2 *flm, const double *wl, const int *ring_nphi, const long long *ring_start,
                          const int *ring_shift, const int *ring_fft, const FftArgs *ffts, double2 *map,
                          double2 *fscr);
hipError_t launch_phi_fwd(hipStream_t st, const DftShape &dft, int nring, int hstride, int L, double q, Items it,
                          int nitem, Strides sm, Strides sF, const double2 *map, const int *ring_nphi,
                          const long long *ring_start, const int *ring_shift, const int *ring_fft, const FftArgs *ffts,
                          const double *ringq, double *F, double2 *fscr);
hipError_t launch_mw_filter(hipStream_t st, const DftShape &dft, int L, int ss, int hstride, Items it, int nitem,
                            Strides sF, Strides sh, const FftArgs *fN, const double *wq, const double *ph, double *F,
                            double2 *hpole, double2 *hpoleN, double2 *fscr, int half, int adj);
hipError_t launch_ring_scale(hipStream_t st, int nmap, long long sm, int nring, int nphi, const double *w,
                             double2 *map);
hipError_t launch_ring_scale_real(hipStream_t st, int nmap, long long sm, int nring, const long long *ring_start,
                                  const int *ring_nphi, const double *w, double *map);
hipError_t launch_hermitian_part(hipStream_t st, int nmap, long long sG, long long so, int L, const double2 *G,
                                 double2 *out);
// gtab null: the sums hold d already (matrix-core path)
hipError_t launch_finish_fwd(hipStream_t st, int L, int nblk, Items it, int nitem, Strides sQ, Strides sQx, Strides sh,
                             Strides sf, const double *gtab, const double *Q, const double *Qx, int nxp,
                             const double *wl, const double2 *hpole, const double2 *hpoleN, double2 *flm,
                             int half = 0);
// real signals (spin 0): pairs of rings share one complex DFT; maps are real doubles
hipError_t launch_phi_inv_real(hipStream_t st, const DftShape &dft, int npair, int L, int nreg, int nblk, int nmap,
                               long long sp, long long sf, long long sm, const int *pairs, const double *part,
                               const int *mtop, const double2 *flm, const double *wl, const int *ring_nphi,
                               const long long *ring_start, const int *ring_shift, const int *ring_fft,
                               const FftArgs *ffts, double *map, double2 *fscr);
hipError_t launch_phi_fwd_real(hipStream_t st, const DftShape &dft, int nring, int hstride, int npair, int L,
                               double q, int nmap, long long sm, long long sF, const int *pairs, const double *map,
                               const int *ring_nphi, const long long *ring_start, const int *ring_shift,
                               const int *ring_fft, const FftArgs *ffts, const double *ringq, double *F, double2 *fscr);
hipError_t launch_gamma_dft(hipStream_t st, int nmap, long long si, long long so, int N, long long nper, int sign,
                            double q, const double *roots, const double2 *in, double2 *out);
// Debug unitarity sums: out[i][l] = {sum_{m >= 0} (d^l_{m,n}(theta_{rsel[i]}))^2, d^l_{0,n}}.
hipError_t launch_unitarity(hipStream_t st, int L, int n, int nsel, const int *rsel, const double *cot,
                           const double *csc, const double *lsin, const double *lcos, const double *lbin,
                           const double *kap, const double *gtab, double *out);
hipError_t launch_debug_d(hipStream_t st, int L, int nreg, int n, const double *cot, const double *csc,
                          const double *lsin, const double *lcos, const double *lbin, const double *kap,
                          const double *gtab, double *out);
hipError_t launch_bluestein_filter(hipStream_t st, int nfft, const FftArgs *ffts, int nthreads, size_t lds);
hipError_t launch_fadj_gather(hipStream_t st, int L, int ss, int nblk, Items it, int nitem, Strides sp, Strides sf,
                              Strides sF, const double *part, const int *mtop, const double2 *flm, const double *wl,
                              int hstride, double *F);
hipError_t launch_fadj_scatter(hipStream_t st, int L, int ss, int hstride, double q, Items it, int nitem, Strides sF,
                               Strides sh, Strides so, const double *F, const double2 *hpole, const double2 *hpoleN,
                               double *out);
hipError_t launch_mask_low(hipStream_t st, int nmap, int nrun, const SweepRun *runs, int anmax, int nreg, int hstride,
                           const double *cot, const double *csc, const double *F, double *Hx, long long wsd,
                           long long nF, long long nHx, double *Qx, long long nz);
hipError_t launch_pole_from_F(hipStream_t st, int L, int hstride, int ring, Items it, int nitem, Strides sF, Strides sh,
                              const double *F, double2 *pole);
hipError_t set_kernel_lds_limits(const DftShape &dft);

}  // namespace s2mi
