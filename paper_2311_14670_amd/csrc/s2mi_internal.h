// s2mi_internal.h -- library-internal declarations shared by the host constant
// generator (g++), the kernels and the C-ABI layer (hipcc).
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace s2mi {

// ----------------------------------------------------------------- host constants
struct RingConsts {
    std::vector<double> theta, cot, csc;   // per ring
    std::vector<double> lsin, lcos;        // per ring, double-double (hi, lo): log2 sin(th/2), log2 cos(th/2)
};

#ifdef __SIZEOF_FLOAT128__
#if !defined(__HIP_DEVICE_COMPILE__) && !defined(__HIPCC__)
void fill_ring(RingConsts *rc, int r, __float128 th);
#endif
#endif
void host_mw_rings(int L, RingConsts *rc);
void host_mwss_rings(int L, RingConsts *rc);
void host_dh_rings(int L, RingConsts *rc, std::vector<double> *wq);
void host_gl_rings(int L, RingConsts *rc, std::vector<double> *wq);
void host_healpix_rings(int nside, RingConsts *rc, std::vector<int> *nphi,
                        std::vector<long long> *start, std::vector<int> *shift);
void host_log2_binom(int L, int n, std::vector<double> *out);
void host_recursion_tables(int L, int nx, std::vector<double> *kap, std::vector<double> *gtab);
void host_roots(int n, std::vector<double> *out);
void host_chirp(int n, std::vector<double> *out);
void host_mw_filter(int L, bool ss, std::vector<double> *wq, std::vector<double> *ph);
void host_shift_spectra(int L, int M, std::vector<double> *out);
void host_weights(int L, int kind, int spin, std::vector<double> *w);

// ----------------------------------------------------------------- FFT
constexpr int FFT_MAX_STAGES = 16;
constexpr int FFT_MAX_LEN = 8192;        // LDS-resident engine length (complex doubles)
constexpr size_t FFT_SCRATCH = 2 * (size_t)FFT_MAX_LEN;   // split Bluestein: complex scratch entries per workgroup

// One engine stage (quotients of numbers below 2^16 by one high multiplication: the error
// stays below 1 / 2^13)
struct FftStage {
    int rad;
    int sub;          // size of a block of the stage over its radix: the product of the later radices
    int nbf;          // butterflies, len / rad
    int tstep;        // nbf / sub
    unsigned msub;    // ceil(2^32 / sub)
    unsigned mrad;    // ceil(2^32 / rad)
};

// Everything a kernel needs to run one DFT of length n in LDS (passed by value).
struct FftArgs {
    int n;            // logical DFT length
    int len;          // engine length: n (mixed radix) or a power of two >= 2n-1 (Bluestein);
                      // split Bluestein: half the convolution length M = 2 len
    int blue;         // 1: Bluestein
    int split;        // 1: Bluestein convolution of length 2 len done as two LDS-resident halves
    int nst;          // engine stages
    FftStage stage[FFT_MAX_STAGES];
    int mix;          // LDS places: the bits of (i >> 3) that are mixed into i (below 16, len a multiple of it + 1)
    const uint16_t *slot; // not Bluestein: LDS place of bin k of the spectrum
    const double *tw;     // e^{-2 pi i k/len}, k < len (interleaved)
    const double *chirp;  // Bluestein: e^{+i pi k^2/n}, k < n
    const double *bflt;   // Bluestein: FFT of the chirp filter over the convolution length, divided by it
    const double *twm;    // split: e^{-2 pi i k/(2 len)}, k < len
    int conv;             // 1: a cyclic convolution, not a DFT: bflt is the spectrum of a
                          // kernel the plan supplies
    int perm;             // bflt in the order of the register engine (split: even, odd samples apart)
};

// ----------------------------------------------------------------- d-stage geometry
constexpr int SW_WAVES = 8;             // waves of a sweep workgroup (two per SIMD at 256 registers)
constexpr int INV_BLK = 256;            // degrees of an inverse block at most (8 waves x 4 chunks of 8)
constexpr int FWD_L = 64;               // degrees of a forward group
constexpr int FWD_KS = 8;               // four-ring steps of a forward wave at most
constexpr int FWD_KS_FEW = 2;           // and in the form for few rings
constexpr int FWD_BLK = 4 * FWD_KS * SW_WAVES;   // rings of a forward block at most
// Mirror-ring sweeps from this many rings on: one 64-ring tile instead of two (MI355X, pair of
// transforms, us, unpaired / paired: DH 48 rings 46.8 / 46.9, HEALPix 63 rings 46.8 / 47.4, DH 64
// 45.9 / 45.7, GL 64 48.1 / 46.9, DH 96 49.5 / 48.7, GL 100 58.4 / 55.0, HEALPix 127 59.1 / 56.8).
constexpr int PAIR_MIN_RINGS = 64;
// A batch's maps share launches up to this much work per compute unit (MI355X, MW L = 512, 16
// maps, inverse + forward sweep, ms: 256 orders 0.69 + 0.63, 1024 0.54 + 0.50, 4096 0.54 + 0.48,
// for four times the workspace) ..
constexpr double GROUP_ORDERS = 1024;
constexpr size_t GROUP_BYTES = (size_t)2 << 30;   // .. and this much workspace
constexpr int DSTAGE_MAX_WAVES = 8;     // d-tile generator workgroups: at most 512 threads

// One recursion run: fixed second index n of d^l_{m,n}; its A side feeds the
// slice of spin -n at orders +m, its B side the slice of spin +n at orders -m.
struct Run {
    int n;
    int sliceA;   // slice index or -1
    int sliceB;   // slice index or -1
};

}  // namespace s2mi
