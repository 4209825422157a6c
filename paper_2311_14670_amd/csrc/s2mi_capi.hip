// s2mi_capi.hip -- the C ABI of include/s2mi.h: plan construction, argument
// validation and the launch sequence of each transform.
//
// Paper: Price & McEwen, arXiv 2311.14670.  Spin SHT = phi-DFT (Eqs. 31-32) +
// Wigner d-stage (Eqs. 30, 33) on an isolatitude sampling (Sec. 4.1-4.2);
// Wigner transform = gamma-DFT + one spin SHT per n (Sec. 4.5, Eqs. 15-18).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <deque>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/s2mi.h"
#include "s2mi_conv.h"
#include "s2mi_internal.h"
#include "s2mi_kernels.h"
#include "s2mi_mfma.h"

using namespace s2mi;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int hipfail(hipError_t e, const char *what)
{
    return fail(S2_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIPCHK(expr, what)                      \
    do {                                        \
        hipError_t _e = (expr);                 \
        if (_e != hipSuccess) return hipfail(_e, what); \
    } while (0)

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

// ------------------------------------------------------------------ work of a sweep
// A sweep's blocks of degrees, each swept from its top order down, cut into pieces and
// dealt to slots of about equal length (s2mi_sweep.hip).
struct Work {
    int nblk = 1;                       // blocks (inverse) or degree groups (forward)
    int tiles = 1;                      // ring tiles (inverse) or ring blocks (forward); workgroups per run: tiles x slots
    int cb = 1, nk = 1;                 // inverse: chunks per block; forward: four-ring steps per wave
    int rp = 0;                         // ring stride of a cut's state
    int nslot = 1, quota = 1, pieces = 1;
    std::vector<int4> seg;
    std::vector<int> first;             // [nslot + 1]
    std::vector<int> cfirst;            // [nblk + 1] first cut of each block
    std::vector<int2> cuts;             // {order c, cut index}, descending in a block
    int4 *seg_d = nullptr;
    int *first_d = nullptr;
};

namespace {

// Orders that a slot's fixed cost (state load, start of the pipeline) amounts to, and the
// shortest slot.  A workgroup that runs several slots sweeps a block's consecutive
// pieces as one, so slots may be short: where the grid is small (few rings and degrees) the
// launch takes about 10 us and 1 us per order of a slot, waiting for memory.
// (Measured on MI355X, inverse / forward sweep, us, shortest slot of 16 orders with pieces
// run one by one -> 8 -> 4 orders: MW L = 64 spin 2 34 / 44 -> 21 / 28 -> 19 / 25; HEALPix
// nside 64, L = 128, 8 maps 46 / 75 -> 28 / 46 -> 27 / 39; SO(3) L = 96, N = 4 50 / 62 -> 30 / 43
// -> 32 / 44; MW L = 512, 16 maps, where pieces merge, 882 / 742 -> 537 / 498 -> 545 / 499;
// no difference from L = 1024 on.  The fixed cost at 5 or 20: within 2 %.)
constexpr int PIECE_COST = 10, PIECE_MIN = 4;

// Fills seg / first / cuts for blocks of `orders[b]` orders (largest work last), so
// that `items` runs sharing a launch of `tiles` ring tiles each fill `ncu` compute
// units: the slot count that minimises (rounds of workgroups) x (orders per slot +
// fixed cost).  force > 0: every block in `force` pieces (of at least 16 orders).
void deal_work(Work &W, const std::vector<int> &orders, int items, int ncu, int force)
{
    const int nb = (int)orders.size();
    long long total = 0;
    for (int o : orders) total += o;
    W.nblk = nb;
    W.seg.clear();
    W.first.assign(1, 0);
    W.cuts.clear();
    std::vector<std::vector<int>> cut_of(nb);
    if (force > 0) {
        for (int b = nb - 1; b >= 0; --b) {
            const int k = std::max(1, std::min(force, orders[b] / 16));
            int hi = orders[b] - 1;
            for (int j = k - 1; j >= 0; --j) {
                const int lo = j == 0 ? 0 : orders[b] * j / k / 4 * 4;
                if (lo > hi) continue;
                W.seg.push_back(make_int4(b, hi, lo, hi == orders[b] - 1 ? -1 : 0));
                if (lo > 0) cut_of[b].push_back(lo);
                W.first.push_back((int)W.seg.size());
                hi = lo - 1;
            }
        }
        W.quota = (int)((total + W.first.size() - 2) / std::max<size_t>(1, W.first.size() - 1));
    } else {
        const long long wg1 = (long long)W.tiles * items;
        int best = 1;
        double cost = 1e300;
        for (int s = 1; s <= 4096 && (s == 1 || total / s >= PIECE_MIN); ++s) {
            const double c = (double)((wg1 * s + ncu - 1) / ncu) * ((double)total / s + PIECE_COST);
            if (c < cost * 0.999) { cost = c; best = s; }
        }
        W.quota = std::max(PIECE_MIN, (int)((total + best - 1) / best));
        int room = W.quota;
        for (int b = nb - 1; b >= 0; --b) {
            int hi = orders[b] - 1;
            while (hi >= 0) {
                const int lo = std::max(0, hi + 1 - room) / 4 * 4;       // cuts at multiples of 4
                W.seg.push_back(make_int4(b, hi, lo, hi == orders[b] - 1 ? -1 : 0));
                if (lo > 0) cut_of[b].push_back(lo);
                room -= hi - lo + 1;
                hi = lo - 1;
                if (room < PIECE_MIN) {
                    W.first.push_back((int)W.seg.size());
                    room = W.quota;
                }
            }
        }
        if (W.first.back() != (int)W.seg.size()) W.first.push_back((int)W.seg.size());
    }
    W.nslot = (int)W.first.size() - 1;
    W.cfirst.assign(1, 0);
    W.pieces = 1;
    for (int b = 0; b < nb; ++b) {
        for (int c : cut_of[b]) W.cuts.push_back(make_int2(c, (int)W.cuts.size()));
        W.cfirst.push_back((int)W.cuts.size());
        W.pieces = std::max(W.pieces, (int)cut_of[b].size() + 1);
    }
    for (int4 &g : W.seg)
        if (g.w == 0)
            for (int q = W.cfirst[g.x]; q < W.cfirst[g.x + 1]; ++q)
                if (W.cuts[q].x == g.y + 1) g.w = W.cuts[q].y;
}

// Consecutive slots that one workgroup runs when `items` runs share the launch.
int merge_slots(const Work &W, long long items, int ncu)
{
    int best = 1;
    double cost = 1e300;
    for (int k = 1; k <= W.nslot; ++k) {
        const long long nt = (W.nslot + k - 1) / k, wg = nt * W.tiles * items;
        // a slot that continues the same block saves its state load
        const double c = (double)((wg + ncu - 1) / ncu) * ((double)k * W.quota + PIECE_COST);
        if (c < cost * 0.999) { cost = c; best = k; }
    }
    return best;
}

}  // namespace

// ------------------------------------------------------------------ plan
struct s2_plan_s {
    int L = 0, spin = 0, N = 1, sampling = 0, nside = 0, max_batch = 1, prec = 0;
    int nslice = 1;                       // 1 for S2, 2N-1 for SO(3)
    std::vector<int> slice_spin;          // spin of each slice (SO(3) slice k: n = k-(N-1), spin -n)
    int nring = 0, nreg = 0;              // rings of the sampling; rings the d-stage sweeps
    int nsw = 0;                          // rings the inverse sweep's lanes run (nreg, or the northern
                                          // half when mirror rings come from the symmetry)
    long long nsamp = 0;                  // samples per slice map
    std::vector<Run> runs;
    int ncu = 256;                        // compute units of the plan's device

    // device memory owned by the plan
    std::vector<void *> allocs;
    size_t plan_bytes = 0;

    // geometry (regular rings first; MW adds the south pole as ring nreg)
    double *cot = nullptr, *csc = nullptr, *lsin = nullptr, *lcos = nullptr;
    int *ring_nphi = nullptr, *ring_shift = nullptr, *ring_fft = nullptr;
    int *ring_pairs = nullptr;             // real signals: [npair][2] rings sharing one complex DFT (-1: none)
    int npair = 0;
    long long *ring_start = nullptr;
    // recursion tables
    double *kap = nullptr, *gtab = nullptr;
    std::vector<double *> lbin;   // per run
    std::vector<double2 *> init;  // per run [nreg][L]: start values of Eq. 27
    int *spin_d = nullptr;        // spin of every slice (device)
    // weights [slice][L]: SHT (Eqs. 30, 33), SO(3) inverse (Eq. 13), SO(3) forward (Eq. 14)
    double *w_sht = nullptr, *w_so3i = nullptr, *w_so3f = nullptr;
    double *w_so3f_n1 = nullptr;          // one-slice Wigner forward on the matrix cores: w_so3f times the gamma rule 2 pi
    double *w_fadj = nullptr;             // HEALPix: (4 pi / Npix) w_l, the adjoint of the forward quadrature
    // FFT
    std::vector<FftArgs> ffts_h;
    FftArgs *ffts = nullptr;
    DftShape dft{64, 0, 0, 0};
    FftArgs fN{};                          // MW ring / theta-torus length 2L-1
    double *wq = nullptr, *ph = nullptr;   // MW theta filter
    double *ringq = nullptr;               // DH / GL: forward quadrature weight of each ring (phi rule included)
    double *groots = nullptr;              // e^{-2 pi i k/(2N-1)}
    // d-stage work assignment
    // stable-direction remedy: a run with n cos(theta) < 0 at a ring continues to
    // orders -(|n|-1) and supplies the other run's orders |m| < |n| there
    int nxp = 0;                           // max |n| over the runs (orders below it are remedied)
    int nx = 0;                            // negative orders held in the tables: max(0, nxp - 1)
    Work inv, fwd;                         // work of the inverse and forward sweeps
    int *mtop = nullptr;                   // top order of each inverse block
    bool one = false;                      // runs feed one side each (spin-s sphere plans)
    // forward sweep over the northern rings (spin 0, symmetric samplings: nsw < nreg)
    bool fwd_pair = false;
    int pstride = 0;
    size_t off_Fp = 0;                    // workspace: sums and differences of mirror-ring spectra
    int hstride = 0;                       // ring stride of the forward spectra (padded to the sweep's slots)
    SweepRun *runs_d = nullptr;            // the runs as the sweeps read them
    int order_tiles = 1;                   // most pieces that one block of degrees is cut into
    int group = 1;                         // maps of a batch that share the launches (FP64)
    size_t ws1 = 0;                        // workspace bytes of one map
    // workspace layout (bytes)
    size_t off_C = 0, off_P = 0, off_maps = 0, off_F = 0, off_Q = 0, off_hpole = 0, ws_bytes = 0;
    size_t off_fscr = 0, sz_fscr = 0;      // split-Bluestein scratch: FFT_SCRATCH complex per FFT workgroup
    size_t off_hsym = 0;                   // spin-0 S2 plans: Hermitian part of a coefficient cotangent
    size_t szC = 0, szP = 0, szF = 0, szQ = 0;   // C per run, others per slice
    size_t off_Hx = 0, off_Qx = 0, szHx = 0, szQx = 0;

    // matrix-core contraction path (precision FP32 / split BF16): batched over maps
    bool mfma = false;
    MfmaGeom mg{};
    int mch = 1;                           // orders per generated d chunk
    int gen_nblk = 1, gen_waves = 1;
    int *gen_lchunk = nullptr, *mtop1 = nullptr;
    double2 *kg = nullptr;                 // [m][lrow] {kappa, g}
    size_t nslots = 0;                     // recursion state slots (l) of the generator
    size_t off_D = 0, off_S = 0, off_AH = 0, off_mP = 0, off_mF = 0, off_mQ = 0, off_mhp = 0, off_mmaps = 0;
    size_t off_mQx = 0;
    size_t state_bytes = 0;

    // stage timing
    bool timing = false;
    struct TimedLaunch { int stage; hipEvent_t a, b; };
    std::vector<TimedLaunch> tl;

    template <typename T>
    int dalloc(T **p, size_t count, const char *what)
    {
        void *q = nullptr;
        const size_t bytes = std::max<size_t>(count * sizeof(T), 16);
        hipError_t e = hipMalloc(&q, bytes);
        if (e != hipSuccess) return fail(S2_ERR_OOM, "hipMalloc(%zu) for %s: %s", bytes, what, hipGetErrorString(e));
        allocs.push_back(q);
        plan_bytes += bytes;
        *p = static_cast<T *>(q);
        return S2_OK;
    }
    ~s2_plan_s()
    {
        for (auto &t : tl) { (void)hipEventDestroy(t.a); (void)hipEventDestroy(t.b); }
        for (void *q : allocs) (void)hipFree(q);
    }
};

namespace {

// factor n over the engine radices; returns remainder (1 if fully factored)
int factor_radices(int n, std::vector<int> &rad)
{
    rad.clear();
    while (n % 8 == 0) { rad.push_back(8); n /= 8; }
    while (n % 4 == 0) { rad.push_back(4); n /= 4; }
    while (n % 2 == 0) { rad.push_back(2); n /= 2; }
    while (n % 9 == 0) { rad.push_back(9); n /= 9; }       // one stage instead of two radix-3 ones
    for (int p : {13, 11, 7, 5, 3})
        while (n % p == 0) { rad.push_back(p); n /= p; }
    return n;
}

// host staging kept alive until the plan's upload has completed (deque: references
// to earlier entries stay valid while later ones are added)
struct Staging {
    std::deque<std::vector<double>> d;
    std::deque<std::vector<int>> i;
    std::deque<std::vector<long long>> ll;
    std::vector<SweepRun> sr;
};

template <typename T>
int upload(s2_plan_s *P, T **dst, const std::vector<T> &src, hipStream_t st, const char *what)
{
    int rc = P->dalloc(dst, src.size(), what);
    if (rc) return rc;
    if (!src.empty()) HIPCHK(hipMemcpyAsync(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice, st), what);
    return S2_OK;
}

// position of frequency k in the order that the engine's forward stages leave
int fft_position(const FftArgs &f, int k)
{
    int p = 0;
    for (int s = 0; s < f.nst; k /= f.stage[s].rad, ++s) p += k % f.stage[s].rad * f.stage[s].sub;
    return p;
}

int build_fft(s2_plan_s *P, int n, Staging &stg, hipStream_t st, FftArgs *out)
{
    FftArgs f{};
    std::vector<int> rad;
    const int rem = factor_radices(n, rad);
    f.n = n;
    if (rem == 1) {
        f.blue = 0;
        f.len = n;
    } else {
        f.blue = 1;
        int M = 1;
        while (M < 2 * n - 1) M *= 2;
        f.len = M;
        if (M > FFT_MAX_LEN && M / 2 <= FFT_MAX_LEN && n < M / 2) {
            f.split = 1;                                   // two LDS-resident halves of length M/2
            f.len = M / 2;
        }
        factor_radices(f.len, rad);
    }
    if (f.len > FFT_MAX_LEN)
        return fail(S2_ERR_UNSUPPORTED, "DFT length %d needs an engine of %d points (> %d)", n, f.len, FFT_MAX_LEN);
    if ((int)rad.size() > FFT_MAX_STAGES) return fail(S2_ERR_UNSUPPORTED, "too many FFT stages for %d", n);
    f.nst = (int)rad.size();
    for (int s = f.nst - 1, q = 1; s >= 0; --s) {
        FftStage &g = f.stage[s];
        g.rad = rad[s];
        g.sub = q;
        g.nbf = f.len / rad[s];
        g.tstep = g.nbf / q;
        g.msub = q > 1 ? 0xffffffffu / (unsigned)q + 1u : 0u;
        g.mrad = 0xffffffffu / (unsigned)rad[s] + 1u;
        q *= rad[s];
    }
    f.mix = f.len % 16 == 0 ? 15 : f.len % 8 == 0 ? 7 : 0;
    int rc;
    // twiddles and, behind them, the bins' places: one upload per length (HEALPix plans have
    // nside of them)
    stg.d.emplace_back();
    std::vector<double> &tab = stg.d.back();
    host_roots(f.len, &tab);
    if (!f.blue) {
        std::vector<uint16_t> slot(n);
        for (int k = 0; k < n; ++k) {
            const int p = fft_position(f, k);
            slot[k] = (uint16_t)(p ^ ((p >> 3) & f.mix));
        }
        tab.resize(2 * (size_t)f.len + ((size_t)n + 3) / 4);
        std::memcpy(tab.data() + 2 * (size_t)f.len, slot.data(), (size_t)n * sizeof(uint16_t));
    }
    double *tw;
    rc = upload(P, &tw, tab, st, "fft twiddles");
    if (rc) return rc;
    f.tw = tw;
    if (!f.blue) f.slot = reinterpret_cast<const uint16_t *>(tw + 2 * (size_t)f.len);
    if (f.blue) {
        stg.d.emplace_back();
        host_chirp(n, &stg.d.back());
        double *ch, *bf;
        if ((rc = upload(P, &ch, stg.d.back(), st, "bluestein chirp"))) return rc;
        const int conv = f.split ? 2 * f.len : f.len;    // convolution length
        if ((rc = P->dalloc(&bf, 2 * (size_t)conv, "bluestein filter"))) return rc;
        f.chirp = ch;
        f.bflt = bf;
        if (f.split) {
            stg.d.emplace_back();
            host_roots(conv, &stg.d.back());
            stg.d.back().resize(2 * (size_t)f.len);       // e^{-2 pi i k/conv}, k < len
            double *wm;
            if ((rc = upload(P, &wm, stg.d.back(), st, "bluestein split roots"))) return rc;
            f.twm = wm;
        }
    }
    *out = f;
    return S2_OK;
}

int fft_threads_for(int len) { return std::min(1024, std::max(64, ((len / 8 + 63) / 64) * 64)); }

}  // namespace

extern "C" {

const char *s2_error_string(int code)
{
    switch (code) {
    case S2_OK: return "ok";
    case S2_ERR_INVALID_ARG: return "invalid argument";
    case S2_ERR_UNSUPPORTED: return "unsupported";
    case S2_ERR_OOM: return "out of memory";
    case S2_ERR_HIP: return "HIP runtime error";
    case S2_ERR_CHECK: return "debug check failed";
    default: return "unknown error";
    }
}

const char *s2_last_error_message(void) { return g_last_error.c_str(); }

int s2_plan_info(s2_plan_t P, s2_plan_info_t *info)
{
    if (!P || !info) return fail(S2_ERR_INVALID_ARG, "s2_plan_info: null argument");
    info->L = P->L;
    info->spin = P->spin;
    info->N = P->N;
    info->nside = P->nside;
    info->sampling = P->sampling;
    info->precision = P->prec;
    info->max_batch = P->max_batch;
    info->nrings = P->nring;
    info->nsamples = P->nsamp;
    info->ncoeffs = (long long)P->L * (2 * P->L - 1);
    info->workspace_bytes = P->ws_bytes;
    info->plan_device_bytes = P->plan_bytes;
    info->swept_rings = P->nsw;
    info->order_tiles = P->order_tiles;
    return S2_OK;
}

int s2_plan_destroy(s2_plan_t P)
{
    if (!P) return S2_OK;
    (void)hipDeviceSynchronize();
    delete P;
    return S2_OK;
}

static int plan_create_impl(s2_plan_t *out, int L, int spin, int N, s2_sampling_t sampling, int nside, int max_batch,
                            s2_precision_t prec, void *hip_stream)
{
    if (!out) return fail(S2_ERR_INVALID_ARG, "s2_plan_create: out is NULL");
    *out = nullptr;
    if (L < 2 || L > 4096) return fail(S2_ERR_INVALID_ARG, "L=%d outside [2, 4096]", L);
    if (N < 1 || N > L) return fail(S2_ERR_INVALID_ARG, "N=%d outside [1, L]", N);
    if (N > 8) return fail(S2_ERR_UNSUPPORTED, "N=%d: SO(3) plans support N <= 8", N);
    if (N > 1 && spin != 0) return fail(S2_ERR_INVALID_ARG, "SO(3) plans (N > 1) take spin 0");
    if (spin <= -L || spin >= L) return fail(S2_ERR_INVALID_ARG, "|spin|=%d must be < L=%d", spin, L);
    if (sampling != S2_MW && sampling != S2_HEALPIX && sampling != S2_DH && sampling != S2_GL && sampling != S2_MWSS)
        return fail(S2_ERR_INVALID_ARG, "unknown sampling %d", (int)sampling);
    if (sampling == S2_HEALPIX && (nside < 1 || nside > 2048)) return fail(S2_ERR_INVALID_ARG, "nside=%d outside [1, 2048]", nside);
    if (sampling != S2_MW && N > 1) return fail(S2_ERR_UNSUPPORTED, "SO(3) plans need MW sampling");
    if (sampling != S2_HEALPIX) nside = 0;
    if (max_batch < 1) return fail(S2_ERR_INVALID_ARG, "max_batch=%d < 1", max_batch);
    if (prec != S2_FP64 && prec != S2_CONTRACT_FP32 && prec != S2_CONTRACT_SPLIT_BF16)
        return fail(S2_ERR_INVALID_ARG, "unknown precision mode %d", (int)prec);
    hipStream_t st = (hipStream_t)hip_stream;

    s2_plan_s *P = new (std::nothrow) s2_plan_s();
    if (!P) return fail(S2_ERR_OOM, "host allocation of the plan failed");
    P->L = L; P->spin = spin; P->N = N; P->sampling = sampling; P->nside = nside; P->max_batch = max_batch; P->prec = prec;
    P->nslice = 2 * N - 1;
    const bool so3 = N > 1;
    Staging stg;
    int rc;
    auto bail = [&](int code) { delete P; return code; };
    // a HIP failure while the plan is built releases everything it holds
#define PLANCHK(expr, what)                                  \
    do {                                                     \
        hipError_t _e = (expr);                              \
        if (_e != hipSuccess) return bail(hipfail(_e, what)); \
    } while (0)

    // slices and runs
    P->slice_spin.resize(P->nslice);
    if (!so3) P->slice_spin[0] = spin;
    else for (int k = 0; k < P->nslice; ++k) P->slice_spin[k] = -(k - (N - 1));
    auto slice_of_spin = [&](int s) {
        for (int k = 0; k < P->nslice; ++k) if (P->slice_spin[k] == s) return k;
        return -1;
    };
    {
        std::vector<int> ns;
        for (int k = 0; k < P->nslice; ++k) {
            const int s = P->slice_spin[k];
            for (int n : {-s, s}) if (std::find(ns.begin(), ns.end(), n) == ns.end()) ns.push_back(n);
        }
        for (int n : ns) P->runs.push_back(Run{n, slice_of_spin(-n), slice_of_spin(n)});
    }

    // geometry
    RingConsts rc_h;
    std::vector<int> nphi, shift;
    std::vector<long long> start;
    if (sampling == S2_MW) {
        host_mw_rings(L, &rc_h);
        P->nreg = L - 1;
        P->nring = L;
        nphi.assign(L, 2 * L - 1);
        shift.assign(L, 0);
        start.resize(L);
        for (int t = 0; t < L; ++t) start[t] = (long long)t * (2 * L - 1);
        P->nsamp = (long long)L * (2 * L - 1);
    } else if (sampling == S2_MWSS) {
        // rings 0 .. L-2: theta = pi (r+1)/L; ring L-1: south pole; ring L: north pole
        host_mwss_rings(L, &rc_h);
        P->nreg = L - 1;
        P->nring = L + 1;
        nphi.assign(L + 1, 2 * L);
        shift.assign(L + 1, 0);
        start.resize(L + 1);
        for (int r = 0; r < L - 1; ++r) start[r] = (long long)(r + 1) * 2 * L;
        start[L - 1] = (long long)L * 2 * L;
        start[L] = 0;
        P->nsamp = (long long)(L + 1) * 2 * L;
    } else if (sampling == S2_DH || sampling == S2_GL) {
        // equiangular-phi rings without poles, each ring swept; forward by quadrature
        stg.d.emplace_back(); std::vector<double> &rq = stg.d.back();
        if (sampling == S2_DH) host_dh_rings(L, &rc_h, &rq);
        else host_gl_rings(L, &rc_h, &rq);
        P->nring = (int)rq.size();
        P->nreg = P->nring;
        nphi.assign(P->nring, 2 * L - 1);
        shift.assign(P->nring, 0);
        start.resize(P->nring);
        for (int t = 0; t < P->nring; ++t) start[t] = (long long)t * (2 * L - 1);
        P->nsamp = (long long)P->nring * (2 * L - 1);
        if ((rc = upload(P, &P->ringq, rq, st, "ring weights"))) return bail(rc);
    } else {
        host_healpix_rings(nside, &rc_h, &nphi, &start, &shift);
        P->nring = 4 * nside - 1;
        P->nreg = P->nring;
        P->nsamp = 12LL * nside * nside;
    }
    if ((rc = upload(P, &P->cot, rc_h.cot, st, "cot"))) return bail(rc);
    if ((rc = upload(P, &P->csc, rc_h.csc, st, "csc"))) return bail(rc);
    if ((rc = upload(P, &P->lsin, rc_h.lsin, st, "lsin"))) return bail(rc);
    if ((rc = upload(P, &P->lcos, rc_h.lcos, st, "lcos"))) return bail(rc);
    if ((rc = upload(P, &P->ring_nphi, nphi, st, "ring_nphi"))) return bail(rc);
    if ((rc = upload(P, &P->ring_shift, shift, st, "ring_shift"))) return bail(rc);
    if ((rc = upload(P, &P->ring_start, start, st, "ring_start"))) return bail(rc);
    {
        // real signals: rings of equal length and phase offset pair up in ring order
        // (MW-type grids: (0,1), (2,3), ...; HEALPix: a cap ring with its mirror ring)
        stg.i.emplace_back();
        std::vector<int> &pr = stg.i.back();
        std::map<std::pair<int, int>, int> open_ring;
        for (int r = 0; r < P->nring; ++r) {
            const auto key = std::make_pair(nphi[r], shift[r]);
            auto it = open_ring.find(key);
            if (it == open_ring.end()) { open_ring[key] = r; continue; }
            pr.push_back(it->second);
            pr.push_back(r);
            open_ring.erase(it);
        }
        for (const auto &kv : open_ring) { pr.push_back(kv.second); pr.push_back(-1); }
        P->npair = (int)pr.size() / 2;
        if ((rc = upload(P, &P->ring_pairs, pr, st, "ring pairs"))) return bail(rc);
    }

    // FFTs: one per distinct ring length
    {
        std::vector<int> lens, rf(P->nring);
        for (int r = 0; r < P->nring; ++r) {
            auto it = std::find(lens.begin(), lens.end(), nphi[r]);
            if (it == lens.end()) { lens.push_back(nphi[r]); rf[r] = (int)lens.size() - 1; }
            else rf[r] = (int)(it - lens.begin());
        }
        int maxlen = 0;
        for (int n : lens) {
            FftArgs f;
            if ((rc = build_fft(P, n, stg, st, &f))) return bail(rc);
            P->ffts_h.push_back(f);
            maxlen = std::max(maxlen, f.len);
        }
        // rings of one length that needs Bluestein's identity: the register engine
        if (lens.size() == 1 && P->ffts_h[0].blue) {
            FftArgs &f = P->ffts_h[0];
            f.perm = 1;
            P->dft.conv = (f.split ? 2 : 1) * f.len;
            P->dft.n = f.n;
        }
        if (sampling == S2_MW || sampling == S2_MWSS) P->fN = P->ffts_h[0];
        // MW with a ring length N = 2L - 1 that needs Bluestein's identity: the theta
        // filter's two half-step shifts are circular convolutions of length N, each run
        // as one convolution of the same length M instead of two Bluestein DFTs
        if (sampling == S2_MW && P->fN.blue) {
            const int M = P->fN.split ? 2 * P->fN.len : P->fN.len;
            stg.d.emplace_back();
            std::vector<double> nat;
            host_shift_spectra(L, M, &nat);
            stg.d.back().resize(nat.size());
            const int len = P->fN.len;
            for (int which = 0; which < 2; ++which)
                for (int k = 0; k < M; ++k) {
                    const int at = P->fN.split ? (k & 1) * len + conv_index(len, k / 2) : conv_index(len, k);
                    for (int c = 0; c < 2; ++c)
                        stg.d.back()[2 * ((size_t)which * M + at) + c] = nat[2 * ((size_t)which * M + k) + c];
                }
            double *cs;
            if ((rc = upload(P, &cs, stg.d.back(), st, "theta filter shift spectra"))) return bail(rc);
            FftArgs f = P->fN;                             // same engine; entries 1 and 2
            f.conv = 1;
            f.bflt = cs;
            P->ffts_h.push_back(f);
            f.bflt = cs + 2 * (size_t)M;
            P->ffts_h.push_back(f);
        }
        P->dft.threads = fft_threads_for(maxlen);
        P->dft.lds = (size_t)maxlen * sizeof(double2);
        if ((rc = upload(P, &P->ring_fft, rf, st, "ring_fft"))) return bail(rc);
        if ((rc = upload(P, &P->ffts, P->ffts_h, st, "fft table"))) return bail(rc);
        PLANCHK(set_kernel_lds_limits(P->dft), "LDS limits");
        int nblue = 0;
        for (auto &f : P->ffts_h) nblue += f.blue;
        if (nblue) PLANCHK(launch_bluestein_filter(st, (int)P->ffts_h.size(), P->ffts, P->dft.threads, P->dft.lds), "bluestein filters");
    }
    if (sampling == S2_MW || sampling == S2_MWSS) {
        stg.d.emplace_back(); std::vector<double> &wq = stg.d.back();
        stg.d.emplace_back(); std::vector<double> &ph = stg.d.back();
        host_mw_filter(L, sampling == S2_MWSS, &wq, &ph);
        if ((rc = upload(P, &P->wq, wq, st, "mw filter weights"))) return bail(rc);
        if (!P->dft.conv) {                                // in the order of the LDS engine's positions
            const std::vector<double> nat(ph);
            const FftArgs &f = P->fN;
            for (int k = 0; k < f.n; ++k) {
                const int p = fft_position(f, k);
                ph[2 * p] = nat[2 * k];
                ph[2 * p + 1] = nat[2 * k + 1];
            }
        }
        if ((rc = upload(P, &P->ph, ph, st, "mw half-shift phases"))) return bail(rc);
    }
    if (sampling == S2_MW && spin == 0) {
        stg.d.emplace_back();
        host_roots(2 * N - 1, &stg.d.back());
        if ((rc = upload(P, &P->groots, stg.d.back(), st, "gamma roots"))) return bail(rc);
    }

    // recursion tables, rows m in [-nx, L) (device pointers at row m = 0)
    {
        for (const Run &r : P->runs) P->nxp = std::max(P->nxp, r.n < 0 ? -r.n : r.n);
        P->nx = std::max(0, P->nxp - 1);
        stg.d.emplace_back(); std::vector<double> &kap = stg.d.back();
        stg.d.emplace_back(); std::vector<double> &g = stg.d.back();
        host_recursion_tables(L, P->nx, &kap, &g);
        if ((rc = upload(P, &P->kap, kap, st, "kappa table"))) return bail(rc);
        if ((rc = upload(P, &P->gtab, g, st, "g table"))) return bail(rc);
        P->kap += (size_t)P->nx * L;
        P->gtab += (size_t)P->nx * L;
    }
    for (const Run &r : P->runs) {
        stg.d.emplace_back();
        host_log2_binom(L, r.n, &stg.d.back());
        double *lb;
        if ((rc = upload(P, &lb, stg.d.back(), st, "log2 binomials"))) return bail(rc);
        P->lbin.push_back(lb);
    }
    for (int kind = 0; kind < 3; ++kind) {
        stg.d.emplace_back();
        std::vector<double> &all = stg.d.back();
        for (int k = 0; k < P->nslice; ++k) {
            std::vector<double> w;
            host_weights(L, kind, P->slice_spin[k], &w);
            all.insert(all.end(), w.begin(), w.begin() + L);
        }
        if ((rc = upload(P, kind == 0 ? &P->w_sht : kind == 1 ? &P->w_so3i : &P->w_so3f, all, st, "weights")))
            return bail(rc);
    }
    stg.i.emplace_back(P->slice_spin);
    if ((rc = upload(P, &P->spin_d, stg.i.back(), st, "slice spins"))) return bail(rc);
    if (!so3 && sampling == S2_MW && spin == 0 && prec != S2_FP64) {
        // so3_forward with N = 1 on the matrix-core path folds the gamma rule 2 pi/(2N-1) = 2 pi
        // (Eq. 16) into the finish's weights instead of scaling a copy of the samples
        stg.d.emplace_back();
        host_weights(L, 2, 0, &stg.d.back());
        for (double &v : stg.d.back()) v *= 2.0 * M_PI;
        if ((rc = upload(P, &P->w_so3f_n1, stg.d.back(), st, "one-slice Wigner forward weights"))) return bail(rc);
    }

    // Sweep work.  Spin-0 plans of the N/S-symmetric samplings sweep only the northern
    // rings and produce each mirror ring from d^l_{m,0}(pi - theta) = (-1)^{l+m}
    // d^l_{m,0}(theta), halving the recursion and the products.
    // S2MI_RING_PAIRING=0 / 1 turns that off / on wherever it applies (tests, tuning).
    P->one = !so3 && spin != 0;
    const int nrun = (int)P->runs.size();
    {
        int dev = 0;
        PLANCHK(hipGetDevice(&dev), "hipGetDevice");
        PLANCHK(hipDeviceGetAttribute(&P->ncu, hipDeviceAttributeMultiprocessorCount, dev), "CU count");
        P->nsw = P->nreg;
        const bool sym = sampling == S2_DH || sampling == S2_GL || sampling == S2_MWSS || sampling == S2_HEALPIX;
        const char *pm = std::getenv("S2MI_RING_PAIRING");
        const int mode = pm && pm[0] == '0' ? 0 : pm && pm[0] == '1' ? 1 : -1;
        if (sym && spin == 0 && !so3 && prec == S2_FP64 && mode != 0 && (mode == 1 || P->nreg >= PAIR_MIN_RINGS))
            P->nsw = (P->nreg + 1) / 2;
        P->fwd_pair = P->nsw < P->nreg;
        // S2MI_ORDER_TILES=k cuts every block into k pieces (1: none)
        int force = 0;
        if (const char *ev = std::getenv("S2MI_ORDER_TILES")) force = std::max(1, std::min(8, std::atoi(ev)));
        if (prec != S2_FP64) force = 1;                  // the matrix-core path has no FP64 sweeps
        // inverse: blocks of at most 256 degrees, of equal size
        const int nb = (L + INV_BLK - 1) / INV_BLK, nq = (L + 7) / 8;
        P->inv.cb = (nq + nb - 1) / nb;
        P->inv.tiles = std::max(1, (P->nsw + 63) / 64);
        P->inv.rp = P->inv.tiles * 64;
        std::vector<int> orders;
        for (int q = 0; q < nq; q += P->inv.cb) orders.push_back(std::min(L, 8 * (q + P->inv.cb)));
        deal_work(P->inv, orders, nrun, P->ncu, force);
        stg.i.emplace_back(); std::vector<int> &mt = stg.i.back();
        for (int o : orders) mt.push_back(o - 1);
        if ((rc = upload(P, &P->mtop, mt, st, "inverse mtop"))) return bail(rc);
        // forward: groups of 64 degrees (mirror-ring sweep: of one parity), ring blocks of
        // equal size
        P->fwd.tiles = std::max(1, (P->nsw + FWD_BLK - 1) / FWD_BLK);
        P->fwd.nk = std::max(1, (P->nsw + P->fwd.tiles * 4 * SW_WAVES - 1) / (P->fwd.tiles * 4 * SW_WAVES));
        const int slots = P->fwd.tiles * 4 * SW_WAVES * P->fwd.nk;
        P->fwd.rp = (P->nsw + 3) / 4 * 4;
        P->hstride = std::max(P->nring, P->fwd_pair ? 0 : slots);
        if (P->fwd_pair) P->pstride = slots;
        orders.clear();
        const int ng = P->fwd_pair ? 2 * ((L + 127) / 128) : (L + 63) / 64;
        for (int g = 0; g < ng; ++g) {
            const int lmin = P->fwd_pair ? 128 * (g >> 1) + (g & 1) : 64 * g;
            orders.push_back(lmin < L ? std::min(L, lmin + (P->fwd_pair ? 127 : 64)) : 0);
        }
        deal_work(P->fwd, orders, nrun, P->ncu, force);
        P->order_tiles = P->inv.pieces;
    }

    std::vector<SweepRun> &sr = stg.sr;
    for (size_t ri = 0; ri < P->runs.size(); ++ri) {
        const Run &r = P->runs[ri];
        double2 *ini;
        if ((rc = P->dalloc(&ini, (size_t)L * P->nreg, "start values"))) return bail(rc);
        PLANCHK(launch_init_table(st, L, P->nreg, r.n, P->lsin, P->lcos, P->lbin[ri], ini), "start values");
        P->init.push_back(ini);
        sr.push_back(SweepRun{r.n, r.sliceA, r.sliceB, 0, ini, nullptr, nullptr});
    }
    // the work tables and, per run, the recursion state at each cut
    const int *cf_d[2] = {};
    const int2 *cu_d[2] = {};
    for (int f = 0; f < 2 && prec == S2_FP64; ++f) {
        Work &W = f ? P->fwd : P->inv;
        const int D = f ? FWD_L : 8 * W.cb;
        // pieces, cuts, slots and first cuts in one upload
        stg.i.emplace_back();
        std::vector<int> &tab = stg.i.back();
        for (const int4 &g : W.seg) tab.insert(tab.end(), {g.x, g.y, g.z, g.w});
        for (const int2 &c : W.cuts) tab.insert(tab.end(), {c.x, c.y});
        tab.insert(tab.end(), W.first.begin(), W.first.end());
        tab.insert(tab.end(), W.cfirst.begin(), W.cfirst.end());
        int *tab_d;
        if ((rc = upload(P, &tab_d, tab, st, "work of the sweeps"))) return bail(rc);
        W.seg_d = reinterpret_cast<int4 *>(tab_d);
        cu_d[f] = reinterpret_cast<const int2 *>(tab_d + 4 * W.seg.size());
        W.first_d = tab_d + 4 * W.seg.size() + 2 * W.cuts.size();
        cf_d[f] = W.first_d + W.first.size();
        if (W.cuts.empty()) continue;
        for (SweepRun &s : sr) {
            double *ck;
            if ((rc = P->dalloc(&ck, W.cuts.size() * D * 3 * (size_t)W.rp, "recursion states"))) return bail(rc);
            (f ? s.ckF : s.ckI) = ck;
        }
    }
    if ((rc = upload(P, &P->runs_d, sr, st, "runs"))) return bail(rc);
    for (int f = 0; f < 2 && prec == S2_FP64; ++f) {
        const Work &W = f ? P->fwd : P->inv;
        if (!W.cuts.empty())
            PLANCHK(launch_cut_state(st, f == 1, L, P->nsw, W.rp, f ? FWD_L : 8 * W.cb, W.nblk, P->fwd_pair, nrun,
                                     P->runs_d, P->cot, P->csc, P->kap, cf_d[f], cu_d[f]),
                    "recursion states");
    }

    // S2MI_DEBUG_CHECKS=1: check sum_{|m| <= l} (d^l_{m,n})^2 = 1 (d^l is orthogonal) on
    // sampled rings, for every degree and every run whose partner -n is in the plan,
    // with the same start values, tables and stable-direction continuation as the
    // sweeps; a violation fails the plan (S2_ERR_CHECK).  S2MI_DEBUG_CHECKS_TOL sets
    // the tolerance on |sum - 1| (default 1e-10).
    if (const char *dc = std::getenv("S2MI_DEBUG_CHECKS"); dc && dc[0] == '1' && P->nreg > 0) {
        const int nreg = P->nreg;
        std::vector<int> rs = {0, 1, nreg / 8, nreg / 4, nreg / 2, (3 * nreg) / 4, nreg - 2, nreg - 1};
        std::sort(rs.begin(), rs.end());
        rs.erase(std::unique(rs.begin(), rs.end()), rs.end());
        rs.erase(std::remove_if(rs.begin(), rs.end(), [&](int r) { return r < 0 || r >= nreg; }), rs.end());
        const int nsel = (int)rs.size();
        double tol = 1e-10;
        if (const char *tv = std::getenv("S2MI_DEBUG_CHECKS_TOL")) tol = std::atof(tv);
        int *rsel = nullptr;
        double *sums = nullptr;
        if ((rc = upload(P, &rsel, rs, st, "check rings"))) return bail(rc);
        const size_t per_run = (size_t)nsel * L * 2;
        if ((rc = P->dalloc(&sums, per_run * P->runs.size(), "check sums"))) return bail(rc);
        for (size_t ri = 0; ri < P->runs.size(); ++ri)
            PLANCHK(launch_unitarity(st, L, P->runs[ri].n, nsel, rsel, P->cot, P->csc, P->lsin, P->lcos, P->lbin[ri],
                                     P->kap, P->gtab, sums + ri * per_run),
                    "unitarity check");
        std::vector<double> h(per_run * P->runs.size());
        PLANCHK(hipMemcpyAsync(h.data(), sums, h.size() * sizeof(double), hipMemcpyDeviceToHost, st), "check copy");
        PLANCHK(hipStreamSynchronize(st), "check sync");
        for (size_t ri = 0; ri < P->runs.size(); ++ri) {
            const int n = P->runs[ri].n, an = n < 0 ? -n : n;
            int rj = -1;
            for (size_t k = 0; k < P->runs.size(); ++k)
                if (P->runs[k].n == -n) rj = (int)k;
            if (rj < 0) continue;
            const double *a = h.data() + ri * per_run, *b = h.data() + rj * per_run;
            for (int i = 0; i < nsel; ++i)
                for (int l = an; l < L; ++l) {
                    const size_t o = ((size_t)i * L + l) * 2;
                    // m >= 0 from run n, m < 0 from run -n at -m > 0
                    const double sum = a[o] + b[o] - b[o + 1] * b[o + 1];
                    if (!(std::fabs(sum - 1.0) <= tol))
                        return bail(fail(S2_ERR_CHECK,
                                         "debug check: sum over |m| <= l of d^l_{m,n}(theta)^2 = %.17g at l = %d, "
                                         "n = %d, ring %d (tolerance %g)", sum, l, n, rs[i], tol));
                }
        }
    }

    // workspace layout
    {
        const size_t S = P->nslice;
        const size_t nq = (L + 7) / 8;
        P->szC = align256((nq * P->nx + 4 * nq * (nq + 1)) * (P->one ? 24 : 40) * sizeof(double));
        P->szP = (size_t)P->inv.nblk * P->nreg * L * 4 * sizeof(double);
        // (the forward sweep's operand loads run up to 28 rings past a row's end)
        P->szF = ((size_t)L * P->hstride + 32) * 4 * sizeof(double);
        // forward partials [blk][l][m][4]; the adjoint of the MW / MWSS forward reuses the
        // buffer for ring partials [nring][m][4] (nring = L + 1 for MWSS)
        const int adj_rows = (sampling == S2_MW || sampling == S2_MWSS) ? P->nring : 0;
        P->szQ = std::max((size_t)P->fwd.tiles * L, (size_t)adj_rows) * L * 4 * sizeof(double);
        size_t o = 0;
        P->off_C = o; o += P->szC * P->runs.size();
        P->off_P = o; o += align256(P->szP * S);
        P->off_maps = o; o += (sampling == S2_MW && spin == 0) ? align256((size_t)P->nsamp * S * sizeof(double2)) : 0;
        P->off_F = o; o += align256(P->szF * S);
        P->off_Q = o; o += align256(P->szQ * S);
        P->off_hpole = o; o += align256((size_t)(2 * L - 1) * S * 2 * sizeof(double2));   // south, north
        // low-order machinery of runs with n != 0: masked spectra copies per run, continuation sums per slice
        P->szHx = ((size_t)std::max(P->nxp, 1) * P->hstride + 32) * 4 * sizeof(double);
        P->szQx = (size_t)P->fwd.tiles * L * std::max(P->nxp, 1) * 4 * sizeof(double);
        P->off_Hx = o; o += P->nxp > 0 ? align256(2 * P->szHx * P->runs.size()) : 0;
        P->off_Qx = o; o += P->nxp > 0 ? align256(P->szQx * S) : 0;
        P->off_hsym = o; o += (spin == 0 && !so3) ? align256((size_t)L * (2 * L - 1) * sizeof(double2)) : 0;
        P->off_Fp = o; o += P->fwd_pair ? align256((2 * (size_t)L * P->pstride + 32) * 4 * sizeof(double)) : 0;
        P->ws1 = o;
        // Maps of a batch that share the launches: enough to give every compute unit about
        // GROUP_ORDERS orders of work (fixed costs are then a few per cent), within
        // GROUP_BYTES of workspace.
        if (prec == S2_FP64) {
            long long ord = 0;
            for (const int4 &g : P->inv.seg) ord += g.y - g.z + 1;
            const double per = (double)ord * P->inv.tiles * P->runs.size() / P->ncu;
            const double want = std::ceil(GROUP_ORDERS / std::max(per, 1e-3));
            P->group = (int)std::max(1.0, std::min({(double)max_batch, want, std::floor((double)GROUP_BYTES / (double)o),
                                                               32768.0 / (double)std::max(S, P->runs.size())}));
            // S2MI_MAP_GROUP=k: at most k maps (a smaller workspace; tests)
            if (const char *mg = std::getenv("S2MI_MAP_GROUP")) {
                const int k = std::atoi(mg);
                if (k > 0) P->group = std::min(P->group, k);
            }
        }
        o *= P->group;
        bool split = false;
        for (const FftArgs &f : P->ffts_h) split = split || (f.blue && f.split && !f.perm);
        // one FFT_SCRATCH slice per workgroup of the phi-DFT (hstride), inverse phi-DFT
        // (nring) and MW filter (L) launches of one item (items then run one by one)
        P->sz_fscr = split ? (size_t)std::max({P->hstride, P->nring, L + 16}) * FFT_SCRATCH * sizeof(double2) : 0;
        P->off_fscr = o; o += align256(P->sz_fscr);
        P->ws_bytes = o;
    }

    {
        stg.i.emplace_back(1, L - 1);
        if ((rc = upload(P, &P->mtop1, stg.i.back(), st, "single-block mtop"))) return bail(rc);
    }
    // HEALPix forward = q x adjoint of the inverse, so its adjoint is the inverse with weights q w_l;
    // DH / GL: the inverse with weights w_l, then each ring scaled by its quadrature weight
    if (sampling != S2_MW && sampling != S2_MWSS && !so3) {
        stg.d.emplace_back();
        host_weights(L, 0, spin, &stg.d.back());
        if (sampling == S2_HEALPIX)
            for (double &v : stg.d.back()) v *= 4.0 * M_PI / (double)P->nsamp;
        double *a;
        if ((rc = upload(P, &a, stg.d.back(), st, "forward-adjoint weights"))) return bail(rc);
        P->w_fadj = a;
    }

    // matrix-core path: generator assignment, {kappa, g} table, batched workspace
    if (prec != S2_FP64) {
        P->mfma = true;
        MfmaGeom &g = P->mg;
        g.L = L;
        g.nreg = P->nreg;
        g.rpad = (P->nreg + 63) / 64 * 64;
        g.lp = (L + 63) / 64 * 64;
        g.kc = (L + 7) / 8;
        g.lrow = 8 * g.kc;
        g.rows = (4 * max_batch + 31) / 32 * 32;
        {
            const int nch = g.kc;
            // a wave per chunk of 8 degrees, the longest (largest degrees) first
            P->gen_nblk = (nch + DSTAGE_MAX_WAVES - 1) / DSTAGE_MAX_WAVES;
            P->gen_waves = (nch + P->gen_nblk - 1) / P->gen_nblk;
            const int nslot = P->gen_nblk * P->gen_waves;
            stg.i.emplace_back(nslot, -1);
            for (int k = 0; k < nch; ++k) stg.i.back()[k] = 8 * (nch - 1 - k);
            if ((rc = upload(P, &P->gen_lchunk, stg.i.back(), st, "generator chunks"))) return bail(rc);
            P->nslots = (size_t)nslot * 8;
        }
        if ((rc = P->dalloc(&P->kg, (size_t)(L + P->nx) * g.lrow, "kappa/g table"))) return bail(rc);
        P->kg += (size_t)P->nx * g.lrow;                     // rows m in [-nx, L)
        PLANCHK(launch_kg_table(st, L, P->nx, g.lrow, P->kap, P->gtab, P->kg), "kappa/g table");
        const size_t per_m_d = std::max((size_t)g.kc * g.rpad, (size_t)(g.rpad / 8) * g.lp) * 32;
        // up to 4 GiB of staged D (256 orders at L = 2048): larger chunks mean fewer, larger
        // generator and product launches (64 maps at L = 2048, FP32 pair: 32 orders per
        // chunk 145 ms, 64: 130 ms, 128: 123 ms, 256: 119 ms; split BF16 115 -> 101 ms)
        P->mch = (int)std::max<size_t>(4, std::min<size_t>((size_t)L, ((size_t)4 << 30) / per_m_d));
        // S2MI_MFMA_ORDER_CHUNK=k stages k orders of D per generator launch instead (tests: the
        // recursion state carried across order chunks at small L; results do not depend on it)
        if (const char *mc = std::getenv("S2MI_MFMA_ORDER_CHUNK")) {
            const int k = std::atoi(mc);
            if (k > 0) P->mch = std::min(L, k);
        }
        const size_t per_m_ah = (size_t)std::max(g.kc, g.rpad / 8) * g.rows * 32;
        const size_t S = P->nslice, B = max_batch;
        const size_t nP1 = (size_t)P->nreg * L * 4, nQ1 = (size_t)L * L * 4;
        P->state_bytes = P->nslots * g.rpad * (2 * sizeof(double) + sizeof(int));
        size_t o = P->ws_bytes;
        P->off_D = o; o += align256(per_m_d * P->mch);
        P->off_S = o; o += align256(P->state_bytes);
        P->off_AH = o; o += align256(per_m_ah * P->mch);
        P->off_mP = o; o += align256(B * S * nP1 * sizeof(double));
        P->off_mF = o; o += align256(B * S * P->szF);
        P->off_mQ = o; o += align256(B * S * nQ1 * sizeof(double));
        P->off_mhp = o; o += align256(B * S * (2 * L - 1) * 2 * sizeof(double2));        // [south, north][b][slice]
        P->off_mmaps = o; o += (S > 1) ? align256(B * S * (size_t)P->nsamp * sizeof(double2)) : 0;
        P->off_mQx = o; o += P->nxp > 0 ? align256(B * S * (size_t)L * P->nxp * 4 * sizeof(double)) : 0;
        P->ws_bytes = o;
    }
    PLANCHK(hipStreamSynchronize(st), "plan upload");
    PLANCHK(hipGetLastError(), "plan kernels");
    *out = P;
    return S2_OK;
}
#undef PLANCHK

int s2_plan_create(s2_plan_t *out, int L, int spin, int N, s2_sampling_t sampling, int nside, int max_batch,
                   s2_precision_t prec, void *hip_stream)
{
    try {
        return plan_create_impl(out, L, spin, N, sampling, nside, max_batch, prec, hip_stream);
    } catch (const std::bad_alloc &) {
        return fail(S2_ERR_OOM, "host allocation failed during plan creation");
    } catch (...) {
        return fail(S2_ERR_HIP, "unexpected exception during plan creation");
    }
}

}  // extern "C"

// ------------------------------------------------------------------ transforms
namespace {

// Bracket one launch with events when the plan records stage timing.
// Set for the duration of a call that must not allocate (s2_inverse_noalloc):
// event creation and the timing record are skipped.
thread_local bool g_no_timing = false;

struct StageTimer {
    s2_plan_t P;
    int stage;
    hipStream_t st;
    hipEvent_t a = nullptr, b = nullptr;
    StageTimer(s2_plan_t P_, int stage_, hipStream_t st_) : P(P_), stage(stage_), st(st_)
    {
        if (P->timing && !g_no_timing && hipEventCreate(&a) == hipSuccess && hipEventCreate(&b) == hipSuccess)
            (void)hipEventRecord(a, st);
    }
    ~StageTimer()
    {
        if (a && b) {
            (void)hipEventRecord(b, st);
            P->tl.push_back({stage, a, b});
        }
    }
};
#define S2_CAT2(a, b) a##b
#define S2_CAT(a, b) S2_CAT2(a, b)
#define TIMED(stage) StageTimer S2_CAT(_timer_, __LINE__)(P, stage, st)

int check_call(const char *fn, s2_plan_t P, const void *in, const void *out, int batch, void *ws)
{
    if (!P) return fail(S2_ERR_INVALID_ARG, "%s: plan is NULL", fn);
    if (batch == 0) return S2_OK;                 // an empty batch: nothing is read or written
    if (!in || !out) return fail(S2_ERR_INVALID_ARG, "%s: NULL data pointer", fn);
    if (!ws) return fail(S2_ERR_INVALID_ARG, "%s: NULL workspace", fn);
    if (((uintptr_t)in | (uintptr_t)out) & 15) return fail(S2_ERR_INVALID_ARG, "%s: data pointers must be 16-byte aligned", fn);
    if ((uintptr_t)ws & 255) return fail(S2_ERR_INVALID_ARG, "%s: workspace must be 256-byte aligned", fn);
    if (batch < 0 || batch > P->max_batch)
        return fail(S2_ERR_INVALID_ARG, "%s: batch=%d outside [0, max_batch=%d]", fn, batch, P->max_batch);
    return S2_OK;
}

// the workspace's split-Bluestein scratch (nullptr when no DFT of the plan needs it)
double2 *fft_scratch(const s2_plan_s *P, char *ws)
{
    return P->sz_fscr ? reinterpret_cast<double2 *>(ws + P->off_fscr) : nullptr;
}

Items all_slices(const s2_plan_s *P) { return Items{P->nslice, 0, P->spin_d}; }
// strides of the workspace's per-map buffers (doubles), of coefficients and of maps
long long wsd(const s2_plan_s *P) { return (long long)(P->ws1 / sizeof(double)); }
long long coef_n(const s2_plan_s *P) { return (long long)P->L * (2 * P->L - 1); }
Strides coef_strides(const s2_plan_s *P) { return Strides{P->nslice * coef_n(P), coef_n(P)}; }
// complex entries between the slice maps of consecutive maps in the workspace
long long tmp_stride(const s2_plan_s *P) { return (long long)(P->ws1 / sizeof(double2)); }
Strides map_strides(const s2_plan_s *P) { return Strides{P->nslice * P->nsamp, P->nsamp}; }
Strides ws_strides(const s2_plan_s *P, size_t slice_bytes)
{
    return Strides{wsd(P), (long long)(slice_bytes / sizeof(double))};
}
// pole lines: [south, north][slice][2L-1] complex per map
Strides pole_strides(const s2_plan_s *P) { return Strides{(long long)(P->ws1 / sizeof(double2)), 2 * P->L - 1}; }

// inverse d-stage of nm maps, all slices: flm [nm][S][L][2L-1] (fstride per map) ->
// partials P[map][slice][blk][ring][m][4]  (half: real signal of a spin-0 plan, orders
// m >= 0 and components 0,1 only)
int run_inverse_dstage(s2_plan_t P, const double2 *flm, long long fstride, int nm, const double *wl, char *ws,
                       hipStream_t st, int half = 0)
{
    InvArgs a{};
    a.L = P->L; a.nx = P->nx; a.nreg = P->nreg; a.nsw = P->nsw; a.nrun = (int)P->runs.size(); a.half = half;
    a.rt = P->inv.tiles; a.nslot = P->inv.nslot; a.cb = P->inv.cb; a.rp = P->inv.rp;
    a.merge = merge_slots(P->inv, (long long)nm * a.nrun, P->ncu);
    a.wsd = wsd(P); a.nC = (long long)(P->szC / sizeof(double)); a.nP = (long long)(P->szP / sizeof(double));
    a.runs = P->runs_d; a.seg = P->inv.seg_d; a.first = P->inv.first_d;
    a.C = (double *)(ws + P->off_C); a.P = (double *)(ws + P->off_P);
    const bool one = P->one || half;
    {
        TIMED(S2_STAGE_PACK);
        HIPCHK(launch_pack_inv(st, a, nm, one, flm, fstride, wl, P->kap, P->gtab), "pack");
    }
    if (P->nreg < 1) return S2_OK;
    TIMED(S2_STAGE_DSTAGE_INV);
    HIPCHK(launch_sweep_inv(st, a, nm, one, P->cot, P->csc), "inverse d-stage");
    return S2_OK;
}

// inverse of nm maps, all slices: flm -> slice maps [nm][S][nsamp] (strides sm)
// (tight: one map on a workspace of inverse_extent bytes, the DFT scratch right behind
// its partial sums)
int run_inverse(s2_plan_t P, const double2 *flm, double2 *maps, Strides sm, int nm, const double *wl, char *ws,
                hipStream_t st, bool tight = false)
{
    const Strides sf = coef_strides(P);
    int rc = run_inverse_dstage(P, flm, sf.map, nm, wl, ws, st);
    if (rc) return rc;
    TIMED(S2_STAGE_PHI_INV);
    HIPCHK(launch_phi_inv(st, P->dft, P->nring, P->L, P->nreg, P->inv.nblk, all_slices(P),
                          nm * P->nslice, ws_strides(P, P->szP), sf, sm, (const double *)(ws + P->off_P), P->mtop, flm,
                          wl, P->ring_nphi, P->ring_start, P->ring_shift, P->ring_fft, P->ffts, maps,
                          tight && P->sz_fscr ? (double2 *)(ws + align256(P->off_P + P->szP * P->nslice))
                                              : fft_scratch(P, ws)),
           "inverse phi-DFT");
    return S2_OK;
}

// the theta filter (adj: its adjoint) of nm maps in place on F, or the pole lines alone
int run_theta(s2_plan_t P, int nm, char *ws, hipStream_t st, int half, int adj)
{
    const int L = P->L, ss = P->sampling == S2_MWSS;
    double2 *hp = (double2 *)(ws + P->off_hpole);
    double2 *hpN = ss ? hp + (size_t)P->nslice * (2 * L - 1) : nullptr;
    HIPCHK(launch_mw_filter(st, P->dft, L, ss, P->hstride, all_slices(P), nm * P->nslice,
                            ws_strides(P, P->szF), pole_strides(P), P->ffts, P->wq, P->ph, (double *)(ws + P->off_F), hp,
                            hpN, fft_scratch(P, ws), half, adj), "MW theta filter");
    return S2_OK;
}

int run_pole_lines(s2_plan_t P, int nm, char *ws, hipStream_t st)
{
    const int L = P->L;
    double2 *hp = (double2 *)(ws + P->off_hpole);
    const double *F = (const double *)(ws + P->off_F);
    HIPCHK(launch_pole_from_F(st, L, P->hstride, L - 1, all_slices(P), nm * P->nslice, ws_strides(P, P->szF),
                              pole_strides(P), F, hp), "pole line");
    if (P->sampling == S2_MWSS)
        HIPCHK(launch_pole_from_F(st, L, P->hstride, L, all_slices(P), nm * P->nslice, ws_strides(P, P->szF),
                                  pole_strides(P), F, hp + (size_t)P->nslice * (2 * L - 1)), "north pole line");
    return S2_OK;
}

// the partials of an adjoint's inverse-type sweep through the theta filter's adjoint,
// into the ring partials Q[map][slice][ring][m][4] of the phi-DFT
int run_theta_adjoint(s2_plan_t P, const double2 *G, Strides sf, int nm, const double *wl, char *ws, hipStream_t st,
                      int half)
{
    const int L = P->L, ss = P->sampling == S2_MWSS;
    double *F = (double *)(ws + P->off_F), *Q = (double *)(ws + P->off_Q);
    double2 *hp = (double2 *)(ws + P->off_hpole);
    double2 *hpN = ss ? hp + (size_t)P->nslice * (2 * L - 1) : nullptr;
    const double q = 2.0 * M_PI / (double)(ss ? 2 * L : 2 * L - 1);
    TIMED(S2_STAGE_MW_THETA);
    HIPCHK(launch_fadj_gather(st, L, ss, P->inv.nblk, all_slices(P), nm * P->nslice, ws_strides(P, P->szP), sf,
                              ws_strides(P, P->szF), (const double *)(ws + P->off_P), P->mtop, G, wl, P->hstride, F),
           "adjoint gather");
    int rc = run_theta(P, nm, ws, st, half, 1);
    if (rc) return rc;
    HIPCHK(launch_fadj_scatter(st, L, ss, P->hstride, q, all_slices(P), nm * P->nslice, ws_strides(P, P->szF),
                               pole_strides(P), ws_strides(P, P->szQ), F, hp, hpN, Q), "adjoint scatter");
    return S2_OK;
}

// adjoint of the MW / MWSS forward of nm maps, all slices (finish weights wl, spin
// slice_spin[k]): coefficient cotangents -> slice maps.  MWSS adds the north-pole row
// and runs the adjoint form of its theta filter.
int run_forward_adjoint_mw(s2_plan_t P, const double2 *G, double2 *maps, Strides sm, int nm, const double *wl, char *ws,
                           hipStream_t st)
{
    const Strides sf = coef_strides(P);
    int rc = run_inverse_dstage(P, G, sf.map, nm, wl, ws, st);
    if (rc || (rc = run_theta_adjoint(P, G, sf, nm, wl, ws, st, 0))) return rc;
    TIMED(S2_STAGE_PHI_INV);
    HIPCHK(launch_phi_inv(st, P->dft, P->nring, P->L, P->nring, 1, all_slices(P), nm * P->nslice,
                          ws_strides(P, P->szQ), sf, sm, (const double *)(ws + P->off_Q), P->mtop1, G, wl, P->ring_nphi,
                          P->ring_start, P->ring_shift, P->ring_fft, P->ffts, maps, fft_scratch(P, ws)),
           "adjoint phi-DFT");
    return S2_OK;
}

// forward d-stage of nm maps from the (filtered) ring spectra F -> flm
int run_forward_dstage(s2_plan_t P, bool poles, double2 *flm, int nm, const double *wl, char *ws, hipStream_t st,
                       int half = 0)
{
    const int L = P->L;
    FwdArgs a{};
    a.L = L; a.nxp = std::max(P->nxp, 1); a.nx = P->nx; a.nreg = P->nsw; a.hstride = P->fwd_pair ? P->pstride : P->hstride;
    a.nrun = (int)P->runs.size(); a.half = half ? 1 : 0;
    a.rb = P->fwd.tiles; a.nk = P->fwd.nk; a.nslot = P->fwd.nslot; a.rp = P->fwd.rp;
    a.merge = merge_slots(P->fwd, (long long)nm * a.nrun, P->ncu);
    a.wsd = wsd(P);
    a.nF = (long long)(P->szF / sizeof(double)); a.nQ = (long long)(P->szQ / sizeof(double));
    a.nHx = (long long)(P->szHx / sizeof(double)); a.nQx = (long long)(P->szQx / sizeof(double));
    a.runs = P->runs_d; a.seg = P->fwd.seg_d; a.first = P->fwd.first_d;
    a.F = (const double *)(ws + P->off_F);
    a.Q = (double *)(ws + P->off_Q);
    double *Hx = P->nxp > 0 ? (double *)(ws + P->off_Hx) : nullptr;
    a.Hx = Hx;
    a.Qx = P->nxp > 0 ? (double *)(ws + P->off_Qx) : nullptr;
    const bool one = P->one || half;
    {
        TIMED(S2_STAGE_DSTAGE_FWD);
        if (P->fwd_pair) {
            // spin-0 S2 plan (one slice, run n = 0): sweep the northern rings on the sums and
            // differences of each ring's and its mirror's spectra
            double *S = (double *)(ws + P->off_Fp), *D = S + (size_t)L * P->pstride * 4;
            HIPCHK(launch_pair_spectra(st, nm, a.wsd, L, P->nreg, P->nsw, P->hstride, P->pstride, a.F, S, D),
                   "mirror spectra");
            a.S = S;
            a.D = D;
        } else if (P->nxp > 0) {
            HIPCHK(launch_mask_low(st, nm, a.nrun, P->runs_d, P->nxp, P->nreg, P->hstride, P->cot, P->csc, a.F, Hx,
                                   a.wsd, a.nF, a.nHx, a.Qx, (long long)(P->szQx * P->nslice / sizeof(double))),
                   "low-order spectra, continuation sums clear");
        }
        HIPCHK(launch_sweep_fwd(st, a, nm, one, P->cot, P->csc, P->kap), "forward d-stage");
    }
    TIMED(S2_STAGE_FINISH);
    const double2 *hp = poles ? (const double2 *)(ws + P->off_hpole) : nullptr;
    const double2 *hpN = poles && P->sampling == S2_MWSS ? hp + (size_t)P->nslice * (2 * L - 1) : nullptr;
    HIPCHK(launch_finish_fwd(st, L, P->fwd.tiles, all_slices(P), nm * P->nslice, ws_strides(P, P->szQ),
                             ws_strides(P, P->szQx), pole_strides(P), coef_strides(P), P->gtab, a.Q, a.Qx, a.nxp, wl, hp,
                             hpN, flm, half),
           "forward finish");
    return S2_OK;
}

// phi weight of the forward (adjoint: unit)
double phi_weight(const s2_plan_s *P, bool adjoint)
{
    if (adjoint) return 1.0;
    if (P->sampling == S2_MW) return 2.0 * M_PI / (double)(2 * P->L - 1);
    if (P->sampling == S2_MWSS) return 2.0 * M_PI / (double)(2 * P->L);
    return 4.0 * M_PI / (double)P->nsamp;                 // HEALPix (DH / GL: per-ring weights)
}

// forward of nm maps: slice maps (strides sm) -> flm.  adjoint: unit phi weight, no theta filter.
int run_forward(s2_plan_t P, const double2 *maps, Strides sm, double2 *flm, int nm, const double *wl, char *ws,
                hipStream_t st, bool adjoint)
{
    const bool mw = P->sampling == S2_MW || P->sampling == S2_MWSS;   // theta-torus samplings
    {
        TIMED(S2_STAGE_PHI_FWD);
        HIPCHK(launch_phi_fwd(st, P->dft, P->nring, P->hstride, P->L, phi_weight(P, adjoint),
                              all_slices(P), nm * P->nslice, sm, ws_strides(P, P->szF), maps, P->ring_nphi,
                              P->ring_start, P->ring_shift, P->ring_fft, P->ffts, adjoint ? nullptr : P->ringq,
                              (double *)(ws + P->off_F), fft_scratch(P, ws)), "forward phi-DFT");
    }
    if (mw) {
        TIMED(S2_STAGE_MW_THETA);
        int rc = adjoint ? run_pole_lines(P, nm, ws, st) : run_theta(P, nm, ws, st, 0, 0);
        if (rc) return rc;
    }
    return run_forward_dstage(P, mw, flm, nm, wl, ws, st);
}

// Real signals (spin-0 S2 plan, Hermitian symmetry of the coefficients): the
// sweeps carry the orders m >= 0 only and pairs of rings share a phi-DFT.
int run_inverse_real(s2_plan_t P, const double2 *flm, long long fstride, double *map, int nm, const double *wl,
                     char *ws, hipStream_t st)
{
    int rc = run_inverse_dstage(P, flm, fstride, nm, wl, ws, st, 1);
    if (rc) return rc;
    TIMED(S2_STAGE_PHI_INV);
    HIPCHK(launch_phi_inv_real(st, P->dft, P->npair, P->L, P->nreg, P->inv.nblk, nm, wsd(P),
                               fstride, P->nsamp, P->ring_pairs, (const double *)(ws + P->off_P), P->mtop, flm, wl,
                               P->ring_nphi, P->ring_start, P->ring_shift, P->ring_fft, P->ffts, map,
                               fft_scratch(P, ws)), "real inverse phi-DFT");
    return S2_OK;
}

// vjp: the gradient of run_inverse_real with respect to its complex input for a
// real map cotangent: 2 A^H g at m > 0 and Re (A^H g) at m = 0 (A the complex
// inverse), i.e. the unnormalised phi-DFT, no theta filter, the forward-type
// sweep with the SHT weights, and the finish in its gradient mode.
int run_forward_real(s2_plan_t P, const double *map, double2 *flm, int nm, char *ws, hipStream_t st, bool vjp = false)
{
    const bool mw = P->sampling == S2_MW || P->sampling == S2_MWSS;   // theta-torus samplings
    {
        TIMED(S2_STAGE_PHI_FWD);
        HIPCHK(launch_phi_fwd_real(st, P->dft, P->nring, P->hstride, P->npair, P->L,
                                   phi_weight(P, vjp), nm, P->nsamp, wsd(P), P->ring_pairs, map, P->ring_nphi,
                                   P->ring_start, P->ring_shift, P->ring_fft, P->ffts, vjp ? nullptr : P->ringq,
                                   (double *)(ws + P->off_F), fft_scratch(P, ws)), "real forward phi-DFT");
    }
    if (mw) {
        TIMED(S2_STAGE_MW_THETA);
        int rc = vjp ? run_pole_lines(P, nm, ws, st) : run_theta(P, nm, ws, st, 1, 0);
        if (rc) return rc;
    }
    return run_forward_dstage(P, mw, flm, nm, P->w_sht, ws, st, vjp ? 2 : 1);
}

// The adjoint of the forward transform restricted to real maps: Re(F^H G) =
// F^H h with h the Hermitian part of G, so the real-signal machinery applies:
// MW / MWSS as the complex adjoint (gather, adjoint theta filter on one side,
// scatter) ending in the paired real phi-DFT; DH / GL / HEALPix the real
// inverse with the forward-adjoint weights, then the ring weights (DH / GL).
int run_forward_real_adjoint(s2_plan_t P, const double2 *G, double *map, int nm, char *ws, hipStream_t st)
{
    double2 *H = (double2 *)(ws + P->off_hsym);
    const long long hs = (long long)(P->ws1 / sizeof(double2));
    HIPCHK(launch_hermitian_part(st, nm, coef_n(P), hs, P->L, G, H), "Hermitian part");
    int rc;
    if (P->sampling != S2_MW && P->sampling != S2_MWSS) {
        if ((rc = run_inverse_real(P, H, hs, map, nm, P->w_fadj, ws, st))) return rc;
        if (P->ringq)
            HIPCHK(launch_ring_scale_real(st, nm, P->nsamp, P->nring, P->ring_start, P->ring_nphi, P->ringq, map),
                   "ring weights");
        return S2_OK;
    }
    // side B of the gathered rows is not produced by the half sweep and is never read
    if ((rc = run_inverse_dstage(P, H, hs, nm, P->w_sht, ws, st, 1))) return rc;
    if ((rc = run_theta_adjoint(P, H, Strides{hs, 0}, nm, P->w_sht, ws, st, 1))) return rc;
    TIMED(S2_STAGE_PHI_INV);
    HIPCHK(launch_phi_inv_real(st, P->dft, P->npair, P->L, P->nring, 1, nm, wsd(P), hs, P->nsamp,
                               P->ring_pairs, (const double *)(ws + P->off_Q), P->mtop1, H, P->w_sht, P->ring_nphi,
                               P->ring_start, P->ring_shift, P->ring_fft, P->ffts, map, fft_scratch(P, ws)),
           "real adjoint phi-DFT");
    return S2_OK;
}

// maps [0, batch) in groups that share the launches: go(first map, maps of the group)
template <typename F>
int over_groups(int batch, int group, F go)
{
    for (int b = 0; b < batch; b += group) {
        const int rc = go(b, std::min(group, batch - b));
        if (rc) return rc;
    }
    return S2_OK;
}

// ---------------------------------------------------------------- matrix-core path
// Batched inverse: flm [B][S][L][2L-1] -> slice maps [B][S][nsamp].
int run_inverse_mfma(s2_plan_t P, const double2 *flm, int B, double2 *maps, const double *wl, char *ws,
                     hipStream_t st)
{
    const int L = P->L, S = P->nslice, fmt = P->prec;
    const MfmaGeom &g = P->mg;
    const size_t slab = (size_t)L * (2 * L - 1);
    const size_t nP1 = (size_t)P->nreg * L * 4;
    uint4 *D = (uint4 *)(ws + P->off_D);
    uint4 *A = (uint4 *)(ws + P->off_AH);
    double *SX = (double *)(ws + P->off_S);
    double *SY = SX + P->nslots * g.rpad;
    int *SE = (int *)(SY + P->nslots * g.rpad);
    double *Pm = (double *)(ws + P->off_mP);
    for (size_t ri = 0; ri < P->runs.size(); ++ri) {
        const Run &r = P->runs[ri];
        const double2 *fa = r.sliceA >= 0 ? flm + r.sliceA * slab : nullptr;
        const double2 *fb = r.sliceB >= 0 ? flm + r.sliceB * slab : nullptr;
        double *PA = r.sliceA >= 0 ? Pm + r.sliceA * nP1 : nullptr;
        double *PB = r.sliceB >= 0 ? Pm + r.sliceB * nP1 : nullptr;
        const int an = r.n < 0 ? -r.n : r.n;
        const int mend = an > 1 ? -(an - 1) : 0;          // continuation below m = 0
        HIPCHK(launch_zero(st, SX, P->state_bytes), "recursion state clear");
        for (int mhi = L - 1; mhi >= mend; mhi -= P->mch) {
            const int mlo = std::max(mend, mhi - P->mch + 1), mcn = mhi - mlo + 1;
            {
            TIMED(S2_STAGE_DGEN);
            HIPCHK(launch_dgen(st, 0, fmt, P->gen_waves, P->gen_nblk, g, r.n, mhi, mlo, P->cot, P->csc, P->init[ri],
                               P->kg, P->gen_lchunk, SX, SY, SE, D), "d-tile generator");
            }
            {
            TIMED(S2_STAGE_PACK);
            HIPCHK(launch_pack_a(st, fmt, g, r.n, mlo, mcn, B, (long long)(S * slab), fa, fb,
                                 r.sliceA >= 0 ? wl + (size_t)r.sliceA * L : nullptr,
                                 r.sliceB >= 0 ? wl + (size_t)r.sliceB * L : nullptr, A),
                   "coefficient pack");
            }
            TIMED(S2_STAGE_MFMA);
            HIPCHK(launch_mfma_inv(st, fmt, g, r.n, P->cot, P->csc, mlo, mcn, B, A, D, PA, PB, (long long)(S * nP1)),
                   "inverse contraction");
        }
    }
    TIMED(S2_STAGE_PHI_INV);
    HIPCHK(launch_phi_inv(st, P->dft, P->nring, L, P->nreg, 1, all_slices(P), B * S,
                          Strides{(long long)(S * nP1), (long long)nP1}, coef_strides(P), map_strides(P), Pm, P->mtop1, flm,
                          wl, P->ring_nphi, P->ring_start, P->ring_shift, P->ring_fft, P->ffts, maps,
                          fft_scratch(P, ws)), "inverse phi-DFT");
    return S2_OK;
}

// Batched forward (adjoint: unit phi weight, no theta filter): slice maps [B][S][nsamp] -> flm [B][S][L][2L-1].
int run_forward_mfma(s2_plan_t P, const double2 *maps, int B, double2 *flm, const double *wl, char *ws,
                     hipStream_t st, bool adjoint)
{
    const int L = P->L, S = P->nslice, fmt = P->prec;
    const MfmaGeom &g = P->mg;
    const size_t slab = (size_t)L * (2 * L - 1);
    const size_t nF = P->szF / sizeof(double), nQ1 = (size_t)L * L * 4;
    const bool mw = P->sampling == S2_MW || P->sampling == S2_MWSS;   // theta-torus samplings
    const int ss = P->sampling == S2_MWSS;
    uint4 *D = (uint4 *)(ws + P->off_D);
    uint4 *H = (uint4 *)(ws + P->off_AH);
    double *SX = (double *)(ws + P->off_S);
    double *SY = SX + P->nslots * g.rpad;
    int *SE = (int *)(SY + P->nslots * g.rpad);
    double *Fm = (double *)(ws + P->off_mF);
    double *Qm = (double *)(ws + P->off_mQ);
    double2 *hp = (double2 *)(ws + P->off_mhp);
    double2 *hpN = mw && ss ? hp + (size_t)B * S * (2 * L - 1) : nullptr;
    const int nxp1 = std::max(P->nxp, 1);
    const size_t nQx1 = (size_t)L * nxp1 * 4;
    double *Qxm = P->nxp > 0 ? (double *)(ws + P->off_mQx) : nullptr;
    if (Qxm) HIPCHK(launch_zero(st, Qxm, (size_t)B * S * nQx1 * sizeof(double)), "continuation sums clear");
    const Strides sF{(long long)(S * nF), (long long)nF}, sh{(long long)S * (2 * L - 1), 2 * L - 1};
    {
        TIMED(S2_STAGE_PHI_FWD);
        HIPCHK(launch_phi_fwd(st, P->dft, P->nring, P->hstride, L, phi_weight(P, adjoint),
                              all_slices(P), B * S, map_strides(P), sF, maps, P->ring_nphi, P->ring_start, P->ring_shift,
                              P->ring_fft, P->ffts, adjoint ? nullptr : P->ringq, Fm, fft_scratch(P, ws)),
               "forward phi-DFT");
    }
    if (mw) {
        TIMED(S2_STAGE_MW_THETA);
        if (!adjoint) {
            HIPCHK(launch_mw_filter(st, P->dft, L, ss, P->hstride, all_slices(P), B * S, sF, sh,
                                    P->ffts, P->wq, P->ph, Fm, hp, hpN, fft_scratch(P, ws), 0, 0),
                   "MW theta filter");
        } else {
            HIPCHK(launch_pole_from_F(st, L, P->hstride, L - 1, all_slices(P), B * S, sF, sh, Fm, hp), "pole line");
            if (ss)
                HIPCHK(launch_pole_from_F(st, L, P->hstride, L, all_slices(P), B * S, sF, sh, Fm, hpN),
                       "north pole line");
        }
    }
    for (size_t ri = 0; ri < P->runs.size(); ++ri) {
        const Run &r = P->runs[ri];
        const double *FA = r.sliceA >= 0 ? Fm + r.sliceA * nF : Fm + r.sliceB * nF;
        const double *FB = r.sliceB >= 0 ? Fm + r.sliceB * nF : FA;
        double *QA = r.sliceA >= 0 ? Qm + r.sliceA * nQ1 : nullptr;
        double *QB = r.sliceB >= 0 ? Qm + r.sliceB * nQ1 : nullptr;
        const int an = r.n < 0 ? -r.n : r.n;
        const int mend = an > 1 ? -(an - 1) : 0;          // continuation below m = 0
        double *QxA = (an > 0 && r.sliceA >= 0) ? Qxm + r.sliceA * nQx1 : nullptr;
        double *QxB = (an > 0 && r.sliceB >= 0) ? Qxm + r.sliceB * nQx1 : nullptr;
        HIPCHK(launch_zero(st, SX, P->state_bytes), "recursion state clear");
        for (int mhi = L - 1; mhi >= mend; mhi -= P->mch) {
            const int mlo = std::max(mend, mhi - P->mch + 1), mcn = mhi - mlo + 1;
            {
            TIMED(S2_STAGE_DGEN);
            HIPCHK(launch_dgen(st, 1, fmt, P->gen_waves, P->gen_nblk, g, r.n, mhi, mlo, P->cot, P->csc, P->init[ri],
                               P->kg, P->gen_lchunk, SX, SY, SE, D), "d-tile generator");
            }
            {
            TIMED(S2_STAGE_PACK);
            HIPCHK(launch_pack_h(st, fmt, g, P->hstride, r.n, P->cot, P->csc, mlo, mcn, B, (long long)(S * nF), FA, FB, H),
                   "spectra pack");
            }
            TIMED(S2_STAGE_MFMA);
            HIPCHK(launch_mfma_fwd(st, fmt, g, r.n, nxp1, mlo, mcn, B, H, D, QA, QB, (long long)(S * nQ1), QxA, QxB,
                                   (long long)(S * nQx1)), "forward contraction");
        }
    }
    TIMED(S2_STAGE_FINISH);
    HIPCHK(launch_finish_fwd(st, L, 1, all_slices(P), B * S, Strides{(long long)(S * nQ1), (long long)nQ1},
                             Strides{(long long)(S * nQx1), (long long)nQx1}, sh, coef_strides(P), nullptr, Qm, Qxm, nxp1,
                             wl, mw ? hp : nullptr, hpN, flm), "forward finish");
    return S2_OK;
}

}  // namespace

extern "C" {

int s2_inverse(s2_plan_t P, const void *flm, void *f, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_inverse", P, flm, f, batch, workspace);
    if (rc) return rc;
    if (P->N != 1) return fail(S2_ERR_INVALID_ARG, "s2_inverse: plan was created for SO(3) (N=%d)", P->N);
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    if (P->mfma) return run_inverse_mfma(P, (const double2 *)flm, batch, (double2 *)f, P->w_sht, (char *)workspace, st);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_inverse(P, (const double2 *)flm + b * slab, (double2 *)f + (size_t)b * P->nsamp, map_strides(P), nm,
                           P->w_sht, (char *)workspace, st);
    });
}

}  // extern "C"

// ------------------------------------------------------------------ no-allocation inverse
// The workspace of s2_inverse_noalloc: a fixed device array, one copy per GPU the
// library runs on, held until the process ends.  Host code never uses the name
// `scratch` as an address (on the host it is only a stand-in for the symbol): the
// device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[S2_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[SCRATCH_MAX_DEVICES] = {};   // per device index; nullptr until looked up

// device address of `scratch` on the current device (looked up on the first call there)
int scratch_on_current_device(void **out)
{
    int dev = 0;
    HIPCHK(hipGetDevice(&dev), "hipGetDevice");
    if (dev < 0 || dev >= SCRATCH_MAX_DEVICES)
        return fail(S2_ERR_UNSUPPORTED, "s2_inverse_noalloc: device index %d beyond %d", dev, SCRATCH_MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return S2_OK;
}

// bytes of the workspace the FP64 inverse touches (records, partials, and the
// split-Bluestein scratch when a ring DFT needs it)
size_t inverse_extent(const s2_plan_s *P)
{
    return P->off_P + P->szP * P->nslice + (P->sz_fscr ? 256 + P->sz_fscr : 0);
}

}  // namespace

extern "C" {

int s2_inverse_noalloc(s2_plan_t P, const void *flm, void *f, int batch, void *hip_stream)
{
    if (!P) return fail(S2_ERR_INVALID_ARG, "s2_inverse_noalloc: plan is NULL");
    if (P->N != 1) return fail(S2_ERR_INVALID_ARG, "s2_inverse_noalloc: plan was created for SO(3) (N=%d)", P->N);
    if (P->mfma) return fail(S2_ERR_UNSUPPORTED, "s2_inverse_noalloc: available for FP64 plans");
    const size_t need = inverse_extent(P);
    if (need > (size_t)S2_NOALLOC_SCRATCH_BYTES)
        return fail(S2_ERR_INVALID_ARG,
                    "s2_inverse_noalloc: this plan's inverse needs %zu bytes of scratch, more than the fixed %zu "
                    "(use s2_inverse with a workspace)", need, (size_t)S2_NOALLOC_SCRATCH_BYTES);
    void *ws = nullptr;
    int rc = scratch_on_current_device(&ws);
    if (rc) return rc;
    if ((rc = check_call("s2_inverse_noalloc", P, flm, f, batch, ws))) return rc;
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    g_no_timing = true;
    for (int b = 0; b < batch && rc == S2_OK; ++b)       // one map's workspace at a time
        rc = run_inverse(P, (const double2 *)flm + b * slab, (double2 *)f + (size_t)b * P->nsamp, map_strides(P), 1,
                         P->w_sht, (char *)ws, st, true);
    g_no_timing = false;
    return rc;
}

int s2_forward(s2_plan_t P, const void *f, void *flm, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_forward", P, f, flm, batch, workspace);
    if (rc) return rc;
    if (P->N != 1) return fail(S2_ERR_INVALID_ARG, "s2_forward: plan was created for SO(3) (N=%d)", P->N);
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    if (P->mfma)
        return run_forward_mfma(P, (const double2 *)f, batch, (double2 *)flm, P->w_sht, (char *)workspace, st, false);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_forward(P, (const double2 *)f + (size_t)b * P->nsamp, map_strides(P), (double2 *)flm + b * slab, nm,
                           P->w_sht, (char *)workspace, st, false);
    });
}

int s2_inverse_adjoint(s2_plan_t P, const void *g, void *g_flm, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_inverse_adjoint", P, g, g_flm, batch, workspace);
    if (rc) return rc;
    if (P->N != 1) return fail(S2_ERR_INVALID_ARG, "s2_inverse_adjoint: plan was created for SO(3) (N=%d)", P->N);
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    if (P->mfma)
        return run_forward_mfma(P, (const double2 *)g, batch, (double2 *)g_flm, P->w_sht, (char *)workspace, st, true);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_forward(P, (const double2 *)g + (size_t)b * P->nsamp, map_strides(P), (double2 *)g_flm + b * slab, nm,
                           P->w_sht, (char *)workspace, st, true);
    });
}

int s2_forward_adjoint(s2_plan_t P, const void *g_flm, void *g, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_forward_adjoint", P, g_flm, g, batch, workspace);
    if (rc) return rc;
    if (P->N != 1) return fail(S2_ERR_INVALID_ARG, "s2_forward_adjoint: plan was created for SO(3) (N=%d)", P->N);
    if (P->mfma) return fail(S2_ERR_UNSUPPORTED, "s2_forward_adjoint: available for FP64 plans");
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    return over_groups(batch, P->group, [&](int b, int nm) {
        const double2 *G = (const double2 *)g_flm + b * slab;
        double2 *out = (double2 *)g + (size_t)b * P->nsamp;
        if (P->sampling == S2_MW || P->sampling == S2_MWSS)
            return run_forward_adjoint_mw(P, G, out, map_strides(P), nm, P->w_sht, (char *)workspace, st);
        int rc = run_inverse(P, G, out, map_strides(P), nm, P->w_fadj, (char *)workspace, st);
        if (rc) return rc;
        if (P->ringq)
            HIPCHK(launch_ring_scale(st, nm, P->nsamp, P->nring, 2 * P->L - 1, P->ringq, out), "quadrature weights");
        return S2_OK;
    });
}

int so3_inverse(s2_plan_t P, const void *flmn, void *f, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("so3_inverse", P, flmn, f, batch, workspace);
    if (rc) return rc;
    if (P->sampling != S2_MW || P->spin != 0) return fail(S2_ERR_INVALID_ARG, "so3_inverse: needs an MW spin-0 plan");
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const int S = P->nslice;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    if (P->mfma) {
        double2 *tmp = (S > 1) ? (double2 *)((char *)workspace + P->off_mmaps) : (double2 *)f;
        if ((rc = run_inverse_mfma(P, (const double2 *)flmn, batch, tmp, P->w_so3i, (char *)workspace, st))) return rc;
        if (S > 1) {
            TIMED(S2_STAGE_GAMMA);
            HIPCHK(launch_gamma_dft(st, batch, S * P->nsamp, S * P->nsamp, P->N, P->nsamp, +1, 1.0, P->groots, tmp,
                                    (double2 *)f), "gamma DFT");
        }
        return S2_OK;
    }
    return over_groups(batch, P->group, [&](int b, int nm) {
        double2 *out = (double2 *)f + (size_t)b * S * P->nsamp;
        double2 *tmp = S > 1 ? (double2 *)((char *)workspace + P->off_maps) : out;
        const Strides sm = S > 1 ? Strides{tmp_stride(P), P->nsamp} : map_strides(P);
        int rc = run_inverse(P, (const double2 *)flmn + (size_t)b * S * slab, tmp, sm, nm, P->w_so3i,
                             (char *)workspace, st);
        if (rc || S == 1) return rc;
        TIMED(S2_STAGE_GAMMA);
        HIPCHK(launch_gamma_dft(st, nm, sm.map, S * P->nsamp, P->N, P->nsamp, +1, 1.0, P->groots, tmp, out), "gamma DFT");
        return S2_OK;
    });
}

int so3_forward(s2_plan_t P, const void *f, void *flmn, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("so3_forward", P, f, flmn, batch, workspace);
    if (rc) return rc;
    if (P->sampling != S2_MW || P->spin != 0) return fail(S2_ERR_INVALID_ARG, "so3_forward: needs an MW spin-0 plan");
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const int S = P->nslice;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    if (P->mfma) {
        const double2 *src = (const double2 *)f;
        if (S > 1) {
            double2 *tmp = (double2 *)((char *)workspace + P->off_mmaps);
            TIMED(S2_STAGE_GAMMA);
            HIPCHK(launch_gamma_dft(st, batch, S * P->nsamp, S * P->nsamp, P->N, P->nsamp, -1, 2.0 * M_PI / (double)S,
                                    P->groots, src, tmp), "gamma DFT");
            src = tmp;
        }
        // one slice (N = 1): the gamma rule is the weight 2 pi alone, folded into the finish
        return run_forward_mfma(P, src, batch, (double2 *)flmn, S > 1 ? P->w_so3f : P->w_so3f_n1, (char *)workspace, st,
                                false);
    }
    return over_groups(batch, P->group, [&](int b, int nm) {
        const double2 *in = (const double2 *)f + (size_t)b * S * P->nsamp;
        double2 *tmp = (double2 *)((char *)workspace + P->off_maps);
        // f_n = 2pi/(2N-1) sum_k f(gamma_k) e^{-i n gamma_k}  (Eq. 16, exact equispaced rule)
        {
            TIMED(S2_STAGE_GAMMA);
            HIPCHK(launch_gamma_dft(st, nm, S * P->nsamp, tmp_stride(P), P->N, P->nsamp, -1, 2.0 * M_PI / (double)S,
                                    P->groots, in, tmp), "gamma DFT");
        }
        return run_forward(P, tmp, Strides{tmp_stride(P), P->nsamp}, (double2 *)flmn + (size_t)b * S * slab, nm,
                           P->w_so3f, (char *)workspace, st, false);
    });
}

static int check_real(const char *fn, s2_plan_t P)
{
    if (P->N != 1) return fail(S2_ERR_INVALID_ARG, "%s: plan was created for SO(3) (N=%d)", fn, P->N);
    if (P->spin != 0) return fail(S2_ERR_UNSUPPORTED, "%s: real signals need a spin-0 plan", fn);
    if (P->mfma) return fail(S2_ERR_UNSUPPORTED, "%s: available for FP64 plans", fn);
    return S2_OK;
}

int s2_inverse_real(s2_plan_t P, const void *flm, void *f, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_inverse_real", P, flm, f, batch, workspace);
    if (rc || (rc = check_real("s2_inverse_real", P))) return rc;
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_inverse_real(P, (const double2 *)flm + b * slab, (long long)slab, (double *)f + (size_t)b * P->nsamp,
                                nm, P->w_sht, (char *)workspace, st);
    });
}

int s2_forward_real(s2_plan_t P, const void *f, void *flm, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_forward_real", P, f, flm, batch, workspace);
    if (rc || (rc = check_real("s2_forward_real", P))) return rc;
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_forward_real(P, (const double *)f + (size_t)b * P->nsamp, (double2 *)flm + b * slab, nm,
                                (char *)workspace, st);
    });
}

int s2_inverse_real_adjoint(s2_plan_t P, const void *g, void *g_flm, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_inverse_real_adjoint", P, g, g_flm, batch, workspace);
    if (rc || (rc = check_real("s2_inverse_real_adjoint", P))) return rc;
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_forward_real(P, (const double *)g + (size_t)b * P->nsamp, (double2 *)g_flm + b * slab, nm,
                                (char *)workspace, st, true);
    });
}

int s2_forward_real_adjoint(s2_plan_t P, const void *g_flm, void *g, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("s2_forward_real_adjoint", P, g_flm, g, batch, workspace);
    if (rc || (rc = check_real("s2_forward_real_adjoint", P))) return rc;
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    return over_groups(batch, P->group, [&](int b, int nm) {
        return run_forward_real_adjoint(P, (const double2 *)g_flm + b * slab, (double *)g + (size_t)b * P->nsamp, nm,
                                        (char *)workspace, st);
    });
}

int so3_inverse_adjoint(s2_plan_t P, const void *g, void *g_flmn, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("so3_inverse_adjoint", P, g, g_flmn, batch, workspace);
    if (rc) return rc;
    if (P->sampling != S2_MW || P->spin != 0)
        return fail(S2_ERR_INVALID_ARG, "so3_inverse_adjoint: needs an MW spin-0 plan");
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const int S = P->nslice;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    // so3_inverse = (gamma synthesis, sign +1) after the per-n inverses, so its adjoint is the
    // gamma analysis with unit weight (sign -1) followed by the per-n inverse adjoints.
    if (P->mfma) {
        const double2 *src = (const double2 *)g;
        if (S > 1) {
            double2 *tmp = (double2 *)((char *)workspace + P->off_mmaps);
            TIMED(S2_STAGE_GAMMA);
            HIPCHK(launch_gamma_dft(st, batch, S * P->nsamp, S * P->nsamp, P->N, P->nsamp, -1, 1.0, P->groots, src, tmp),
                   "gamma DFT");
            src = tmp;
        }
        return run_forward_mfma(P, src, batch, (double2 *)g_flmn, P->w_so3i, (char *)workspace, st, true);
    }
    return over_groups(batch, P->group, [&](int b, int nm) {
        const double2 *src = (const double2 *)g + (size_t)b * S * P->nsamp;
        Strides sm = map_strides(P);
        if (S > 1) {
            double2 *tmp = (double2 *)((char *)workspace + P->off_maps);
            TIMED(S2_STAGE_GAMMA);
            HIPCHK(launch_gamma_dft(st, nm, sm.map, tmp_stride(P), P->N, P->nsamp, -1, 1.0, P->groots, src, tmp),
                   "gamma DFT");
            src = tmp;
            sm.map = tmp_stride(P);
        }
        return run_forward(P, src, sm, (double2 *)g_flmn + (size_t)b * S * slab, nm, P->w_so3i, (char *)workspace, st,
                           true);
    });
}

int so3_forward_adjoint(s2_plan_t P, const void *g_flmn, void *g, int batch, void *workspace, void *hip_stream)
{
    int rc = check_call("so3_forward_adjoint", P, g_flmn, g, batch, workspace);
    if (rc) return rc;
    if (P->sampling != S2_MW || P->spin != 0)
        return fail(S2_ERR_INVALID_ARG, "so3_forward_adjoint: needs an MW spin-0 plan");
    if (P->mfma) return fail(S2_ERR_UNSUPPORTED, "so3_forward_adjoint: available for FP64 plans");
    if (batch == 0) return S2_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const int S = P->nslice;
    const size_t slab = (size_t)P->L * (2 * P->L - 1);
    // so3_forward = per-n MW forwards after the gamma analysis (sign -1, weight 2pi/(2N-1)), so
    // its adjoint is the per-n forward adjoints followed by the gamma synthesis with that weight.
    double2 *tmp = (double2 *)((char *)workspace + P->off_maps);
    return over_groups(batch, P->group, [&](int b, int nm) {
        int rc = run_forward_adjoint_mw(P, (const double2 *)g_flmn + (size_t)b * S * slab, tmp,
                                        Strides{tmp_stride(P), P->nsamp}, nm, P->w_so3f, (char *)workspace, st);
        if (rc) return rc;
        TIMED(S2_STAGE_GAMMA);
        HIPCHK(launch_gamma_dft(st, nm, tmp_stride(P), S * P->nsamp, P->N, P->nsamp, +1, 2.0 * M_PI / (double)S,
                                P->groots, tmp, (double2 *)g + (size_t)b * S * P->nsamp), "gamma DFT");
        return S2_OK;
    });
}

int s2_plan_set_timing(s2_plan_t P, int enable)
{
    if (!P) return fail(S2_ERR_INVALID_ARG, "s2_plan_set_timing: plan is NULL");
    P->timing = enable != 0;
    return S2_OK;
}

int s2_plan_read_timing(s2_plan_t P, s2_timing_t *out)
{
    if (!P || !out) return fail(S2_ERR_INVALID_ARG, "s2_plan_read_timing: null argument");
    for (int s = 0; s < S2_NSTAGES; ++s) { out->ms[s] = 0.0; out->launches[s] = 0; }
    int rc = S2_OK;
    for (auto &t : P->tl) {
        float ms = 0.0f;
        hipError_t e = hipEventSynchronize(t.b);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, t.a, t.b);
        if (e != hipSuccess && rc == S2_OK) rc = hipfail(e, "stage timing");
        if (t.stage >= 0 && t.stage < S2_NSTAGES) { out->ms[t.stage] += ms; out->launches[t.stage] += 1; }
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
    }
    P->tl.clear();
    return rc;
}

int s2_debug_wigner_d(s2_plan_t P, int n, void *out, void *hip_stream)
{
    if (!P || !out) return fail(S2_ERR_INVALID_ARG, "s2_debug_wigner_d: null argument");
    int ri = -1;
    for (size_t i = 0; i < P->runs.size(); ++i) if (P->runs[i].n == n) ri = (int)i;
    if (ri < 0) return fail(S2_ERR_INVALID_ARG, "s2_debug_wigner_d: n=%d is not a run of this plan", n);
    hipStream_t st = (hipStream_t)hip_stream;
    HIPCHK(hipMemsetAsync(out, 0, (size_t)P->nreg * P->L * P->L * sizeof(double), st), "memset");
    HIPCHK(launch_debug_d(st, P->L, P->nreg, n, P->cot, P->csc, P->lsin, P->lcos, P->lbin[ri], P->kap, P->gtab,
                          (double *)out), "debug d");
    return S2_OK;
}

}  // extern "C"
