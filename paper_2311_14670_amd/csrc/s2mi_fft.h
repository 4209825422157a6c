// s2mi_fft.h -- device DFT engine: one workgroup transforms one sequence held
// in LDS.  Used for the per-ring phi-DFTs (Eqs. 31-32) and the MW theta
// half-sample shifts.
//
// Engine: mixed-radix FFT over radices {2,3,4,5,7,8,9,11,13}, every butterfly in place
// in LDS.  Forward (sign -1) by decimation in frequency: natural order in, the spectrum
// at fft_pos(k); inverse (sign +1) by decimation in time, the same stages backwards.  So a
// stage is one read and one write of the sequence and one barrier, a thread holds one
// butterfly at a time, a forward transform followed by an inverse one never reorders, and
// its innermost two stages (with a product in between) are one pass, as are an inverse's
// last stage and the first of the forward that follows.  First loads and last stores go
// straight to their source and target.  Lengths with a larger
// prime factor go through Bluestein's chirp-z identity
//   X_k = conj(c_k) sum_j (x_j conj(c_j)) c_{k-j},  c_j = e^{i pi j^2 / n},
// evaluated as a power-of-two circular convolution (rings of one length: s2mi_conv.h).
//
// What bounds it: latency (barriers, first loads of a stage) and the FP64 work of the
// butterflies; 64 KiB of LDS at 4095 points leave two workgroups on a compute unit.
// Measured on MI355X, ms, self-sorting stages with a barrier on both sides of each -> this
// form: 4095 points (MW L = 2048, one map / 64 maps) inverse phi-DFT 0.178 / 4.6 -> 0.176 /
// 4.6, forward 0.113 / 7.9 -> 0.097 / 6.5, theta filter 0.253 / 15.0 -> 0.221 / 13.1; HEALPix
// nside 1024, L = 2048, real 0.54, 0.32 -> 0.48, 0.24; nside 64, L = 128, 8 maps 0.026, 0.021
// -> 0.023, 0.017.  (The filter's rings kept in registers to its end: no gain, spills.)
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "s2mi_internal.h"

namespace s2mi {

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ double2 cmulc(double2 a, double2 b)   // a * conj(b)
{
    return make_double2(fma(a.x, b.x, a.y * b.y), fma(a.y, b.x, -a.x * b.y));
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// multiply by sign * i  (sign = -1: -i, +1: +i)
__device__ __forceinline__ double2 cmuli(double2 a, int sign)
{
    return sign < 0 ? make_double2(a.y, -a.x) : make_double2(-a.y, a.x);
}

__device__ __forceinline__ double2 ldroot(const double *tw, int idx, int sign)
{
    const double2 t = reinterpret_cast<const double2 *>(tw)[idx];
    return sign < 0 ? t : make_double2(t.x, -t.y);
}

// cos(2 pi k / R), sin(2 pi k / R) for the odd radices, k = 0 .. R-1.
template <int R> struct OddRoots;
template <> struct OddRoots<3> {
    static constexpr double c[3] = {1.0, -0.5, -0.5};
    static constexpr double s[3] = {0.0, 0.86602540378443864676, -0.86602540378443864676};
};
template <> struct OddRoots<5> {
    static constexpr double c[5] = {1.0, 0.3090169943749474241, -0.8090169943749474241, -0.8090169943749474241,
                                    0.3090169943749474241};
    static constexpr double s[5] = {0.0, 0.95105651629515357212, 0.58778525229247312917, -0.58778525229247312917,
                                    -0.95105651629515357212};
};
template <> struct OddRoots<7> {
    static constexpr double c[7] = {1.0, 0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624,
                                    -0.90096886790241912624, -0.22252093395631440429, 0.62348980185873353053};
    static constexpr double s[7] = {0.0, 0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048,
                                    -0.43388373911755812048, -0.97492791218182360702, -0.78183148246802980871};
};
template <> struct OddRoots<11> {
    static constexpr double c[11] = {1.0, 0.84125353283118116886, 0.41541501300188642553, -0.14231483827328514044,
                                     -0.65486073394528506406, -0.95949297361449738989, -0.95949297361449738989,
                                     -0.65486073394528506406, -0.14231483827328514044, 0.41541501300188642553,
                                     0.84125353283118116886};
    static constexpr double s[11] = {0.0, 0.54064081745559758211, 0.90963199535451837141, 0.98982144188093273238,
                                     0.75574957435425828377, 0.28173255684142969771, -0.28173255684142969771,
                                     -0.75574957435425828377, -0.98982144188093273238, -0.90963199535451837141,
                                     -0.54064081745559758211};
};
template <> struct OddRoots<13> {
    static constexpr double c[13] = {1.0, 0.8854560256532098959, 0.56806474673115580251, 0.12053668025532305335,
                                     -0.35460488704253562597, -0.74851074817110109863, -0.97094181742605202716,
                                     -0.97094181742605202716, -0.74851074817110109863, -0.35460488704253562597,
                                     0.12053668025532305335, 0.56806474673115580251, 0.8854560256532098959};
    static constexpr double s[13] = {0.0, 0.46472317204376854566, 0.82298386589365639458, 0.9927088740980539928,
                                     0.93501624268541482344, 0.66312265824079520238, 0.23931566428755776715,
                                     -0.23931566428755776715, -0.66312265824079520238, -0.93501624268541482344,
                                     -0.9927088740980539928, -0.82298386589365639458, -0.46472317204376854566};
};

// In-place DFT of N = 2, 4, 8, 16 registers, natural order: v_q = sum_r v_r e^{S 2 pi i r q / N}.
template <int N, int S>
__device__ __forceinline__ void dft_reg(double2 *v)
{
    if constexpr (N == 2) {
        const double2 a = v[0];
        v[0] = cadd(a, v[1]);
        v[1] = csub(a, v[1]);
    } else if constexpr (N == 4) {
        const double2 a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
        const double2 b0 = cadd(v[1], v[3]), b1 = cmuli(csub(v[1], v[3]), S);
        v[0] = cadd(a0, b0);
        v[1] = cadd(a1, b1);
        v[2] = csub(a0, b0);
        v[3] = csub(a1, b1);
    } else if constexpr (N == 8) {
        double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft_reg<4, S>(e);
        dft_reg<4, S>(o);
        constexpr double h = 0.70710678118654752440;
        const double2 o1 = make_double2(h * (o[1].x - S * o[1].y), h * (o[1].y + S * o[1].x));
        const double2 o3 = make_double2(h * (-o[3].x - S * o[3].y), h * (-o[3].y + S * o[3].x));
        o[2] = cmuli(o[2], S);
        v[0] = cadd(e[0], o[0]);
        v[4] = csub(e[0], o[0]);
        v[1] = cadd(e[1], o1);
        v[5] = csub(e[1], o1);
        v[2] = cadd(e[2], o[2]);
        v[6] = csub(e[2], o[2]);
        v[3] = cadd(e[3], o3);
        v[7] = csub(e[3], o3);
    } else {
        // r = r0 + 4 r1, q = q0 + 4 q1
        constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
        double2 a[4][4];                                 // [r0][q0]
#pragma unroll
        for (int r0 = 0; r0 < 4; ++r0) {
#pragma unroll
            for (int r1 = 0; r1 < 4; ++r1) a[r0][r1] = v[r0 + 4 * r1];
            dft_reg<4, S>(a[r0]);
        }
        auto mul8 = [](double2 x) { return make_double2(h * (x.x - S * x.y), h * (x.y + S * x.x)); };   // e^{S i pi/4}
        a[1][1] = cmul(a[1][1], make_double2(c1, S * s1));
        a[1][2] = mul8(a[1][2]);
        a[1][3] = cmul(a[1][3], make_double2(s1, S * c1));
        a[2][1] = mul8(a[2][1]);
        a[2][2] = cmuli(a[2][2], S);
        a[2][3] = cmuli(mul8(a[2][3]), S);
        a[3][1] = cmul(a[3][1], make_double2(s1, S * c1));
        a[3][2] = cmuli(mul8(a[3][2]), S);
        a[3][3] = cmul(a[3][3], make_double2(-c1, -S * s1));
#pragma unroll
        for (int q0 = 0; q0 < 4; ++q0) {
            double2 b[4] = {a[0][q0], a[1][q0], a[2][q0], a[3][q0]};
            dft_reg<4, S>(b);
#pragma unroll
            for (int q1 = 0; q1 < 4; ++q1) v[q0 + 4 * q1] = b[q1];
        }
    }
}

// The same for R = 9.
template <int S>
__device__ __forceinline__ void dft_nine(double2 (&v)[9])
{
    // 9 = 3 x 3: with r = 3j + k and q = p + 3s, y_q = sum_k w9^{kp} w3^{ks}
    // (sum_j v_{3j+k} w3^{jp}): three radix-3 DFTs, twiddles, three more
    constexpr double c3 = -0.5, s3 = 0.86602540378443864676;   // cos, sin of 2 pi / 3
    auto dft3 = [](double2 a, double2 b, double2 c, double2 &y0, double2 &y1, double2 &y2) {
        const double2 t = cadd(b, c), d = csub(b, c);
        y0 = cadd(a, t);
        const double2 mid = make_double2(fma(c3, t.x, a.x), fma(c3, t.y, a.y));
        const double2 rot = cmuli(make_double2(s3 * d.x, s3 * d.y), S);   // S i s3 (b - c)
        y1 = cadd(mid, rot);
        y2 = csub(mid, rot);
    };
    double2 t[3][3];                                  // t[k][p]
#pragma unroll
    for (int k = 0; k < 3; ++k) dft3(v[k], v[3 + k], v[6 + k], t[k][0], t[k][1], t[k][2]);
    constexpr double sg = S;                          // w9^e = cos(2 pi e / 9) + S i sin(2 pi e / 9)
    const double2 w1 = make_double2(0.76604444311897803520, sg * 0.64278760968653932632);
    const double2 w2 = make_double2(0.17364817766693034885, sg * 0.98480775301220805937);
    const double2 w4 = make_double2(-0.93969262078590838405, sg * 0.34202014332566873304);
    t[1][1] = cmul(t[1][1], w1);
    t[1][2] = cmul(t[1][2], w2);
    t[2][1] = cmul(t[2][1], w2);
    t[2][2] = cmul(t[2][2], w4);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        double2 y0, y1, y2;
        dft3(t[0][p], t[1][p], t[2][p], y0, y1, y2);
        v[p] = y0;
        v[p + 3] = y1;
        v[p + 6] = y2;
    }
}

// v[q] times w^q, q < R, w = e^{S 2 pi i idx / len}; the powers as products of two lower
// ones, so their rounding grows with log2 q
template <int R, int S>
__device__ __forceinline__ void twiddle(double2 (&v)[R], const double *tw, int idx)
{
    double2 w[R];
    w[1] = ldroot(tw, idx, S);
#pragma unroll
    for (int q = 1; q < R; ++q) {
        if (q > 1) w[q] = cmul(w[q / 2], w[q - q / 2]);
        v[q] = cmul(v[q], w[q]);
    }
}

// One butterfly of radix R: the twiddled or plain inputs and outputs of a stage.
template <int R, bool PAIRS = (R % 2 == 1 && R != 9)>
struct Butterfly {                                       // 2, 4, 8, 9
    double2 v[R];
    template <int S>
    __device__ __forceinline__ void twiddle_in(const double *tw, int idx)
    {
        twiddle<R, S>(v, tw, idx);
    }
    // out(q, y_q w^q), w = e^{S 2 pi i idx / len} (TW; else w = 1)
    template <int S, bool TW, class Out>
    __device__ __forceinline__ void run(const double *tw, int idx, Out out)
    {
        if constexpr (R == 9) dft_nine<S>(v);
        else dft_reg<R, S>(v);
        if (TW && idx > 0) twiddle<R, S>(v, tw, idx);
#pragma unroll
        for (int q = 0; q < R; ++q) out(q, v[q]);
    }
};

// Odd R: with a_r = v_r + v_{R-r}, b_r = v_r - v_{R-r} (r <= (R-1)/2),
//   y_q, y_{R-q} = v_0 + sum_r a_r cos(2 pi rq/R) +- S i sum_r b_r sin(2 pi rq/R),
// a pair at a time, so that the outputs need no registers of their own; the twiddles of a
// pair are w^q, by repeated products, and w^{R-q} = w^R conj(w^q), w^R from the table.
template <int R>
struct Butterfly<R, true> {
    static constexpr int H = (R - 1) / 2;
    double2 v[R];
    template <int S>
    __device__ __forceinline__ void twiddle_in(const double *tw, int idx)
    {
        const double2 w1 = ldroot(tw, idx, S), wR = ldroot(tw, R * idx, S);
        double2 w = w1;
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            if (r > 1) w = cmul(w, w1);
            v[r] = cmul(v[r], w);
            v[R - r] = cmul(v[R - r], cmulc(wR, w));
        }
    }
    template <int S, bool TW, class Out>
    __device__ __forceinline__ void run(const double *tw, int idx, Out out)
    {
        double2 w1, wR, w;
        if constexpr (TW) {
            w1 = ldroot(tw, idx, S);
            wR = ldroot(tw, R * idx, S);
        }
        double2 y0 = v[0];
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            const double2 a = cadd(v[r], v[R - r]), b = csub(v[r], v[R - r]);
            v[r] = a;
            v[R - r] = b;
            y0 = cadd(y0, a);
        }
        out(0, y0);
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            double2 A = v[0], B = make_double2(0.0, 0.0);
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const double c = OddRoots<R>::c[(r * q) % R], s = OddRoots<R>::s[(r * q) % R];
                A.x = fma(v[r].x, c, A.x);
                A.y = fma(v[r].y, c, A.y);
                B.x = fma(v[R - r].x, s, B.x);
                B.y = fma(v[R - r].y, s, B.y);
            }
            const double2 iB = cmuli(B, S);
            if constexpr (TW) {
                w = q > 1 ? cmul(w, w1) : w1;
                out(q, cmul(cadd(A, iB), w));
                out(R - q, cmul(csub(A, iB), cmulc(wR, w)));
            } else {
                out(q, cadd(A, iB));
                out(R - q, csub(A, iB));
            }
        }
    }
};

// LDS place of point i: in lengths with enough factors of two the low bits are mixed with
// the next ones, so that a last stage of radix 8 (a thread's points side by side) meets
// the banks without conflict.
__device__ __forceinline__ int fft_place(const FftArgs *f, int i) { return i ^ ((i >> 3) & f->mix); }

// position of frequency k in the order the forward stages leave
__device__ __forceinline__ int fft_pos(const FftArgs *f, int k)
{
    int p = 0;
    for (int s = 0; s < f->nst; ++s) {
        const int q = (int)__umulhi((unsigned)k, f->stage[s].mrad);   // k / rad
        p += (k - q * f->stage[s].rad) * f->stage[s].sub;
        k = q;
    }
    return p;
}

// P2: lengths that are powers of two; SMALL: radices up to 9
template <bool P2, bool SMALL, class G>
__device__ __forceinline__ void fft_radix(int R, G g)
{
    if constexpr (P2) {
        if (R == 8) g(std::integral_constant<int, 8>());
        else if (R == 4) g(std::integral_constant<int, 4>());
        else g(std::integral_constant<int, 2>());
        return;
    }
    switch (R) {
    case 2: g(std::integral_constant<int, 2>()); break;
    case 3: g(std::integral_constant<int, 3>()); break;
    case 4: g(std::integral_constant<int, 4>()); break;
    case 5: g(std::integral_constant<int, 5>()); break;
    case 7: g(std::integral_constant<int, 7>()); break;
    case 8: g(std::integral_constant<int, 8>()); break;
    case 9: g(std::integral_constant<int, 9>()); break;
    default: break;
    }
    if constexpr (!SMALL) switch (R) {
    case 11: g(std::integral_constant<int, 11>()); break;
    case 13: g(std::integral_constant<int, 13>()); break;
    default: break;
    }
}

// Stage s over the sequence: a butterfly's points i = base + sub r come from load(i) and go
// to store(i, v).
//   FWD: stage s of the forward transform (butterfly, twiddles)
//   INV: of the inverse (twiddles, butterfly)
//   TURN, s = 0: the last inverse and the first forward stage, mid(i, v) on the points between
//   INNER, s = nst - 1: the last forward and the first inverse stage, mid(p, v) on the
//   positions of the spectrum
enum { FFT_FWD, FFT_INV, FFT_TURN, FFT_INNER };
template <int KIND, bool P2 = false, class Load, class Mid, class Store>
__device__ __forceinline__ void fft_stage(const FftArgs *f, int s, Load load, Mid mid, Store store)
{
    const FftStage *g = f->stage + s;
    const double *tw = f->tw;
    const int sub = g->sub, nbf = g->nbf, tstep = g->tstep, T = blockDim.x;
    const unsigned msub = g->msub;                           // j / sub = umulhi(j, msub), sub > 1
    fft_radix<P2, KIND == FFT_TURN || KIND == FFT_INNER>(g->rad, [&](auto Rc) {
        constexpr int R = decltype(Rc)::value;
        const int B = sub * R;
#pragma unroll 1
        for (int j = threadIdx.x; j < nbf; j += T) {
            const int blk = sub > 1 ? (int)__umulhi((unsigned)j, msub) : j, jj = j - blk * sub;
            const int base = blk * B + jj;
            const int idx = jj * tstep;
            Butterfly<R> x;
#pragma unroll
            for (int r = 0; r < R; ++r) x.v[r] = load(base + sub * r);
            auto out = [&](int q, double2 y) { store(base + sub * q, y); };
            if constexpr (KIND == FFT_FWD) {
                x.template run<-1, true>(tw, idx, out);
            } else if constexpr (KIND == FFT_INV) {
                if (sub > 1) x.template twiddle_in<1>(tw, idx);
                x.template run<1, false>(tw, 0, out);
            } else {
                Butterfly<R> y;
                auto turn = [&](int q, double2 z) { y.v[q] = mid(base + sub * q, z); };
                if constexpr (KIND == FFT_INNER) {
                    x.template run<-1, false>(tw, 0, turn);
                    y.template run<1, false>(tw, 0, out);
                } else {
                    if (sub > 1) x.template twiddle_in<1>(tw, idx);
                    x.template run<1, false>(tw, 0, turn);
                    y.template run<-1, true>(tw, idx, out);
                }
            }
        }
    });
    __syncthreads();
}

// INNER and TURN for any radix: 11 and 13 as two stages (both butterflies at once take more
// registers than the 128 of a wave with three others)
template <class Load, class Mid, class Store>
__device__ __forceinline__ void fft_inner(const FftArgs *f, int s, Load load, Mid mid, Store store)
{
    if (f->stage[s].rad <= 9) {
        fft_stage<FFT_INNER>(f, s, load, mid, store);
    } else {
        fft_stage<FFT_FWD>(f, s, load, mid, [&](int i, double2 v) { store(i, mid(i, v)); });
        fft_stage<FFT_INV>(f, s, load, mid, store);
    }
}
template <class Load, class Mid, class Store>
__device__ __forceinline__ void fft_turn(const FftArgs *f, Load load, Mid mid, Store store)
{
    if (f->stage[0].rad <= 9) {
        fft_stage<FFT_TURN>(f, 0, load, mid, store);
    } else {
        fft_stage<FFT_INV>(f, 0, load, mid, [&](int i, double2 v) { store(i, mid(i, v)); });
        fft_stage<FFT_FWD>(f, 0, load, mid, store);
    }
}

struct FftNone {
    __device__ double2 operator()(int) const { return make_double2(0.0, 0.0); }
    __device__ double2 operator()(int, double2 v) const { return v; }
};

// forward stages a .. b - 1 in LDS (inverse: b - 1 down to a)
template <bool P2 = false>
__device__ __forceinline__ void fft_forward(double2 *buf, const FftArgs *f, int a, int b)
{
    auto get = [&](int i) { return buf[fft_place(f, i)]; };
    auto put = [&](int i, double2 v) { buf[fft_place(f, i)] = v; };
#pragma unroll 1
    for (int s = a; s < b; ++s) fft_stage<FFT_FWD, P2>(f, s, get, FftNone(), put);
}
template <bool P2 = false>
__device__ __forceinline__ void fft_inverse(double2 *buf, const FftArgs *f, int a, int b)
{
    auto get = [&](int i) { return buf[fft_place(f, i)]; };
    auto put = [&](int i, double2 v) { buf[fft_place(f, i)] = v; };
#pragma unroll 1
    for (int s = b - 1; s >= a; --s) fft_stage<FFT_INV, P2>(f, s, get, FftNone(), put);
}

// The cyclic convolution of len points, a power of two above 8, in LDS: load(i) -> spectrum ->
// mid(position, value) -> store(i, value).
template <class Load, class Mid, class Store>
__device__ __forceinline__ void fft_convolve(double2 *buf, const FftArgs *f, Load load, Mid mid, Store store)
{
    const int last = f->nst - 1;
    auto get = [&](int i) { return buf[fft_place(f, i)]; };
    auto put = [&](int i, double2 v) { buf[fft_place(f, i)] = v; };
    fft_stage<FFT_FWD, true>(f, 0, load, FftNone(), put);
    fft_forward<true>(buf, f, 1, last);
    fft_stage<FFT_INNER, true>(f, last, get, mid, put);
    fft_inverse<true>(buf, f, 1, last);
    fft_stage<FFT_INV, true>(f, 0, get, FftNone(), store);
}

// Where bin k of the spectrum (not Bluestein: the order of the stages) lies in LDS.  (From a
// table: the digits of k by multiplications took 6 % of a phi-DFT of 4095 points.)
__device__ __forceinline__ int fft_slot(const FftArgs *f, int k) { return f->blue ? fft_place(f, k) : f->slot[k]; }

// DFTs of length n = f->n in LDS (f->len places).  sign = -1: of load(k), k < n, the result in
// the slots of its bins; sign = +1: of the bins in their slots, the result to store(k, value).
// load may read buf at point k's place.
//
// Bluestein: the inverse is conj(DFT(conj(x))); the chirped input u_j = x_j conj(c_j) is
// convolved with the chirp, then de-chirped.
//
// Split Bluestein (convolution length M = 2H, H = f.len the LDS engine length,
// n < H): u is zero past n < H, so the even spectrum samples U[2k] are
// DFT_H(u)[k] and the odd ones U[2k+1] are DFT_H(u w^j)[k], w = e^{-2 pi i/M}.
// The inverse transform of V = U b~ is needed only at t < n < H, where it is
// IDFT_H(V_even)[t] + conj(w)^t IDFT_H(V_odd)[t].  The halves run one after the
// other in the same LDS buffer; u and the even result wait in scr (2H entries
// of this workgroup's global scratch, each read back only by the thread that
// wrote it).
template <int SIGN, class Load, class Store>
__device__ __forceinline__ void dft_lds(double2 *buf, const FftArgs *f, double2 *scr, Load load, Store store)
{
    const int n = f->n, len = f->len, nst = f->nst;
    auto get = [&](int i) { return buf[fft_place(f, i)]; };
    auto put = [&](int i, double2 v) { buf[fft_place(f, i)] = v; };
    if (!f->blue) {
        if constexpr (SIGN < 0) {
            fft_stage<FFT_FWD>(f, 0, load, FftNone(), put);
            fft_forward(buf, f, 1, nst);
        } else {
            fft_inverse(buf, f, 1, nst);
            fft_stage<FFT_INV>(f, 0, get, FftNone(), store);
        }
        return;
    }
    const double2 *ch = reinterpret_cast<const double2 *>(f->chirp);
    const double2 *bf = reinterpret_cast<const double2 *>(f->bflt);
    const double2 *wm = reinterpret_cast<const double2 *>(f->twm);
    const int split = f->split;
#pragma unroll 1
    for (int half = 0; half <= split; ++half) {
        const double2 *b = bf + half * len;
        fft_convolve(
            buf, f,
            [&](int i) {
                if (half) return cmul(scr[i], wm[i]);
                double2 x = make_double2(0.0, 0.0);
                if (i < n) {
                    x = SIGN > 0 ? cconj(get(i)) : load(i);
                    x = cmulc(x, ch[i]);
                }
                if (split) scr[i] = x;
                return x;
            },
            [&](int p, double2 v) { return cmul(v, b[p]); },
            [&](int i, double2 v) {
                if (split && !half) {
                    scr[len + i] = v;
                    return;
                }
                if (i >= n) return;
                if (split) v = cadd(scr[len + i], cmulc(v, wm[i]));
                v = cmulc(v, ch[i]);
                if constexpr (SIGN > 0) store(i, cconj(v));
                else put(i, v);
            });
    }
}

}  // namespace s2mi
