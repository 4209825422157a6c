// s2mi_conv.h -- cyclic convolutions of power-of-two length in registers, and the DFTs
// that run as one (Bluestein's chirp-z identity), for plans whose rings all have one length.
//
// A workgroup of T = M / V threads holds a sequence of M points, V per thread (thread t:
// points t + T i).  Forward FFT by decimation in frequency (radix V, the last stage the
// rest), product with the filter's spectrum, inverse FFT by decimation in time with the
// same stages backwards: the spectrum is never put in natural order, the filter is stored
// in the order the stages leave (conv_index).  Between stages the points change threads
// through LDS, real and imaginary parts one after the other, so a sequence takes 8 M
// bytes: M = 4096 32 KiB and 128 registers, four workgroups on a compute unit.
//
// What bounds it: LDS traffic and the latency between barriers.  The engine of s2mi_fft.h
// takes M = 4096 through 8 radix-8 stages and 4 passes over LDS for the products (12
// reads and writes of 64 KiB, two workgroups per compute unit); here it is four exchanges.
// Measured on MI355X, inverse phi-DFT / forward / theta filter, one map unless stated, ms
// with that engine -> with this one: MW L = 64 (M = 256) 0.013 / 0.013 / 0.022 -> 0.007 /
// 0.007 / 0.011; L = 512 forward and adjoints, 16 maps (M = 2048) 0.27 / 0.23 / - -> 0.13 /
// 0.12; L = 1024 (4096) 0.078 / 0.074 / 0.133 -> 0.043 / 0.040 / 0.061; 32 maps of it
// 1.87 / 2.05 / 3.63 -> 0.92 / 1.12 / 1.51; L = 4096 (16384 in two halves) 2.38 / 1.52 /
// 2.74 -> 1.71 / 0.93 / 1.50.  It wins at every M, so every plan of one ring length
// that needs the identity takes it; HEALPix rings (many lengths in a launch) do not.
#pragma once

#include <hip/hip_runtime.h>

#include "s2mi_fft.h"

namespace s2mi {

// values per thread for an engine of M points
constexpr int conv_values(int M) { return M <= 256 ? 4 : M <= 512 ? 8 : 16; }

// where a convolution kernel's spectrum at frequency k is stored: [value i][thread t]
__host__ __device__ inline int conv_index(int M, int k)
{
    const int V = conv_values(M);
    int p = 0, B = M;                                    // p: position in the order of the stages
    while (B > 1) {
        const int R = B >= V ? V : B;
        B /= R;
        p += (k % R) * B;
        k /= R;
    }
    return (p % V) * (M / V) + p / V;
}

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

// The engine: M points of which a sequence occupies the first n <= (M + 1) / 2 (SPLIT: a
// convolution of 2 M points of which n < M are occupied, as two of M: the even samples of
// the spectrum are the transform of u, the odd ones that of u w^j, w = e^{-pi i / M}, and the
// result at t < M is the sum of the two inverses, the second times conj(w)^t).
template <int M, bool SPLIT>
struct ConvDft {
    static constexpr int V = conv_values(M), T = M / V, MAXT = T, WPE = SPLIT ? 2 : 4;
    static constexpr bool CONV = true;

    // Registers: a thread's points are numbered afresh at each use (the compiler would keep
    // V addresses and conditions from one to the next), and loads around them go in groups
    // of four.
    static __device__ __forceinline__ int first_point()
    {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    }
    static __device__ __forceinline__ void few_loads(int i)
    {
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }

    // LDS place of a point: the low five bits (the bank of a double) mixed with higher ones
    // so that every exchange pattern of 32 lanes below meets 32 banks.  Linear in the bits:
    // place(a + b) = place(a) ^ place(b) where a and b share none.
    static constexpr __device__ int place(int i)
    {
        if constexpr (V == 16) return i ^ ((i >> 4) & 14) ^ (((i >> 8) & 1) * 0x11);
        else if constexpr (V == 8) return i ^ ((i >> 5) & 1) ^ (((i >> 6) & 3) * 0x0a);
        else return i ^ (((i >> 5) & 1) * 0x09) ^ (((i >> 6) & 1) * 0x16);
    }

    // v[i] goes to point wb + ws i, then comes from point rb + rs i (powers of two, no
    // shared bits)
    template <int WS, int RS>
    static __device__ __forceinline__ void exchange(double2 (&v)[V], double *xb, int wb, int rb)
    {
        // only the low five bits need the exclusive or; the rest of a place is an offset of
        // the instruction.  The bases are opaque: the addresses are formed again for each
        // part rather than held in registers across the stages.
        int w0 = place(wb), r0 = place(rb);
        auto at = [xb](int base, int c) -> double & { return xb[(base ^ (c & 31)) + (c & ~31)]; };
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            asm volatile("" : "+v"(w0), "+v"(r0));
            __syncthreads();
#pragma unroll
            for (int i = 0; i < V; ++i) at(w0, place(WS * i)) = part ? v[i].y : v[i].x;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < V; ++i) (part ? v[i].y : v[i].x) = at(r0, place(RS * i));
        }
    }

    // v[q] times w^q, q < V, w = e^{S 2 pi i j / B} (from the roots of M points); the
    // powers as products of two lower ones, so their rounding grows with log2 q
    template <int S>
    static __device__ __forceinline__ void twiddle(double2 (&v)[V], const double *tw, int idx)
    {
        double2 w[V];
        w[1] = ldroot(tw, idx, S);
#pragma unroll
        for (int q = 1; q < V; ++q) {
            if (q > 1) w[q] = cmul(w[q / 2], w[q - q / 2]);
            v[q] = cmul(v[q], w[q]);
        }
    }

    template <int B>
    static __device__ __forceinline__ void forward(double2 (&v)[V], double *xb, const double *tw)
    {
        constexpr int Q = B / V;                         // block size of the next stage
        const int t = threadIdx.x;
        dft_reg<V, -1>(v);
        if constexpr (Q > 1) {
            const int j = t & (Q - 1), b = t / Q * B;
            twiddle<-1>(v, tw, j * (M / B));
            if constexpr (Q >= V) {
                exchange<Q, Q / V>(v, xb, b + j, t / (Q / V) * Q + (t & (Q / V - 1)));
                forward<Q>(v, xb, tw);
            } else {
                exchange<Q, 1>(v, xb, b + j, t * V);
#pragma unroll
                for (int s = 0; s < V; s += Q) dft_reg<Q, -1>(v + s);
            }
        }
    }

    template <int B>
    static __device__ __forceinline__ void inverse(double2 (&v)[V], double *xb, const double *tw)
    {
        constexpr int Q = B / V;
        const int t = threadIdx.x;
        if constexpr (Q > 1) {
            const int j = t & (Q - 1), b = t / Q * B;
            if constexpr (Q >= V) {
                inverse<Q>(v, xb, tw);
                exchange<Q / V, Q>(v, xb, t / (Q / V) * Q + (t & (Q / V - 1)), b + j);
            } else {
#pragma unroll
                for (int s = 0; s < V; s += Q) dft_reg<Q, 1>(v + s);
                exchange<1, Q>(v, xb, t * V, b + j);
            }
            twiddle<1>(v, tw, j * (M / B));
        }
        dft_reg<V, 1>(v);
    }

    static __device__ __forceinline__ void convolve_m(double2 (&v)[V], double *xb, const FftArgs *f, int half)
    {
        forward<M>(v, xb, f->tw);
        const double2 *s = reinterpret_cast<const double2 *>(f->bflt) + half * M + first_point();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            v[i] = cmul(v[i], s[i * T]);
            few_loads(i);
        }
        inverse<M>(v, xb, f->tw);
    }

    // v (points t + T i, zero from n on) <- its convolution with f's kernel, valid below n
    static __device__ __forceinline__ void convolve(double2 (&v)[V], double *xb, const FftArgs *f)
    {
        if constexpr (!SPLIT) {
            convolve_m(v, xb, f, 0);
        } else {
            const double2 *wm = reinterpret_cast<const double2 *>(f->twm);
            double2 u[V];
#pragma unroll
            for (int i = 0; i < V; ++i) u[i] = v[i];
            double2 e[V];
#pragma unroll 1
            for (int half = 0; half < 2; ++half) {
                const double2 *w = wm + first_point();
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    e[i] = v[i];
                    v[i] = half ? cmul(u[i], w[i * T]) : u[i];
                    few_loads(i);
                }
                convolve_m(v, xb, f, half);
            }
            const double2 *w = wm + first_point();
#pragma unroll
            for (int i = 0; i < V; ++i) {
                v[i] = cadd(e[i], cmulc(v[i], w[i * T]));
                few_loads(i);
            }
        }
    }

    // DFT of get(k), k < n = f->n: KEEP: into buf (natural order), else handed to
    // put(k, value).  get may read buf.
    template <bool FILL, bool KEEP, class Get, class Put>
    static __device__ __forceinline__ void dft(double2 *buf, const FftArgs *f, int sign, double2 *, Get get, Put put)
    {
        const int n = f->n;
        const double2 *ch = reinterpret_cast<const double2 *>(f->chirp);
        double2 v[V];
        int t = first_point();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int k = t + T * i;
            v[i] = make_double2(0.0, 0.0);
            if (k < n) {
                double2 x = get(k);
                if (sign > 0) x.y = -x.y;
                v[i] = cmulc(x, ch[k]);
            }
            few_loads(i);
        }
        convolve(v, reinterpret_cast<double *>(buf), f);
        if (KEEP) __syncthreads();
        t = first_point();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int k = t + T * i;
            if (k < n) {
                double2 y = cmulc(v[i], ch[k]);
                if (sign > 0) y.y = -y.y;
                if constexpr (KEEP) buf[k] = y;
                else put(k, y);
            }
            few_loads(i);
        }
        if (KEEP) __syncthreads();
    }
};

// The same interface over the engine of s2mi_fft.h: any length, rings of different ones.
struct LdsDft {
    static constexpr int MAXT = 1024, WPE = 4;
    static constexpr bool CONV = false;

    template <bool FILL, bool KEEP, class Get, class Put>
    static __device__ __forceinline__ void dft(double2 *buf, const FftArgs *f, int sign, double2 *scr, Get get, Put put)
    {
        const int n = f->n;
        if constexpr (FILL) {
            for (int k = threadIdx.x; k < n; k += blockDim.x) buf[k] = get(k);
            __syncthreads();
        }
        dft_lds(buf, f, sign, scr);
        if constexpr (!KEEP)
            for (int k = threadIdx.x; k < n; k += blockDim.x) put(k, buf[k]);
    }
};

}  // namespace s2mi
