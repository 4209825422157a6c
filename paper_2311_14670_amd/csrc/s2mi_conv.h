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
    // so that 32 lanes meet 32 banks in every exchange below (16 in the last one of M = 128).
    // Linear in the bits:
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

    template <int B>
    static __device__ __forceinline__ void forward(double2 (&v)[V], double *xb, const double *tw)
    {
        constexpr int Q = B / V;                         // block size of the next stage
        const int t = threadIdx.x;
        dft_reg<V, -1>(v);
        if constexpr (Q > 1) {
            const int j = t & (Q - 1), b = t / Q * B;
            twiddle<V, -1>(v, tw, j * (M / B));
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
            twiddle<V, 1>(v, tw, j * (M / B));
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

    static __device__ __forceinline__ int slot(const FftArgs *, int k) { return k; }
    static __device__ __forceinline__ int point(const FftArgs *, int t) { return t; }

    // sign = -1: DFT of get(k), k < n = f->n, into the bins' slots of buf; +1: of the bins in their
    // slots, handed to put(k, value) (LDS: which stores into buf)
    template <int SIGN, bool LDS, class Get, class Put>
    static __device__ __forceinline__ void dft(double2 *buf, const FftArgs *f, double2 *, Get get, Put put)
    {
        constexpr bool KEEP = SIGN < 0;
        const int n = f->n;
        const double2 *ch = reinterpret_cast<const double2 *>(f->chirp);
        double2 v[V];
        int t = first_point();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int k = t + T * i;
            v[i] = make_double2(0.0, 0.0);
            if (k < n) {
                const double2 x = KEEP ? get(k) : cconj(buf[k]);
                v[i] = cmulc(x, ch[k]);
            }
            few_loads(i);
        }
        convolve(v, reinterpret_cast<double *>(buf), f);
        if (KEEP || LDS) __syncthreads();
        t = first_point();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int k = t + T * i;
            if (k < n) {
                const double2 y = cmulc(v[i], ch[k]);
                if constexpr (KEEP) buf[k] = y;
                else put(k, cconj(y));
            }
            few_loads(i);
        }
        if (KEEP || LDS) __syncthreads();
    }
};

// The same interface over the engine of s2mi_fft.h: any length, rings of different ones.
struct LdsDft {
    static constexpr int MAXT = 1024, WPE = 4;
    static constexpr bool CONV = false;

    static __device__ __forceinline__ int slot(const FftArgs *f, int k) { return fft_slot(f, k); }
    static __device__ __forceinline__ int point(const FftArgs *f, int t) { return fft_place(f, t); }

    template <int SIGN, bool LDS, class Get, class Put>
    static __device__ __forceinline__ void dft(double2 *buf, const FftArgs *f, double2 *scr, Get get, Put put)
    {
        dft_lds<SIGN>(buf, f, scr, get, put);
    }
};

}  // namespace s2mi
