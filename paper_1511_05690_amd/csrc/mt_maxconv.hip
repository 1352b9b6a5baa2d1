// Max-convolution (Sec. 1) and the top k of x + y (Sec. 2.3) on FFT ring
// results.
//
// Estimate: z[t] = max_i x[i] y[t - i] from the norm sequence
// S_p[t] = (x'^p * y'^p)[t] with x' = x / max x, y' = y / max y (terms in
// [0, 1], the scaling of Sec. 2.1), computed by FFT convolution in FP64 (the
// fast ring kernel H, Sec. 2.1, whose threshold there is tau = 1e-12); per
// index the largest p of the family with S_p >= tau, and
// z = max x max y S_{p*}^(1/p*).
//
// LDS path (n + m - 1 <= 4096): a transform of N = max(16, 2^ceil(log2(n + m
// - 1))) points is done by N / 16 threads that hold 16 complex values each in
// registers (N = 4096: 256 threads, one pair per workgroup; smaller N packs
// 4096 / N pairs into a workgroup).  Passes are Stockham radix-16 (the last
// one radix 2, 4 or 8 when log2 N is not a multiple of 4), natural order in
// and out, through one LDS buffer per pair padded by one element every 16
// (the stride-16 writes of the first pass then hit distinct banks).
// Twiddles exp(-2 pi i m / N) come from one LDS table of cos and sin of
// 2 pi k / N for k <= N / 8 (the other octants by symmetry); a thread looks up
// w and w^4 of its butterflies once and forms the other powers by products.
// Per p, largest first:
//   forward: x'^p + i y'^p (x, y re-read per p, times 1 / max), so both real
//            transforms come out of one complex FFT;
//   product: thread t reads Z_t and Z_{N-t} and forms conj(W_t),
//            W = X Y with X_t = (Z_t + conj Z_{N-t}) / 2, Y_t = (Z_t - conj
//            Z_{N-t}) / 2i (the first pass of the inverse reads these pairs);
//   inverse: the forward FFT of conj(W), whose real part / N is S_p; the
//            last pass leaves S in registers at the positions the thread
//            owns, where the p* test runs.
// Indices decided at a larger p keep their S; a workgroup stops once every
// index of its pairs is decided, and the roots are taken once per index.
// When every index still open has at most kDirectTerms terms (they sit at
// the ends of the output, where few products meet), the workgroup finishes
// them by direct sums of x'^p y'^p for the remaining p instead of further
// transforms.
//
// Global path (n + m - 1 <= 16384): a four-step transform through a buffer in
// the workspace, three kernels per convolution, several p of the whole batch
// at a time.
//
// Top k of x + y: the ring results of both runs (y and y reversed) for every
// p by either path, the initial estimates, a one-wave NormQueue per run and
// the index pairing.
//
// Exact: z[t] = max_i x[i] y[t - i] by the definition, one thread per output
// index, products in the input precision.

#include <algorithm>
#include <atomic>
#include <climits>
#include <type_traits>

#include "mt_internal.h"

namespace mt {
namespace {

constexpr int kConvThreads = 256;  // kMaxConvN / 16
static_assert(kConvThreads * 16 == kMaxConvN, "16 values per thread at the largest N");
constexpr int kConvMinLog = 4;
// padded LDS elements per workgroup: one buffer of N + N / 16 per pair, 4096 / N pairs
constexpr int kConvLdsElems = kMaxConvN + kMaxConvN / 16;
// twiddle octant: cos and sin of 2 pi k / N, k = 0 .. N / 8
constexpr int kConvTwElems = kMaxConvN / 8 + 1;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// -i a
__device__ __forceinline__ double2 cmul_mi(double2 a) { return make_double2(a.y, -a.x); }

__device__ __forceinline__ double ipow_d(double v, int p) {
    double r = 1.0;
    while (p) {
        if (p & 1) r *= v;
        v *= v;
        p >>= 1;
    }
    return r;
}

// v[i] <- v[i]^p componentwise for the 16 values of a thread.  A power of two
// is one loop of squarings over all values (uniform, in place); other p go
// value by value (a second array of 16 would not fit beside the rest).  The
// same products in the same order as ipow_d either way.
__device__ __forceinline__ void pow_all(double2 (&v)[16], int p) {
    if ((p & (p - 1)) == 0) {
        for (int e = p; e > 1; e >>= 1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = make_double2(v[i].x * v[i].x, v[i].y * v[i].y);
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = make_double2(ipow_d(v[i].x, p), ipow_d(v[i].y, p));
}

__device__ __forceinline__ int padi(int i) { return i + (i >> 4); }

// An empty asm that claims to change v: values derived from it are then
// recomputed where they are used instead of being hoisted out of the p loop
// and held in registers for all of it.
__device__ __forceinline__ void opaque(double2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// cos(pi / 8), sin(pi / 8), sqrt(2) / 2
constexpr double kC8 = 0.92387953251128674;
constexpr double kS8 = 0.38268343236508978;
constexpr double kH = 0.70710678118654752;

__device__ __forceinline__ void dft4(double2& a0, double2& a1, double2& a2, double2& a3) {
    const double2 t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3), t3 = cmul_mi(csub(a1, a3));
    a0 = cadd(t0, t2);
    a1 = cadd(t1, t3);
    a2 = csub(t0, t2);
    a3 = csub(t1, t3);
}

// Forward DFT of the R values v[o + s * e], e = 0 .. R - 1, in place.  Output
// k ends in register o + s * oreg<R>(k).
template <int R>
__device__ __forceinline__ constexpr int oreg(int k) {
    if constexpr (R == 16) return (k >> 2) + 4 * (k & 3);
    if constexpr (R == 8) return 2 * (k & 3) + (k >> 2);
    return k;
}

template <int R>
__device__ __forceinline__ void dft(double2 (&v)[16], int o, int s) {
    if constexpr (R == 2) {
        const double2 a = v[o], b = v[o + s];
        v[o] = cadd(a, b);
        v[o + s] = csub(a, b);
    } else if constexpr (R == 4) {
        dft4(v[o], v[o + s], v[o + 2 * s], v[o + 3 * s]);
    } else if constexpr (R == 8) {
        // e = c + 2 n2, k = k1 + 4 k2: two DFT4 over n2, twiddle W8^(c k1), DFT2 over c
#pragma unroll
        for (int c = 0; c < 2; ++c) dft4(v[o + s * c], v[o + s * (c + 2)], v[o + s * (c + 4)], v[o + s * (c + 6)]);
        // u[c][k1] sits at c + 2 k1
        v[o + s * 3] = make_double2(kH * (v[o + s * 3].x + v[o + s * 3].y), kH * (v[o + s * 3].y - v[o + s * 3].x));
        v[o + s * 5] = cmul_mi(v[o + s * 5]);
        v[o + s * 7] = make_double2(kH * (v[o + s * 7].y - v[o + s * 7].x), -kH * (v[o + s * 7].x + v[o + s * 7].y));
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            const double2 a = v[o + s * (2 * k1)], b = v[o + s * (2 * k1 + 1)];
            v[o + s * (2 * k1)] = cadd(a, b);
            v[o + s * (2 * k1 + 1)] = csub(a, b);
        }
    } else {
        static_assert(R == 16, "radix 2, 4, 8 or 16");
        // e = c + 4 n2, k = k1 + 4 k2: four DFT4 over n2, twiddle W16^(c k1), four DFT4 over c
#pragma unroll
        for (int c = 0; c < 4; ++c) dft4(v[o + s * c], v[o + s * (c + 4)], v[o + s * (c + 8)], v[o + s * (c + 12)]);
        // u[c][k1] sits at c + 4 k1; W16^1 = (C, -S), ^2 = (H, -H), ^3 = (S, -C), ^4 = -i,
        // ^6 = (-H, -H), ^9 = (-C, S)
        const double2 w1 = make_double2(kC8, -kS8), w3 = make_double2(kS8, -kC8), w9 = make_double2(-kC8, kS8);
        v[o + s * 5] = cmul(v[o + s * 5], w1);                                                         // c1 k1 1
        v[o + s * 9] = make_double2(kH * (v[o + s * 9].x + v[o + s * 9].y), kH * (v[o + s * 9].y - v[o + s * 9].x));  // c1 k2
        v[o + s * 13] = cmul(v[o + s * 13], w3);                                                       // c1 k3
        v[o + s * 6] = make_double2(kH * (v[o + s * 6].x + v[o + s * 6].y), kH * (v[o + s * 6].y - v[o + s * 6].x));  // c2 k1
        v[o + s * 10] = cmul_mi(v[o + s * 10]);                                                        // c2 k2
        v[o + s * 14] = make_double2(kH * (v[o + s * 14].y - v[o + s * 14].x), -kH * (v[o + s * 14].x + v[o + s * 14].y));  // c2 k3
        v[o + s * 7] = cmul(v[o + s * 7], w3);                                                         // c3 k1
        v[o + s * 11] = make_double2(kH * (v[o + s * 11].y - v[o + s * 11].x), -kH * (v[o + s * 11].x + v[o + s * 11].y));  // c3 k2
        v[o + s * 15] = cmul(v[o + s * 15], w9);                                                       // c3 k3
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1)
            dft4(v[o + s * (4 * k1)], v[o + s * (4 * k1 + 1)], v[o + s * (4 * k1 + 2)], v[o + s * (4 * k1 + 3)]);
    }
}

template <int LOGN>
struct Fft {
    static constexpr int N = 1 << LOGN;
    static constexpr int T = N / 16;               // threads per pair
    static constexpr int G = kConvThreads / T;     // pairs per workgroup
    static constexpr int NP = N + N / 16;          // padded buffer
    static constexpr int NPASS = (LOGN + 3) / 4;
    static constexpr int radix(int pass) { return pass < LOGN / 4 ? 16 : (1 << (LOGN % 4)); }
    static constexpr int span(int pass) {
        int s = 1;
        for (int i = 0; i < pass; ++i) s *= radix(i);
        return s;
    }
};

// One Stockham pass on the thread's registers: butterfly g (j = tl + g T) takes
// the values at j + e N / R (registers g + e B), twiddles them by
// exp(-2 pi i k e / (Ns R)), k = j mod Ns, and transforms.
// exp(-2 pi i mm / N), 0 <= mm < N, from the octant table tw[k] = (cos, sin)(2 pi k / N):
// mm = q N / 4 + r gives (-i)^q w^r, and w^r = (-i) conj(w^(N/4 - r)) above N / 8.
template <int LOGN>
__device__ __forceinline__ double2 twiddle(const double2* tw, int mm) {
    constexpr int N4 = (1 << LOGN) / 4;
    const int q = mm / N4, r = mm & (N4 - 1);
    const bool refl = r > N4 / 2;
    const double2 t = tw[refl ? N4 - r : r];
    double a = refl ? t.y : t.x, b = refl ? -t.x : -t.y;
    if (q & 1) {
        const double c = a;
        a = b;
        b = -c;
    }
    if (q & 2) {
        a = -a;
        b = -b;
    }
    return make_double2(a, b);
}

// The thread's base twiddles, the same for every p and both directions:
// w1[PASS][g] = exp(-2 pi i k / (Ns R)) for butterfly g (k = j mod Ns) and
// w4[PASS][g] = its fourth power, looked up once (unused entries vanish).
template <int LOGN>
struct PassTwiddles {
    double2 w1[Fft<LOGN>::NPASS][16];
    double2 w4[Fft<LOGN>::NPASS][16];
};

template <int LOGN, int PASS>
__device__ __forceinline__ void load_twiddles(PassTwiddles<LOGN>& pt, int tl, const double2* tw) {
    using F = Fft<LOGN>;
    if constexpr (PASS < F::NPASS) {
        constexpr int R = F::radix(PASS), Ns = F::span(PASS), B = 16 / R;
#pragma unroll
        for (int g = 0; g < B; ++g) {
            const int j = tl + g * F::T;
            const int step = (j & (Ns - 1)) * (F::N / (Ns * R));
            pt.w1[PASS][g] = twiddle<LOGN>(tw, step);
            if constexpr (R >= 8) pt.w4[PASS][g] = twiddle<LOGN>(tw, 4 * step);
        }
        load_twiddles<LOGN, PASS + 1>(pt, tl, tw);
    }
}

// One Stockham pass on the thread's registers: butterfly g (j = tl + g T) takes
// the values at j + e N / R (registers g + e B), twiddles them by w^e,
// w = exp(-2 pi i k / (Ns R)), k = j mod Ns, and transforms.
template <int LOGN, int PASS>
__device__ __forceinline__ void pass_compute(double2 (&v)[16], const PassTwiddles<LOGN>& pt) {
    using F = Fft<LOGN>;
    constexpr int R = F::radix(PASS), Ns = F::span(PASS), B = 16 / R;
    if constexpr (Ns > 1) {
        // w^e from w and w^4 by at most three products each (about 10 ulp)
#pragma unroll
        for (int g = 0; g < B; ++g) {
            double2 w1 = pt.w1[PASS][g];
            opaque(w1);
            v[g + B] = cmul(v[g + B], w1);
            if constexpr (R >= 4) {
                const double2 w2 = cmul(w1, w1), w3 = cmul(w2, w1);
                v[g + 2 * B] = cmul(v[g + 2 * B], w2);
                v[g + 3 * B] = cmul(v[g + 3 * B], w3);
                if constexpr (R >= 8) {
                    double2 w4 = pt.w4[PASS][g];
                    opaque(w4);
                    const double2 w5 = cmul(w4, w1), w6 = cmul(w4, w2), w7 = cmul(w4, w3);
                    v[g + 4 * B] = cmul(v[g + 4 * B], w4);
                    v[g + 5 * B] = cmul(v[g + 5 * B], w5);
                    v[g + 6 * B] = cmul(v[g + 6 * B], w6);
                    v[g + 7 * B] = cmul(v[g + 7 * B], w7);
                    if constexpr (R == 16) {
                        const double2 w8 = cmul(w4, w4);
                        v[g + 8 * B] = cmul(v[g + 8 * B], w8);
                        v[g + 9 * B] = cmul(v[g + 9 * B], cmul(w8, w1));
                        v[g + 10 * B] = cmul(v[g + 10 * B], cmul(w8, w2));
                        v[g + 11 * B] = cmul(v[g + 11 * B], cmul(w8, w3));
                        v[g + 12 * B] = cmul(v[g + 12 * B], cmul(w8, w4));
                        v[g + 13 * B] = cmul(v[g + 13 * B], cmul(w8, w5));
                        v[g + 14 * B] = cmul(v[g + 14 * B], cmul(w8, w6));
                        v[g + 15 * B] = cmul(v[g + 15 * B], cmul(w8, w7));
                    }
                }
            }
        }
    }
#pragma unroll
    for (int g = 0; g < B; ++g) dft<R>(v, g, B);
}

// Output k of butterfly g goes to (j - k0) R + k0 + k Ns, k0 = j mod Ns.
// The padded index of base + k * stride for k = 0 .. 15, as padi(base) plus a
// constant where the stride is a multiple of 16 (or 1 with base a multiple of 16).
template <int STRIDE>
__device__ __forceinline__ int pad_step(int base_padded, int base, int k) {
    if constexpr (STRIDE % 16 == 0)
        return base_padded + k * (STRIDE / 16 * 17);
    else
        return padi(base + k * STRIDE);
}

template <int LOGN, int PASS>
__device__ __forceinline__ void pass_store(const double2 (&v)[16], int tl, double2* buf) {
    using F = Fft<LOGN>;
    constexpr int R = F::radix(PASS), Ns = F::span(PASS), B = 16 / R;
#pragma unroll
    for (int g = 0; g < B; ++g) {
        const int j = tl + g * F::T;
        const int k0 = j & (Ns - 1);
        const int base = (j - k0) * R + k0;
        const int bp = padi(base);
        if constexpr (Ns == 1 && R == 16) {
            // base = 16 j: the 16 outputs are contiguous after padding
#pragma unroll
            for (int k = 0; k < R; ++k) buf[bp + k] = v[g + B * oreg<R>(k)];
        } else {
#pragma unroll
            for (int k = 0; k < R; ++k) buf[pad_step<Ns>(bp, base, k)] = v[g + B * oreg<R>(k)];
        }
    }
}

// Every pass reads the thread's positions tl + i T into register i.
template <int LOGN>
__device__ __forceinline__ void pass_load(double2 (&v)[16], int tl, const double2* buf) {
    constexpr int TP = Fft<LOGN>::T;
    const int bp = padi(tl);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = buf[pad_step<TP>(bp, tl, i)];
}

// Passes 1 .. NPASS - 2 (or - 1): load, compute, barrier, store, barrier.
template <int LOGN, int PASS, int END>
__device__ __forceinline__ void middle_passes(double2 (&v)[16], int tl, double2* buf,
                                              const PassTwiddles<LOGN>& pt) {
    if constexpr (PASS < END) {
        pass_load<LOGN>(v, tl, buf);
        pass_compute<LOGN, PASS>(v, pt);
        __syncthreads();
        pass_store<LOGN, PASS>(v, tl, buf);
        __syncthreads();
        middle_passes<LOGN, PASS + 1, END>(v, tl, buf, pt);
    }
}

// Register holding position tl + i T after the last pass.
template <int LOGN>
__device__ __forceinline__ constexpr int last_reg(int i) {
    using F = Fft<LOGN>;
    constexpr int R = F::radix(F::NPASS - 1), B = 16 / R;
    return (i % B) + B * oreg<R>(i / B);
}

// Maxima of mx and my over the threads of one slot (contiguous lanes; several
// waves when TP > 64); red holds one pair per wave.
template <int TP>
__device__ __forceinline__ void slot_max(double& mx, double& my, double (*red)[kConvThreads / 64]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int d = (TP < 64 ? TP : 64) / 2; d >= 1; d >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, d));
        my = fmax(my, __shfl_xor(my, d));
    }
    if constexpr (TP > 64) {
        if (lane == 0) {
            red[0][wave] = mx;
            red[1][wave] = my;
        }
        __syncthreads();
        constexpr int WPI = TP / 64;
        const int w0 = (wave / WPI) * WPI;
#pragma unroll
        for (int w = 0; w < WPI; ++w) {
            mx = fmax(mx, red[0][w0 + w]);
            my = fmax(my, red[1][w0 + w]);
        }
    }
}

// The octant table cos / sin (2 pi k / N), k = 0 .. N / 8.
template <int LOGN>
__device__ __forceinline__ void build_twiddle_table(double2* tw) {
    constexpr int N = 1 << LOGN;
    for (int k = threadIdx.x; k <= N / 8; k += kConvThreads) {
        double sn, cs;
        sincospi(2.0 * (double)k / (double)N, &sn, &cs);
        tw[k] = make_double2(cs, sn);
    }
}

// One pair's convolution of the two real sequences held as v[i] = (a, b) at
// the thread's positions tl + i T (a = x'^p, b = y'^p, zero beyond the
// lists): the forward transform of a + i b, the product W = X Y formed from
// Z_t and Z_(N-t), and the inverse as the forward transform of conj(W).  On
// return v[last_reg(i)].x * 0.25 / N is (a * b)[tl + i T].  Every thread of
// the workgroup calls it (it holds barriers).
template <int LOGN>
__device__ __forceinline__ void convolve_pair(double2 (&v)[16], int tl, double2* buf,
                                              const PassTwiddles<LOGN>& pt) {
    using F = Fft<LOGN>;
    constexpr int N = F::N, TP = F::T;
    pass_compute<LOGN, 0>(v, pt);
    pass_store<LOGN, 0>(v, tl, buf);
    __syncthreads();
    middle_passes<LOGN, 1, F::NPASS>(v, tl, buf, pt);
    // conj(4 W_t), 4 W_t = (Z_t + conj Z_-t)(Z_t - conj Z_-t) / i
    const int bp = padi(tl), bn = padi(N - tl);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        int ik, in;
        if constexpr (TP % 16 == 0) {
            // t = tl + i TP > 0 for i > 0
            ik = bp + i * (TP / 16 * 17);
            in = i == 0 ? padi((N - tl) & (N - 1)) : bn - i * (TP / 16 * 17);
        } else {
            const int t = tl + i * TP;
            ik = padi(t);
            in = padi((N - t) & (N - 1));
        }
        const double2 zk = buf[ik], zn = buf[in];
        const double2 a = make_double2(zk.x + zn.x, zk.y - zn.y);
        const double2 c = make_double2(zk.y + zn.y, zn.x - zk.x);
        const double2 w = cmul(a, c);
        v[i] = make_double2(w.x, -w.y);
    }
    // the last pass leaves position tl + i TP in register last_reg(i)
    pass_compute<LOGN, 0>(v, pt);
    if constexpr (F::NPASS > 1) {
        __syncthreads();
        pass_store<LOGN, 0>(v, tl, buf);
        __syncthreads();
        middle_passes<LOGN, 1, F::NPASS - 1>(v, tl, buf, pt);
        pass_load<LOGN>(v, tl, buf);
        pass_compute<LOGN, F::NPASS - 1>(v, pt);
    }
}

// An open index with at most this many terms is finished by direct sums.
constexpr int kDirectTerms = 64;

// x^p for p >= 1 by binary powering (p uniform)
__device__ __forceinline__ double pow_int(double x, int p) {
    double r = 1.0;
    for (; p; p >>= 1) {
        if (p & 1) r *= x;
        x *= x;
    }
    return r;
}

template <typename T, int LOGN>
__global__ __launch_bounds__(kConvThreads, 2) void mt_maxconv_kernel(const T* __restrict__ x,
                                                                  const T* __restrict__ y, int64_t b, int64_t n,
                                                                  int64_t m, MaxconvSpec spec,
                                                                  T* __restrict__ z,
                                                                  uint8_t* __restrict__ pstar,
                                                                  unsigned long long* work) {
    using F = Fft<LOGN>;
    constexpr int N = F::N, TP = F::T;
    extern __shared__ double2 lds[];
    __shared__ double red[2][kConvThreads / 64];
    double2* tw = lds;  // kConvTwElems
    const int tid = threadIdx.x;
    if (work && tid == 0) timing_span_begin(work);
    const int slot = tid / TP, tl0 = tid % TP;
    const int64_t item = (int64_t)blockIdx.x * F::G + slot;
    const bool active = item < b;
    const int L = (int)(n + m - 1);
    double2* buf = lds + kConvTwElems + slot * F::NP;
    const T* xi = x + item * n;
    const T* yi = y + item * m;

    // the thread owns positions tl + i TP, i = 0 .. 15
    double mx = 0.0, my = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int t = tl0 + i * TP;
        if (active && t < n) mx = fmax(mx, (double)xi[t]);
        if (active && t < m) my = fmax(my, (double)yi[t]);
    }
    build_twiddle_table<LOGN>(tw);
    slot_max<TP>(mx, my, red);
    __syncthreads();
    PassTwiddles<LOGN> pt;
    load_twiddles<LOGN, 1>(pt, tl0, tw);
    const double rxy = mx * my;
    const double ix = mx > 0.0 ? 1.0 / mx : 0.0, iy = my > 0.0 ? 1.0 / my : 0.0;
    // 1 / N and the 1 / 4 of X Y (both halves carry 1 / 2)
    const double scale = 0.25 / (double)N;
    uint32_t decided = 0u;  // bit i: position tl + i TP
    double s_sel[16];       // S at the selected p
    uint32_t q_sel[4];      // its family index (byte i % 4 of word i / 4; MT_PSTAR_NONE if none stable)
#pragma unroll
    for (int i = 0; i < 16; ++i) s_sel[i] = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) q_sel[i] = 0u;
    int iters = 0;

    for (int q = spec.n - 1; q >= 0; --q) {
        ++iters;
        const int p = spec.p[q];
        // re-derive the addresses per p instead of holding them across the loop
        int tl = tl0;
        asm volatile("" : "+v"(tl));
        double2 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int t = tl + i * TP;
            const double a = (active && t < n) ? (double)xi[t] * ix : 0.0;
            const double c = (active && t < m) ? (double)yi[t] * iy : 0.0;
            v[i] = make_double2(a, c);
        }
        pow_all(v, p);
        convolve_pair<LOGN>(v, tl, buf, pt);
        // p* test: the first stable p from the top decides an index; the
        // smallest p decides what is left (its S, no p stable)
        int open = 0, open_far = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int t = tl + i * TP;
            const double S = v[last_reg<LOGN>(i)].x * scale;
            const bool live = active && t < L && !(decided & (1u << i));
            const bool stable = S >= spec.tau;
            const bool dec = live && (stable || q == 0);
            open |= live && !dec;
            // terms of index t: x[j] y[t - j] for max(0, t - m + 1) <= j <= min(t, n - 1)
            const int nterms = min(t, (int)n - 1) - max(0, t - (int)m + 1) + 1;
            open_far |= live && !dec && nterms > kDirectTerms;
            s_sel[i] = dec ? S : s_sel[i];
            const uint32_t code = stable ? (uint32_t)q : (uint32_t)MT_PSTAR_NONE;
            q_sel[i / 4] = dec ? (q_sel[i / 4] & ~(0xffu << (8 * (i % 4)))) | (code << (8 * (i % 4))) : q_sel[i / 4];
            decided |= dec ? 1u << i : 0u;
        }
        if (!__syncthreads_or(open)) break;
        if (!__syncthreads_or(open_far)) {
            // every open index has few terms: its S for the remaining p as a
            // direct sum (the exact S the transforms approximate), the same
            // selection.  x' and y' go to the pair's LDS buffer first (free
            // after the barrier above; n + m - 1 <= N doubles fit in it).
            double* sx = (double*)buf;
            double* sy = sx + n;
            for (int j = tl; j < (int)n; j += TP) sx[j] = active ? (double)xi[j] * ix : 0.0;
            for (int j = tl; j < (int)m; j += TP) sy[j] = active ? (double)yi[j] * iy : 0.0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int t = tl + i * TP;
                if (!(active && t < L && !(decided & (1u << i)))) continue;
                const int j0 = max(0, t - (int)m + 1), j1 = min(t, (int)n - 1);
                for (int qq = q - 1; qq >= 0; --qq) {
                    const int pp = spec.p[qq];
                    double S = 0.0;
                    for (int j = j0; j <= j1; ++j) S = fma(pow_int(sx[j], pp), pow_int(sy[t - j], pp), S);
                    const bool stable = S >= spec.tau;
                    if (!(stable || qq == 0)) continue;
                    s_sel[i] = S;
                    const uint32_t code = stable ? (uint32_t)qq : (uint32_t)MT_PSTAR_NONE;
                    q_sel[i / 4] = (q_sel[i / 4] & ~(0xffu << (8 * (i % 4)))) | (code << (8 * (i % 4)));
                    decided |= 1u << i;
                    break;
                }
            }
            // the roots below reuse the buffer
            __syncthreads();
            break;
        }
    }
    // roots, once per index: the selected S goes to the thread's own LDS
    // positions, then one index at a time (the buffer is free after the loop's
    // last barrier)
#pragma unroll
    for (int i = 0; i < 16; ++i) buf[padi(tl0 + i * TP)].x = s_sel[i];
    if (active) {
#pragma unroll 1
        for (int i = 0; i < 16; ++i) {
            const int t = tl0 + i * TP;
            if (t >= L) break;
            const double S = buf[padi(t)].x;
            const uint32_t code = (q_sel[i / 4] >> (8 * (i % 4))) & 0xffu;
            const int p = spec.p[code == MT_PSTAR_NONE ? 0 : code];
            double root = 0.0;
            if (S > 0.0) {
                if ((p & (p - 1)) == 0) {
                    root = S;
                    for (int e = p; e > 1; e >>= 1) root = sqrt(root);
                } else {
                    root = exp(log(S) / (double)p);
                }
            }
            z[item * L + t] = (T)(rxy * root);
            if (pstar) pstar[item * L + t] = (uint8_t)code;
        }
    }
    if (work) {
        // timed launch: two complex transforms per p, 5 N log2 N flops each
        // (the usual FFT count), and the end once every wave is done
        __syncthreads();
        if (tid == 0) {
            const int64_t pairs = b - (int64_t)blockIdx.x * F::G < F::G ? b - (int64_t)blockIdx.x * F::G : F::G;
            atomicAdd(work, (unsigned long long)iters * (unsigned long long)pairs * (10ull * N * LOGN));
            timing_span_end(work);
        }
    }
}

// Top k of x + y (Sec. 2.3).  The ring results sigma^(p) = x'^p * y'^p with
// x' = e^(x - max x), y' = e^(y - max y) (terms in (0, 1]), for every p of the
// family and both runs (run 0 with y, run 1 with y reversed): one convolution
// per slot, slot = run |P| + q.  sigma is (2, |P|, 2n - 1), FP64.
template <typename T, int LOGN>
__global__ __launch_bounds__(kConvThreads, 2) void mt_xy_sigma_kernel(const T* __restrict__ x,
                                                                   const T* __restrict__ y, int64_t n,
                                                                   MaxconvSpec spec, double* __restrict__ sigma) {
    using F = Fft<LOGN>;
    constexpr int N = F::N, TP = F::T;
    extern __shared__ double2 lds[];
    __shared__ double red[2][kConvThreads / 64];
    double2* tw = lds;  // kConvTwElems
    const int tid = threadIdx.x;
    const int slot = tid / TP, tl = tid % TP;
    const int item = (int)blockIdx.x * F::G + slot;
    const bool active = item < 2 * spec.n;
    const int run = active ? item / spec.n : 0, q = active ? item % spec.n : 0;
    const int L = (int)(2 * n - 1);
    double2* buf = lds + kConvTwElems + slot * F::NP;

    double mx = -INFINITY, my = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int t = tl + i * TP;
        if (active && t < n) {
            mx = fmax(mx, (double)x[t]);
            my = fmax(my, (double)y[t]);
        }
    }
    build_twiddle_table<LOGN>(tw);
    slot_max<TP>(mx, my, red);
    __syncthreads();
    PassTwiddles<LOGN> pt;
    load_twiddles<LOGN, 1>(pt, tl, tw);
    const int p = spec.p[q];
    double2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int t = tl + i * TP;
        double a = 0.0, c = 0.0;
        if (active && t < n) {
            a = exp((double)x[t] - mx);
            c = exp((double)y[run ? n - 1 - t : t] - my);
        }
        v[i] = make_double2(a, c);
    }
    pow_all(v, p);
    convolve_pair<LOGN>(v, tl, buf, pt);
    if (active) {
        double* out = sigma + ((int64_t)run * spec.n + q) * L;
        const double scale = 0.25 / (double)N;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int t = tl + i * TP;
            if (t < L) out[t] = v[last_reg<LOGN>(i)].x * scale;
        }
    }
}

// psi for every diagonal of both runs before any pop: the root at the largest
// p with sigma^(p)[m] >= tau, 0 if none.  One thread per (run, m).
__global__ __launch_bounds__(256) void mt_xy_psi_kernel(const double* __restrict__ sigma, int64_t L,
                                                       MaxconvSpec spec, double* __restrict__ psi) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= 2 * L) return;
    const int64_t run = g / L, m = g - run * L;
    const double* col = sigma + run * spec.n * L + m;
    double s[MT_MAX_P];
#pragma unroll
    for (int q = 0; q < MT_MAX_P; ++q) s[q] = q < spec.n ? col[q * L] : 0.0;
    int qh = -1;
#pragma unroll
    for (int q = 0; q < MT_MAX_P; ++q) qh = (q < spec.n && s[q] >= spec.tau) ? q : qh;
    double sh = 0.0;
#pragma unroll
    for (int q = 0; q < MT_MAX_P; ++q) sh = q == qh ? s[q] : sh;
    psi[g] = qh >= 0 ? pow(sh, 1.0 / (double)spec.p[qh]) : 0.0;
}

// ---- wave-wide argmax for the queues ----------------------------------
//
// DPP row shifts and row broadcasts (register moves between lanes, no LDS
// round trip) carry the maximum to lane 63 in six steps; lanes a move has no
// source for keep their own value, the identity of max.

template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_i32(int x) {
    return __builtin_amdgcn_update_dpp(x, x, kCtrl, kRowMask, 0xf, false);
}

template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_f64(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = dpp_i32<kCtrl, kRowMask>((int)b);
    const int hi = dpp_i32<kCtrl, kRowMask>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double readlane_f64(double x, int l) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// row_shr:1, 2, 4, 8 leave each row's maximum in its lane 15; row_bcast:15
// into rows 1 and 3 and row_bcast:31 into rows 2 and 3 bring all four to
// lane 63.
__device__ __forceinline__ double wave_max_f64(double m) {
    m = fmax(m, dpp_f64<0x111, 0xf>(m));
    m = fmax(m, dpp_f64<0x112, 0xf>(m));
    m = fmax(m, dpp_f64<0x114, 0xf>(m));
    m = fmax(m, dpp_f64<0x118, 0xf>(m));
    m = fmax(m, dpp_f64<0x142, 0xa>(m));
    m = fmax(m, dpp_f64<0x143, 0xc>(m));
    return readlane_f64(m, 63);
}

__device__ __forceinline__ int wave_min_i32(int m) {
    m = min(m, dpp_i32<0x111, 0xf>(m));
    m = min(m, dpp_i32<0x112, 0xf>(m));
    m = min(m, dpp_i32<0x114, 0xf>(m));
    m = min(m, dpp_i32<0x118, 0xf>(m));
    m = min(m, dpp_i32<0x142, 0xa>(m));
    m = min(m, dpp_i32<0x143, 0xc>(m));
    return __builtin_amdgcn_readlane(m, 63);
}

// The largest v over the wave and, among the lanes holding it, the smallest
// s; every lane receives both.  v must not be NaN.
__device__ __forceinline__ void wave_argmax(double& v, int& s) {
    const double vm = wave_max_f64(v);
    const uint64_t tied = __ballot(v == vm);
    if (__popcll(tied) == 1)
        s = __builtin_amdgcn_readlane(s, (int)__ffsll((unsigned long long)tied) - 1);
    else
        s = wave_min_i32(v == vm ? s : INT_MAX);
    v = vm;
}

constexpr int kQueueGroups = 16;

// The NormQueue of Sec. 2.3 for one run (block = run), one wave: psi[m] is the
// root at the largest stable p of diagonal m (0 if none); k times the largest
// psi (lowest m on ties) is reported as max x + max y + log(psi) and its
// diagonal, psi^p is subtracted from every sigma^(p)[m] (in place) and psi[m]
// is estimated again.  Within a pop the powers and roots go through one
// log psi (exp(p log psi), exp(log S / p)): the same values as pow to a few
// ulp, at half its cost on this serial path.
template <typename T>
__global__ __launch_bounds__(64) void mt_xy_queue_kernel(const T* __restrict__ x, const T* __restrict__ y,
                                                       int64_t n, MaxconvSpec spec, double* __restrict__ sigma,
                                                       const double* __restrict__ psi0, int32_t k,
                                                       double* __restrict__ values0,
                                                       double* __restrict__ values1, int32_t* __restrict__ diag0,
                                                       int32_t* __restrict__ diag1) {
    extern __shared__ double psi[];  // 2n - 1
    __shared__ double gv[64 * kQueueGroups];
    __shared__ int gm[64 * kQueueGroups];
    const int lane = threadIdx.x, run = blockIdx.x;
    const int L = (int)(2 * n - 1), np = spec.n;
    double* sg = sigma + (int64_t)run * np * L;
    double* values = run ? values1 : values0;
    int32_t* diag = run ? diag1 : diag0;

    double mx = -INFINITY, my = -INFINITY;
    for (int i = lane; i < n; i += 64) {
        mx = fmax(mx, (double)x[i]);
        my = fmax(my, (double)y[i]);
    }
    for (int d = 32; d >= 1; d >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, d));
        my = fmax(my, __shfl_xor(my, d));
    }
    const double shift = mx + my;
    for (int m = lane; m < L; m += 64) psi[m] = psi0[(int64_t)run * L + m];
    __syncthreads();
    // The lane owns m = lane + 64 c, c < C, in kQueueGroups groups of GS
    // consecutive c; gv / gm hold each group's largest psi and its m (lowest m
    // on ties), bv / bm the lane's.  A pop rescans one group.
    const int C = (L + 63) / 64;
    const int GS = (C + kQueueGroups - 1) / kQueueGroups;
    double* gvl = gv + lane * kQueueGroups;
    int* gml = gm + lane * kQueueGroups;
    auto group_scan = [&](int g) {
        double v = -1.0;
        int mm = L;
        const int c1 = (g + 1) * GS < C ? (g + 1) * GS : C;
        for (int c = g * GS; c < c1; ++c) {
            const int m = lane + 64 * c;
            if (m < L) {
                const double e = psi[m];
                if (e > v) {
                    v = e;
                    mm = m;
                }
            }
        }
        gvl[g] = v;
        gml[g] = mm;
    };
    double bv = -1.0;
    int bm = L;
    auto lane_best = [&]() {
        bv = -1.0;
        bm = L;
#pragma unroll
        for (int g = 0; g < kQueueGroups; ++g) {
            const double v = gvl[g];
            if (v > bv) {
                bv = v;
                bm = gml[g];
            }
        }
    };
    for (int g = 0; g < kQueueGroups; ++g) group_scan(g);
    lane_best();
    for (int r = 0; r < k; ++r) {
        double a = bv;
        int ms = bm;
        wave_argmax(a, ms);
        // log psi once for the value and every power (psi = 0: -inf, power 0)
        const double la = a > 0.0 ? log(a) : -INFINITY;
        if (lane == 0) {
            values[r] = shift + la;
            diag[r] = ms;
        }
        double s = 0.0;
        bool st = false;
        if (lane < np) {
            double* cell = sg + (int64_t)lane * L + ms;
            s = *cell - exp(la * (double)spec.p[lane]);
            *cell = s;
            st = s >= spec.tau;
        }
        const uint64_t mask = __ballot(st);
        double e = 0.0;
        if (mask) {
            const int qh = 63 - __clzll(mask);
            e = exp(log(__shfl(s, qh)) * (1.0 / (double)spec.p[qh]));
        }
        if (lane == 0) psi[ms] = e;
        __syncthreads();
        if (lane == (ms & 63)) {
            group_scan((ms >> 6) / GS);
            lane_best();
        }
    }
}

// Index recovery (Sec. 2.3): rank r has diagonal m1 = i + j in run 0 and
// anti-diagonal m2 = i + (n - 1 - j) in run 1, so i = (m1 + m2 - n + 1) / 2,
// j = m1 - i; -1 where that is not an integer pair in the n x n grid.
__global__ __launch_bounds__(256) void mt_xy_index_kernel(const int32_t* __restrict__ d0,
                                                         const int32_t* __restrict__ d1, int32_t k, int64_t n,
                                                         int32_t* __restrict__ diag, int32_t* __restrict__ ii,
                                                         int32_t* __restrict__ jj) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= k) return;
    const int64_t m1 = d0[r], m2 = d1[r];
    const int64_t sum = m1 + m2 - (n - 1);
    int64_t i = (sum & 1) == 0 ? sum / 2 : -1;
    int64_t j = i >= 0 ? m1 - i : -1;
    if (!(i >= 0 && i < n && j >= 0 && j < n)) i = j = -1;
    if (diag) diag[r] = (int32_t)m1;
    if (ii) ii[r] = (int32_t)i;
    if (jj) jj[r] = (int32_t)j;
}

// ---- the paired queue (Discussion) -------------------------------------
//
// Within k pops a run only ever pops diagonals among the K = min(k, 2n - 1)
// largest initial estimates (lowest m on ties): an estimate changes only
// when its diagonal is popped, so a diagonal's first pop takes the largest
// never-popped estimate, and at most k diagonals are popped.  The paired
// queue therefore works on those K candidates per run, held in LDS.

constexpr int kSelThreads = 1024;
constexpr int kSelPer = kLongConvN / kSelThreads;  // covers 2n - 1 < kLongConvN

// The K candidates of each run (block = run): the K largest psi, lowest m
// on ties, written in ascending m.  psi >= 0, so its bit pattern orders as
// its value; the K-th largest key is found by counting the keys (held in
// registers) at or above a threshold by ballots until exactly K are, then the
// keys above it and the first keys equal to it (in m order) are kept.  An
// 8-bit radix select spent its time on LDS atomics of neighbouring
// keys to the same bin: 42 us at L = 16383,
// K = 256, |P| = 24, now 21 and 5 for the columns.
__global__ __launch_bounds__(kSelThreads) void mt_xy_select_kernel(const double* __restrict__ psi, int L, int K,
                                                                   int32_t* __restrict__ cand_m,
                                                                   double* __restrict__ cand_psi) {
    __shared__ int wcount[2][kSelThreads / 64];
    __shared__ uint64_t wtop[kSelThreads / 64];
    __shared__ uint32_t wtot[kSelThreads / 64];
    const int tid = threadIdx.x, run = blockIdx.x, lane = tid & 63, wave = tid >> 6;
    const double* ps = psi + (int64_t)run * L;
    uint64_t key[kSelPer];
    // lane l of a wave owns m = m0 + 64 c
    const int m0 = 64 * kSelPer * wave + lane;
#pragma unroll
    for (int c = 0; c < kSelPer; ++c) {
        const int m = m0 + 64 * c;
        key[c] = m < L ? (uint64_t)__double_as_longlong(ps[m]) : 0ull;
    }
    // the largest threshold with at least K keys at or above it: from the
    // largest key down in steps that grow until K keys are there, then bit by
    // bit up again, until exactly K are
    uint64_t top = 0;
#pragma unroll
    for (int c = 0; c < kSelPer; ++c) top = key[c] > top ? key[c] : top;
    for (int d = 32; d >= 1; d >>= 1) {
        const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)top, d);
        top = o > top ? o : top;
    }
    if (lane == 0) wtop[wave] = top;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSelThreads / 64; ++w) top = wtop[w] > top ? wtop[w] : top;
    uint64_t at = 0;
    bool exact = false;
    int step = 0;
    auto enough = [&](uint64_t cand) {
        int n = 0;
#pragma unroll
        for (int c = 0; c < kSelPer; ++c) n += (int)__popcll(__ballot(m0 + 64 * c < L && key[c] >= cand));
        int* counts = wcount[step++ & 1];
        if (lane == 0) counts[wave] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int w = 0; w < kSelThreads / 64; ++w) n += counts[w];
        if (n >= K) at = cand;
        exact = n == K;
        return n >= K;
    };
    // psi >= 0 as bits: one part in 2^7 of a value is 2^45 ... 2^46
    int bit = 46;
    while (bit < 64 && top >> bit != 0 && !enough(top + 1 - (1ull << bit))) bit += 2;
    // at + 2^bit - 1 >= top, so the threshold is in the bits below
    for (bit = bit < 64 ? bit : 64; bit > 0 && !exact;) {
        --bit;
        const uint64_t cand = at + (1ull << bit);
        if (cand > at && cand <= top) enough(cand);
    }
    // exactly K keys from the threshold up: all of them, none left to ties
    const uint64_t prefix = exact && at > 0 ? at - 1 : at;
    // keys above the threshold, and the first `need` keys equal to it in m
    // order: the waves' counts (above | equal << 16), then ballots
    uint32_t count = 0;
#pragma unroll
    for (int c = 0; c < kSelPer; ++c) {
        const bool ok = m0 + 64 * c < L;
        count += (uint32_t)__popcll(__ballot(ok && key[c] > prefix)) |
                 (uint32_t)__popcll(__ballot(ok && key[c] == prefix)) << 16;
    }
    if (lane == 0) wtot[wave] = count;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / 64; ++w) {
        before += w < wave ? wtot[w] : 0u;
        total += wtot[w];
    }
    const int need = K - (int)(total & 0xffffu);
    int gt_before = (int)(before & 0xffffu), eq_before = (int)(before >> 16);
    const uint64_t below = (1ull << lane) - 1;
#pragma unroll
    for (int c = 0; c < kSelPer; ++c) {
        const int m = m0 + 64 * c;
        const bool ok = m < L;
        const bool gt = ok && key[c] > prefix, eq = ok && key[c] == prefix;
        const uint64_t gts = __ballot(gt), eqs = __ballot(eq);
        const int eq_rank = eq_before + (int)__popcll(eqs & below);
        const int pos = gt_before + (int)__popcll(gts & below) + (eq_rank < need ? eq_rank : need);
        if ((gt || (eq && eq_rank < need)) && pos < K) {
            cand_m[(int64_t)run * K + pos] = m;
            cand_psi[(int64_t)run * K + pos] = ps[m];
        }
        gt_before += (int)__popcll(gts);
        eq_before += (int)__popcll(eqs);
    }
}

// The candidates' columns, cand_cols[(run np + q) K + slot]: a kernel of its
// own, for the cells lie a cache line apart each and one compute unit has too
// few of them on their way.
__global__ __launch_bounds__(256) void mt_xy_gather_kernel(const double* __restrict__ sigma, int L, int K, int np,
                                                           const int32_t* __restrict__ cand_m,
                                                           double* __restrict__ cand_cols) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= 2 * np * K) return;
    const int row = u / K, slot = u - row * K;
    cand_cols[u] = sigma[(int64_t)row * L + cand_m[(row >= np ? K : 0) + slot]];
}

__device__ __forceinline__ int diag_len(int m, int n) { return (m < 2 * n - 2 - m ? m : 2 * n - 2 - m) + 1; }

// A lane's candidate slots held in registers (slot u * 32 + q of its run in
// entry u, q = lane % 32; entries beyond K are -inf): the largest log psi,
// the first slot on ties and all -inf (K on a lane without slots).
template <int kS>
__device__ __forceinline__ void slots_best(const double (&rv)[kS], const int (&rm)[kS], int q, int K, double& bv,
                                           int& bs, int& bm) {
    bv = rv[0];
    bs = q < K ? q : K;
    bm = rm[0];
#pragma unroll
    for (int u = 1; u < kS; ++u) {
        const bool more = rv[u] > bv;
        bv = more ? rv[u] : bv;
        bs = more ? u * 32 + q : bs;
        bm = more ? rm[u] : bm;
    }
}

template <int kS>
__device__ __forceinline__ void slots_set(double (&rv)[kS], int u, double e) {
#pragma unroll
    for (int w = 0; w < kS; ++w) rv[w] = w == u ? e : rv[w];
}

// The largest v of each half wave (lanes 0..31 and 32..63) and, among the
// lanes of that half holding it, the smallest s: row_shr 1, 2, 4, 8 leave
// each row's maximum in its lane 15, row_bcast:15 into rows 1 and 3 brings
// the two rows of a half together in lanes 31 and 63.  v must not be NaN.
__device__ __forceinline__ void half_argmax(double v, int s, double& a0, int& s0, double& a1, int& s1) {
    // fmax without its quieting of the operands
    auto max2 = [](double a, double b) {
        double r;
        asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
        return r;
    };
    double m = v;
    m = max2(m, dpp_f64<0x111, 0xf>(m));
    m = max2(m, dpp_f64<0x112, 0xf>(m));
    m = max2(m, dpp_f64<0x114, 0xf>(m));
    m = max2(m, dpp_f64<0x118, 0xf>(m));
    m = max2(m, dpp_f64<0x142, 0xa>(m));
    a0 = readlane_f64(m, 31);
    a1 = readlane_f64(m, 63);
    const bool tie = v == ((threadIdx.x & 32) ? a1 : a0);
    const uint64_t t = __ballot(tie);
    const uint32_t t0 = (uint32_t)t, t1 = (uint32_t)(t >> 32);
    if (__popc(t0) == 1 && __popc(t1) == 1) {
        s0 = __builtin_amdgcn_readlane(s, __ffs(t0) - 1);
        s1 = __builtin_amdgcn_readlane(s, 32 + __ffs(t1) - 1);
        return;
    }
    int w = tie ? s : INT_MAX;
    w = min(w, dpp_i32<0x111, 0xf>(w));
    w = min(w, dpp_i32<0x112, 0xf>(w));
    w = min(w, dpp_i32<0x114, 0xf>(w));
    w = min(w, dpp_i32<0x118, 0xf>(w));
    w = min(w, dpp_i32<0x142, 0xa>(w));
    s0 = __builtin_amdgcn_readlane(w, 31);
    s1 = __builtin_amdgcn_readlane(w, 63);
}

// Both runs' NormQueues in lockstep, one wave, over the candidates: each
// rank pops run 0 (diagonals i + j) and run 1 (anti-diagonals
// i + n - 1 - j) together.  Plain (Sec. 2.3): each run subtracts its own
// estimate and the indices are recovered from the two diagonals.  Paired
// (Discussion): the pair (i, j) the two diagonals meet in is accurate when it
// lies in the grid, no earlier rank reported it (a list in LDS, scanned by
// every lane), and its scaled value v = e^(x_i - max x + y_j - max y) is at
// least psi len^(-1/p*) on both diagonals (the smallest largest term their
// norms admit; none on a diagonal without a stable p); an accurate rank
// reports x_i + y_j and (i, j) and subtracts v^p from both runs, any other
// reports run 0's estimate and i = j = -1, and each run subtracts its own
// estimate.  Lanes 0..31 hold run 0's powers and candidates, lanes 32..63
// run 1's; candidate slot s of run t belongs to lane 32 t + s % 32.  The
// candidates' sigma
// columns are updated in LDS when they fit (kColsLds), else in the
// workspace copy; with kRegS > 0 (K <= 32 kRegS) a lane's slots, estimates
// and diagonals, stay in registers.  The log diagonal lengths of the paired
// acceptance test are kept in LDS when they fit (kLenLds), else taken from
// the popped diagonals each rank (the same values).
//
// A rank is one dependent chain (argmax, x_i and y_j, exp, log, rescan) on one
// wave, so it costs its latencies: the chain has no branches (selects instead,
// results stored every 64 ranks, the first 64 kDoneRegs reported pairs
// compared in registers).  The other waves of the block only help to fill
// LDS.  n = 8192, K = k = 256, |P| = 24, paired: 498 -> 289 us, of which
// filling LDS was 80 with one wave.
constexpr int kLockThreads = 512;
constexpr int kDoneRegs = 4;  // x 64 lanes
template <typename T, bool kPaired, bool kColsLds, int kRegS, bool kLenLds>
__global__ __launch_bounds__(kLockThreads) void mt_xy_lockstep_kernel(const T* __restrict__ x, const T* __restrict__ y,
                                                          int64_t n, MaxconvSpec spec,
                                                          const int32_t* __restrict__ cand_m,
                                                          const double* __restrict__ cand_psi,
                                                          double* __restrict__ cand_cols, int K, int32_t k,
                                                          double* __restrict__ values, int32_t* __restrict__ diag,
                                                          int32_t* __restrict__ anti, int32_t* __restrict__ ii,
                                                          int32_t* __restrict__ jj) {
    // LDS: 2K log estimates, [2K log diagonal lengths], [2 np K column
    // cells], 2K diagonals, [k reported pairs (paired)].  The queue keeps log psi: the argmax
    // order is psi's, the reported value needs the log, the subtraction
    // exp(p log psi) and the new root exp(log S / p) then need no log or exp
    // of their own.
    extern __shared__ double cv[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int np = spec.n, nn = (int)n;
    constexpr int kLen = kPaired && kLenLds ? 1 : 0;
    double* cl = cv + 2 * K;  // used when kLen
    double* cols = kColsLds ? cv + (2 + 2 * kLen) * K : cand_cols;
    int* cm = (int*)(cv + (2 + 2 * kLen) * K + (kColsLds ? 2 * np * K : 0));
    int* done = cm + 2 * K;  // paired only
    int n_done = 0;
    double mx = -INFINITY, my = -INFINITY;
#pragma unroll 8
    for (int i = tid; i < nn; i += kLockThreads) {
        mx = fmax(mx, (double)x[i]);
        my = fmax(my, (double)y[i]);
    }
    for (int d = 32; d >= 1; d >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, d));
        my = fmax(my, __shfl_xor(my, d));
    }
    constexpr int kWaves = kLockThreads / 64;
    if (lane == 0) {
        cv[tid >> 6] = mx;
        cv[kWaves + (tid >> 6)] = my;
    }
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) {
        mx = fmax(mx, cv[w]);
        my = fmax(my, cv[kWaves + w]);
    }
    __syncthreads();
    const double shift = mx + my;
    for (int s = tid; s < 2 * K; s += kLockThreads) {
        const double e = cand_psi[s];
        const int m = cand_m[s];
        cv[s] = e > 0.0 ? log(e) : -INFINITY;
        if (kLen) cl[s] = log((double)diag_len(m, nn));
        cm[s] = m;
    }
    if (kColsLds)
#pragma unroll 8
        for (int s = tid; s < 2 * np * K; s += kLockThreads) cols[s] = cand_cols[s];
    __syncthreads();
    if (tid >= 64) return;
    const int half = lane >> 5, q = lane & 31;
    const int S = (K + 31) / 32;
    // the lane's largest log psi of its run and its slot (the first valid
    // slot always counts, so a run whose estimates are all -inf still names
    // its lowest)
    auto lane_best = [&](double& bv, int& bs) {
        bv = -INFINITY;
        bs = K;
        for (int u = 0; u < S; ++u) {
            const int s = u * 32 + q;
            if (s < K) {
                const double e = cv[half * K + s];
                if (bs == K || e > bv) {
                    bv = e;
                    bs = s;
                }
            }
        }
    };
    constexpr int kSR = kRegS > 0 ? kRegS : 1;
    double rv[kSR];
    int rm[kSR];
    double bv;
    int bs, bm;
    if (kRegS > 0) {
#pragma unroll
        for (int u = 0; u < kSR; ++u) {
            const int s = u * 32 + q;
            rv[u] = s < K ? cv[half * K + s] : -INFINITY;
            rm[u] = s < K ? cm[half * K + s] : 0;
        }
        slots_best(rv, rm, q, K, bv, bs, bm);
    } else {
        lane_best(bv, bs);
        bm = bs < K ? cm[half * K + bs] : 0;
    }
    const bool mine = q < np;
    // this lane's power and its reciprocal; a rank picks other lanes' by readlane
    const double pw = mine ? (double)spec.p[q] : 1.0, ipw = 1.0 / pw;
    // the reported pairs: the first 64 kDoneRegs in registers, the rest in LDS
    int dr[kDoneRegs];
#pragma unroll
    for (int w = 0; w < kDoneRegs; ++w) dr[w] = -1;
    // rank r's results wait in lane r % 64 for the last of 64 ranks
    double out_v = 0.0;
    int out_m1 = 0, out_m2 = 0, out_i = -1, out_j = -1;
    for (int r = 0; r < k; ++r) {
        double a0, a1;
        int s0, s1;
        half_argmax(bv, bs, a0, s0, a1, s1);
        const int m1 = __builtin_amdgcn_readlane(bm, s0 & 31), m2 = __builtin_amdgcn_readlane(bm, 32 + (s1 & 31));
        const int sd = m1 + m2 - (nn - 1);
        const int i = sd >> 1, j = m1 - i;
        bool valid = (sd & 1) == 0 && sd >= 0 && i < nn && j >= 0 && j < nn;
        double xi = 0.0, yj = 0.0, lv = 0.0;
        if (kPaired) {
            xi = (double)x[valid ? i : 0];
            yj = (double)y[valid ? j : 0];
        }
        double* cp = cols + (half * np + (mine ? q : 0)) * K + (half ? s1 : s0);
        const double cell = *cp;
        const double la0 = a0, la1 = a1;
        bool acc = false;
        const int id = i * nn + j;
        if (kPaired) {
            bool seen = false;
#pragma unroll
            for (int w = 0; w < kDoneRegs; ++w) seen |= dr[w] == id;
            for (int u = 64 * kDoneRegs + lane; u < n_done; u += 64) seen |= done[u] == id;
            valid = valid && __ballot(seen) == 0;
            const uint64_t st = __ballot(mine && cell >= spec.tau);
            const uint32_t lo_b = (uint32_t)st, hi_b = (uint32_t)(st >> 32);
            const int q0 = lo_b ? 31 - __clz(lo_b) : -1, q1 = hi_b ? 31 - __clz(hi_b) : -1;
            // in logs: log v >= log psi - log(len) / p* on both diagonals
            lv = (xi - mx) + (yj - my);
            const double ll0 = kLen ? cl[s0] : log((double)diag_len(m1, nn));
            const double ll1 = kLen ? cl[K + s1] : log((double)diag_len(m2, nn));
            const double i0 = readlane_f64(ipw, q0 >= 0 ? q0 : 0), i1 = readlane_f64(ipw, q1 >= 0 ? 32 + q1 : 32);
            acc = valid & (q0 >= 0) & (q1 >= 0) & (lv >= la0 - ll0 * i0) & (lv >= la1 - ll1 * i1);
        }
        const double la = acc ? lv : (half ? la1 : la0);
        const double s = cell - exp(la * pw);
        if (mine) *cp = s;
        const uint64_t nm = __ballot(mine && s >= spec.tau);
        const uint32_t nlo = (uint32_t)nm, nhi = (uint32_t)(nm >> 32);
        const int h0 = nlo ? 31 - __clz(nlo) : -1, h1 = nhi ? 31 - __clz(nhi) : -1;
        const int l0 = h0 >= 0 ? h0 : 0, l1 = h1 >= 0 ? 32 + h1 : 32;
        // both runs' new roots in one log: half 0 takes run 0's sum, half 1 run 1's
        double sv0 = readlane_f64(s, l0), sv1 = readlane_f64(s, l1);
        double iv0 = readlane_f64(ipw, l0), iv1 = readlane_f64(ipw, l1);
        asm volatile("" : "+v"(sv0), "+v"(sv1), "+v"(iv0), "+v"(iv1));  // selects, no branches
        const double sh = half ? sv1 : sv0, ih = half ? iv1 : iv0;
        const double lr = log(sh) * ih;
        const double e = (half ? h1 : h0) >= 0 ? lr : -INFINITY;
        const bool give = kPaired ? acc : valid;
        if (lane == (r & 63)) {
            out_v = acc ? xi + yj : shift + la0;
            out_m1 = m1;
            out_m2 = m2;
            out_i = give ? i : -1;
            out_j = give ? j : -1;
        }
        if ((r & 63) == 63 || r == k - 1) {
            const int at = r - (r & 63) + lane;
            if (at <= r) {
                values[at] = out_v;
                if (diag) diag[at] = out_m1;
                anti[at] = out_m2;
                if (ii) ii[at] = out_i;
                if (jj) jj[at] = out_j;
            }
        }
        if (kPaired && acc && n_done >= 64 * kDoneRegs && lane == 0) done[n_done] = id;
        if (kPaired && acc) {
#pragma unroll
            for (int w = 0; w < kDoneRegs; ++w) dr[w] = n_done == 64 * w + lane ? id : dr[w];
        }
        n_done += acc ? 1 : 0;
        // the owner of each popped slot (one lane per half) takes its new
        // estimate and rescans its slots
        const int so = half ? s1 : s0;
        if (kRegS > 0) {
            slots_set(rv, q == (so & 31) ? so >> 5 : -1, e);
            slots_best(rv, rm, q, K, bv, bs, bm);
        } else if (q == (so & 31)) {
            cv[half * K + so] = e;
            lane_best(bv, bs);
            bm = cm[half * K + bs];
        }
    }
}

// Long transforms (N = 8192 or 16384, up to kLongConvN): the batch in one
// global buffer [slot][N], each direction a four-step transform (N = 128 N2,
// N2 = 64 or 128): with n = N2 n1 + n2 and k = k1 + 128 k2,
//   X[k] = sum_n2 W_N2^(n2 k2) W_N^(n2 k1) sum_n1 x[N2 n1 + n2] W_128^(n1 k1),
// the columns (length 128, stride N2), the twiddles W_N^(n2 k1), then the
// rows (length N2).  A convolution is three kernels:
//   columns  forms the operands, transforms them, stores Y[k1 N2 + n2];
//   middle   the rows k1 of Y, the product, and the inverse's columns;
//   rows     the inverse's rows, and what is done with the result.
// The middle kernel can go on because the product at k needs Z[k] and Z[N - k]
// only, and the inverse's column n2 is made of the elements k = n2 mod N2,
// whole forward rows: a set of rows closed under k1 -> -k1 (and, for N2 = 64,
// k1 -> k1 + 64) is a set of whole columns.  It reads and writes the same
// 1024 elements, so the buffer is transformed in place (f4_place).
// Bound by the buffer's traffic: 2 reads and 2 writes per element and
// convolution.  As seven kernels per p (load, two passes, product, two
// passes, select: 6 reads and 6 writes), one p at a time, 48 pairs at
// N = 16384 over 7 p took 489 us in 53 launches, now 107 in 7: columns 38,
// middle 43, rows 28 (4.9 TB/s each way through the buffer in the middle).
constexpr int kF4Lines = 8;
constexpr int kF4Threads = 128;
constexpr int kF4Stride = 137;  // a line of 128 padded by padi, odd: no bank conflicts across lines

// exp(-2 pi i mm / N), 0 <= mm < N, from the octant table (runtime N, N4 = N / 4).
__device__ __forceinline__ double2 twiddle_rt(const double2* tw, int mm, int N4) {
    const int q = mm / N4, r = mm & (N4 - 1);
    const bool refl = r > N4 / 2;
    const double2 t = tw[refl ? N4 - r : r];
    double a = refl ? t.y : t.x, b = refl ? -t.x : -t.y;
    if (q & 1) {
        const double c = a;
        a = b;
        b = -c;
    }
    if (q & 2) {
        a = -a;
        b = -b;
    }
    return make_double2(a, b);
}

// cmul with its contraction written out: where the compiler knows the octant
// of a twiddle it turns the sign into an addition and fuses the other product.
__device__ __forceinline__ double2 cmul_fma(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

// Block `blk` of the octant table: cos / sin (2 pi k / N), k = 0 .. N / 8.
__device__ __forceinline__ void twiddle_block(double2* tw, int N, int blk) {
    const int k = blk * (int)blockDim.x + (int)threadIdx.x;
    if (k > N / 8) return;
    double sn, cs;
    sincospi(2.0 * (double)k / (double)N, &sn, &cs);
    tw[k] = make_double2(cs, sn);
}
constexpr int kLongSetupThreads = 1024;
inline unsigned twiddle_blocks(int N) { return (unsigned)(N / 8 / kLongSetupThreads + 1); }

// Maxima of mx and my over the block, in every lane of the first wave.
__device__ __forceinline__ void block_max2(double& mx, double& my) {
    __shared__ double red[2][kLongSetupThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int d = 32; d >= 1; d >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, d));
        my = fmax(my, __shfl_xor(my, d));
    }
    if (lane == 0) {
        red[0][wave] = mx;
        red[1][wave] = my;
    }
    __syncthreads();
    for (int w = 0; w < kLongSetupThreads / 64; ++w) {
        mx = fmax(mx, red[0][w]);
        my = fmax(my, red[1][w]);
    }
}

// Block 0: the maxima of x and y in mxy[0], mxy[1]; the others: the twiddles.
template <typename T>
__global__ __launch_bounds__(kLongSetupThreads) void mt_xy_long_setup_kernel(const T* __restrict__ x,
                                                                            const T* __restrict__ y, int64_t n, int N,
                                                                            double2* __restrict__ tw,
                                                                            double* __restrict__ mxy) {
    if (blockIdx.x > 0) {
        twiddle_block(tw, N, (int)blockIdx.x - 1);
        return;
    }
    double mx = -INFINITY, my = -INFINITY;
    for (int64_t i = threadIdx.x; i < n; i += kLongSetupThreads) {
        mx = fmax(mx, (double)x[i]);
        my = fmax(my, (double)y[i]);
    }
    block_max2(mx, my);
    if (threadIdx.x == 0) {
        mxy[0] = mx;
        mxy[1] = my;
    }
}

// Block pair < b: rxy[pair] = max x max y, inv[2 pair] = 1 / max x,
// inv[2 pair + 1] = 1 / max y, open_at[pair] = 0; the others: the twiddles.
template <typename T>
__global__ __launch_bounds__(kLongSetupThreads) void mt_maxconv_long_setup_kernel(
    const T* __restrict__ x, const T* __restrict__ y, int64_t b, int64_t n, int64_t m, int N,
    double2* __restrict__ tw, double* __restrict__ rxy, double* __restrict__ inv, int* __restrict__ open_at) {
    const int64_t pair = blockIdx.x;
    if (pair >= b) {
        twiddle_block(tw, N, (int)(pair - b));
        return;
    }
    double mx = 0.0, my = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kLongSetupThreads) mx = fmax(mx, (double)x[pair * n + i]);
    for (int64_t i = threadIdx.x; i < m; i += kLongSetupThreads) my = fmax(my, (double)y[pair * m + i]);
    block_max2(mx, my);
    if (threadIdx.x == 0) {
        rxy[pair] = mx * my;
        inv[2 * pair] = mx > 0.0 ? 1.0 / mx : 0.0;
        inv[2 * pair + 1] = my > 0.0 ? 1.0 / my : 0.0;
        open_at[pair] = 0;
    }
}

// The operands of the max-convolution: slot s of a chunk holds family index
// q_top - s / b of pair s % b, (x'^p, y'^p), zero beyond the vectors.  A pair
// without an open index after the chunk before (open_at[pair] != chunk) is
// not transformed.
template <typename T>
struct MaxconvLoad {
    const T* x;
    const T* y;
    int64_t b, n, m;
    const double* inv;
    const int* open_at;
    int chunk, q_top;
    MaxconvSpec spec;
    __device__ __forceinline__ bool live(int64_t s) const { return open_at[s % b] == chunk; }
    __device__ __forceinline__ double2 at(int64_t s, int t) const {
        const int64_t pair = s % b;
        const int p = spec.p[q_top - (int)(s / b)];
        const double a = t < n ? ipow_d((double)x[pair * n + t] * inv[2 * pair], p) : 0.0;
        const double c = t < m ? ipow_d((double)y[pair * m + t] * inv[2 * pair + 1], p) : 0.0;
        return make_double2(a, c);
    }
};

// The operands of x + y: slot = run |P| + q holds (x'^p, y'^p), y reversed in
// run 1, zero for t >= n.
template <typename T>
struct XyLoad {
    const T* x;
    const T* y;
    int64_t n;
    const double* mxy;
    MaxconvSpec spec;
    __device__ __forceinline__ bool live(int64_t) const { return true; }
    __device__ __forceinline__ double2 at(int64_t s, int t) const {
        const int run = (int)s / spec.n, p = spec.p[(int)s % spec.n];
        double a = 0.0, c = 0.0;
        if (t < n) {
            a = ipow_d(exp((double)x[t] - mxy[0]), p);
            c = ipow_d(exp((double)y[run ? n - 1 - t : t] - mxy[1]), p);
        }
        return make_double2(a, c);
    }
};

// The two Stockham stages of a line of M = 64 or 128 points (radix 16, then
// M / 16).  First: v[e] is element j + e M / 16, j < M / 16; the result goes
// to the line in LDS.  Second: lane j < 16 of the line; result k = j + 16 e is
// left in v[oreg<M / 16>(e)].
__device__ __forceinline__ void f4_first(double2 (&v)[16], double2* line, int j) {
    dft<16>(v, 0, 1);
#pragma unroll
    for (int e = 0; e < 16; ++e) line[padi(16 * j + e)] = v[oreg<16>(e)];
}

template <int M>
__device__ __forceinline__ void f4_second(double2 (&v)[16], const double2* line, int j, int N, const double2* tw) {
    constexpr int R = M / 16;
#pragma unroll
    for (int e = 0; e < R; ++e) v[e] = line[padi(j + 16 * e)];
    const int step = j * (N / M);
#pragma unroll
    for (int e = 1; e < R; ++e) v[e] = cmul_fma(v[e], twiddle_rt(tw, step * e, N / 4));
    dft<R>(v, 0, 1);
}

// Where the middle kernel leaves element k1 of the inverse's column n2: in
// the forward rows n2 (and n2 + 64 for N2 = 64) that it read.
template <int N2>
__device__ __forceinline__ int f4_place(int n2, int k1) {
    return (n2 + N2 * (k1 / N2)) * N2 + (k1 & (N2 - 1));
}

// Workgroup g: transform g / (N2 / 8), columns 8 (g % (N2 / 8)) ...  Lanes run
// over the 8 columns first: 8 consecutive elements per access.
template <int N2, typename Load>
__global__ __launch_bounds__(kF4Threads) void mt_long_columns_kernel(Load ld, double2* __restrict__ buf,
                                                                    const double2* __restrict__ tw) {
    __shared__ double2 lds[kF4Lines * kF4Stride];
    constexpr int N = 128 * N2, kGroups = N2 / kF4Lines;
    const int64_t slot = blockIdx.x / kGroups;
    if (!ld.live(slot)) return;
    const int t = threadIdx.x, c = t & (kF4Lines - 1), j = t / kF4Lines;
    const int n2 = (int)(blockIdx.x & (kGroups - 1)) * kF4Lines + c;
    double2 v[16];
    if (j < 8) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            v[e] = ld.at(slot, (j + 8 * e) * N2 + n2);
            opaque(v[e]);
        }
        f4_first(v, lds + c * kF4Stride, j);
    }
    __syncthreads();
    f4_second<128>(v, lds + c * kF4Stride, j, N, tw);
    double2* dst = buf + slot * N + n2;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k1 = j + 16 * e;
        dst[k1 * N2] = cmul_fma(v[oreg<8>(e)], twiddle_rt(tw, n2 * k1, N / 4));
    }
}

// Forward row of line l of group g (see above), the line of the row -k1 and
// whether that is the line itself.
template <int N2>
__device__ __forceinline__ int f4_row(int g, int l) {
    if constexpr (N2 == 128) {
        const int j = 4 * g + (l & 3);
        return l < 4 ? j : (j ? 128 - j : 64);
    } else {
        const int j = 2 * g + (l >> 2), r = l & 3;
        return ((r & 1) ? (j ? 64 - j : 32) : j) + 32 * (r & 2);
    }
}
template <int N2>
__device__ __forceinline__ int f4_partner(int l, int k1) {
    if ((k1 & 63) == 0) return l;
    if constexpr (N2 == 128) return l ^ 4;
    return k1 == 32 || k1 == 96 ? l ^ 2 : l ^ 3;
}

// conj(4 W) at element k2 of row k1 (line l) from Z_k and Z_(N-k) (see
// convolve_pair).
template <int N2>
__device__ __forceinline__ double2 f4_product(const double2* lds, int l, int k1, int k2) {
    const int kn = k1 ? N2 - 1 - k2 : (N2 - k2) & (N2 - 1);
    const double2 zk = lds[l * kF4Stride + padi(k2)], zn = lds[f4_partner<N2>(l, k1) * kF4Stride + padi(kn)];
    const double2 a = make_double2(zk.x + zn.x, zk.y - zn.y);
    const double2 c = make_double2(zk.y + zn.y, zn.x - zk.x);
    const double2 w = cmul_fma(a, c);
    return make_double2(w.x, -w.y);
}

// Workgroup g: transform g / 16 and its g % 16-th set of 8 forward rows, which
// are 8 (N2 = 128) or 4 (N2 = 64, every second element from the row + 64)
// columns of the inverse.  Slots of pairs that are not live are left alone.
template <int N2>
__global__ __launch_bounds__(kF4Threads) void mt_long_middle_kernel(double2* __restrict__ buf,
                                                                   const double2* __restrict__ tw,
                                                                   const int* __restrict__ open_at, int64_t b,
                                                                   int chunk) {
    __shared__ double2 lds[kF4Lines * kF4Stride];
    constexpr int N = 128 * N2, R = N2 / 16;
    const int64_t slot = blockIdx.x / 16;
    if (open_at && open_at[slot % b] != chunk) return;
    const int g = (int)(blockIdx.x & 15), t = threadIdx.x;
    double2* z = buf + slot * N;
    double2 v[16];
    // forward rows
    if (t < kF4Lines * R) {
        const int l = t / R, j = t & (R - 1);
        const double2* src = z + f4_row<N2>(g, l) * N2 + j;
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = src[R * e];
        f4_first(v, lds + l * kF4Stride, j);
    }
    __syncthreads();
    {
        const int l = t / 16, j = t & 15;
        f4_second<N2>(v, lds + l * kF4Stride, j, N, tw);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < R; ++e) lds[l * kF4Stride + padi(j + 16 * e)] = v[oreg<R>(e)];
    }
    __syncthreads();
    // the product, and the inverse's columns
    constexpr int kCols = N2 / 16;
    const int cf = t / 8, jf = t & 7;
    if (cf < kCols) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int n1 = jf + 8 * e;
            int l = cf, k2 = n1;
            if constexpr (N2 == 64) {
                l = 4 * (cf >> 1) + (cf & 1) + 2 * (n1 & 1);
                k2 = n1 >> 1;
            }
            v[e] = f4_product<N2>(lds, l, f4_row<N2>(g, l), k2);
            opaque(v[e]);
        }
    }
    __syncthreads();
    if (cf < kCols) f4_first(v, lds + cf * kF4Stride, jf);
    __syncthreads();
    const int c = t / 16, j = t & 15;
    if (c < kCols) {
        f4_second<128>(v, lds + c * kF4Stride, j, N, tw);
        const int n2 = f4_row<N2>(g, N2 == 64 ? 4 * (c >> 1) + (c & 1) : c);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k1 = j + 16 * e;
            z[f4_place<N2>(n2, k1)] = cmul_fma(v[oreg<8>(e)], twiddle_rt(tw, n2 * k1, N / 4));
        }
    }
}

// The inverse's rows 8 g ... 8 g + 7 of one transform: lane j of line c ends
// with result t = 8 g + c + 128 (j + 16 e) in v[oreg<N2 / 16>(e)].  Lanes run
// over the 8 rows first.  lds may be in use by the caller's last call.
template <int N2>
__device__ __forceinline__ void f4_inverse_rows(double2 (&v)[16], double2* lds, const double2* z, int g,
                                                const double2* tw) {
    constexpr int R = N2 / 16;
    const int t = threadIdx.x, c = t & (kF4Lines - 1), j = t / kF4Lines;
    const int k1 = g * kF4Lines + c;
    if (j < R) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = z[f4_place<N2>(j + R * e, k1)];
    }
    __syncthreads();
    if (j < R) f4_first(v, lds + c * kF4Stride, j);
    __syncthreads();
    f4_second<N2>(v, lds + c * kF4Stride, j, 128 * N2, tw);
    // the imaginary parts stay: without them the last sums contract otherwise
#pragma unroll
    for (int e = 0; e < R; ++e) opaque(v[e]);
}

// sigma[slot][t] = Re(result)[t] * 0.25 / N for t < L.
template <int N2>
__global__ __launch_bounds__(kF4Threads) void mt_xy_long_rows_kernel(const double2* __restrict__ buf,
                                                                    const double2* __restrict__ tw, int64_t L,
                                                                    double* __restrict__ sigma) {
    __shared__ double2 lds[kF4Lines * kF4Stride];
    constexpr int N = 128 * N2, R = N2 / 16;
    const int64_t slot = blockIdx.x / 16;
    const int g = (int)(blockIdx.x & 15);
    double2 v[16];
    f4_inverse_rows<N2>(v, lds, buf + slot * N, g, tw);
    const int t0 = g * kF4Lines + (int)(threadIdx.x & (kF4Lines - 1)) + 128 * (int)(threadIdx.x / kF4Lines);
#pragma unroll
    for (int e = 0; e < R; ++e) {
        const int t = t0 + 2048 * e;
        if (t < L) sigma[slot * L + t] = v[oreg<R>(e)].x * (0.25 / (double)N);
    }
}

// z = max x max y S^(1/p), S clamped at 0.
__device__ __forceinline__ double maxconv_root(double S, int p) {
    double root = 0.0;
    if (S > 0.0) {
        if ((p & (p - 1)) == 0) {
            root = S;
            for (int e = p; e > 1; e >>= 1) root = sqrt(root);
        } else {
            root = exp(log(S) / (double)p);
        }
    }
    return root;
}

// Max-convolution of long vectors (kMaxConvN < N <= kLongConvN): the p family
// in chunks of `slots` p, largest first.  Every index keeps the S of its first
// stable p (code = its family index); a workgroup leaves a chunk once its
// indices are decided, a pair without open indices is skipped by the chunks
// after, and the last chunk takes the roots: at the selected p, the smallest
// p where none was stable.
constexpr uint8_t kCodeOpen = 254;

template <typename T, int N2>
__global__ __launch_bounds__(kF4Threads) void mt_maxconv_long_rows_kernel(
    const double2* __restrict__ buf, const double2* __restrict__ tw, int64_t b, int64_t L, MaxconvSpec spec, int chunk,
    int q_top, int q_end, double* __restrict__ s_sel, uint8_t* __restrict__ code, int* __restrict__ open_at,
    const double* __restrict__ rxy, T* __restrict__ z, uint8_t* __restrict__ pstar) {
    __shared__ double2 lds[kF4Lines * kF4Stride];
    constexpr int N = 128 * N2, R = N2 / 16;
    const int64_t pair = blockIdx.x / 16;
    const int g = (int)(blockIdx.x & 15);
    const int t0 = g * kF4Lines + (int)(threadIdx.x & (kF4Lines - 1)) + 128 * (int)(threadIdx.x / kF4Lines);
    double S[R];
    int cd[R];
    bool open = false;
#pragma unroll
    for (int e = 0; e < R; ++e) {
        const int t = t0 + 2048 * e;
        S[e] = 0.0;
        cd[e] = MT_PSTAR_NONE;
        if (t < L) {
            cd[e] = kCodeOpen;
            if (chunk > 0) {
                cd[e] = code[pair * L + t];
                S[e] = s_sel[pair * L + t];
            }
            open |= cd[e] == kCodeOpen;
        }
    }
    int q = q_top;
    // a workgroup with an open index belongs to a pair that is live
    for (; q >= q_end && __syncthreads_or(open); --q) {
        double2 v[16];
        f4_inverse_rows<N2>(v, lds, buf + ((int64_t)(q_top - q) * b + pair) * N, g, tw);
        open = false;
#pragma unroll
        for (int e = 0; e < R; ++e) {
            if (cd[e] != kCodeOpen) continue;
            const double s = v[oreg<R>(e)].x * (0.25 / (double)N);
            const bool stable = s >= spec.tau;
            if (stable || q == 0) {
                S[e] = s;
                cd[e] = stable ? q : MT_PSTAR_NONE;
            } else {
                open = true;
            }
        }
    }
    const bool last = q_end == 0;
    if (!last && open) open_at[pair] = chunk + 1;
#pragma unroll
    for (int e = 0; e < R; ++e) {
        const int t = t0 + 2048 * e;
        if (t >= L) continue;
        const int64_t at = pair * L + t;
        if (last) {
            z[at] = (T)(rxy[pair] * maxconv_root(S[e], spec.p[cd[e] == MT_PSTAR_NONE ? 0 : cd[e]]));
            if (pstar) pstar[at] = (uint8_t)cd[e];
        } else {
            s_sel[at] = S[e];
            code[at] = (uint8_t)cd[e];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void mt_maxconv_exact_kernel(const T* __restrict__ x, const T* __restrict__ y,
                                                              int64_t b, int64_t n, int64_t m,
                                                              T* __restrict__ z) {
    const int64_t L = n + m - 1;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= b * L) return;
    const int64_t bi = g / L, t = g - bi * L;
    const T* xb = x + bi * n;
    const T* yb = y + bi * m;
    const int64_t lo = t - (m - 1) > 0 ? t - (m - 1) : 0;
    const int64_t hi = t < n - 1 ? t : n - 1;
    T best = 0;
    for (int64_t i = lo; i <= hi; ++i) {
        const T v = xb[i] * yb[t - i];
        best = v > best ? v : best;
    }
    z[g] = best;
}

}  // namespace

int maxconv_log_size(int64_t n, int64_t m) {
    const int64_t L = n + m - 1;
    int logN = kConvMinLog;
    while ((int64_t(1) << logN) < L) ++logN;
    return logN;
}

namespace {

template <typename T, int LOGN>
hipError_t launch_maxconv_n(const T* x, const T* y, int64_t b, int64_t n, int64_t m, const MaxconvSpec& spec,
                            T* z, uint8_t* pstar, hipStream_t st) {
    auto kern = mt_maxconv_kernel<T, LOGN>;
    const int lds = (kConvTwElems + kConvLdsElems) * (int)sizeof(double2);
    // the dynamic-LDS limit is a per-device attribute of each kernel
    static std::atomic<uint64_t> attr_set{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load() & bit)) {
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set.fetch_or(bit);
    }
    constexpr int G = Fft<LOGN>::G;
    const int64_t blocks = (b + G - 1) / G;
    timing_before("mt_maxconv", st);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kConvThreads), lds, st, x, y, b, n, m, spec, z, pstar,
                       timing_work_slot());
    timing_after(st);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_maxconv_t(const T* x, const T* y, int64_t b, int64_t n, int64_t m, const MaxconvSpec& spec,
                            T* z, uint8_t* pstar, hipStream_t st) {
    switch (maxconv_log_size(n, m)) {
        case 4: return launch_maxconv_n<T, 4>(x, y, b, n, m, spec, z, pstar, st);
        case 5: return launch_maxconv_n<T, 5>(x, y, b, n, m, spec, z, pstar, st);
        case 6: return launch_maxconv_n<T, 6>(x, y, b, n, m, spec, z, pstar, st);
        case 7: return launch_maxconv_n<T, 7>(x, y, b, n, m, spec, z, pstar, st);
        case 8: return launch_maxconv_n<T, 8>(x, y, b, n, m, spec, z, pstar, st);
        case 9: return launch_maxconv_n<T, 9>(x, y, b, n, m, spec, z, pstar, st);
        case 10: return launch_maxconv_n<T, 10>(x, y, b, n, m, spec, z, pstar, st);
        case 11: return launch_maxconv_n<T, 11>(x, y, b, n, m, spec, z, pstar, st);
        case 12: return launch_maxconv_n<T, 12>(x, y, b, n, m, spec, z, pstar, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace


namespace {

template <typename T, int LOGN>
hipError_t launch_xy_sigma_n(const T* x, const T* y, int64_t n, const MaxconvSpec& spec, double* sigma,
                             hipStream_t st) {
    auto kern = mt_xy_sigma_kernel<T, LOGN>;
    const int lds = (kConvTwElems + kConvLdsElems) * (int)sizeof(double2);
    static std::atomic<uint64_t> attr_set{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load() & bit)) {
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set.fetch_or(bit);
    }
    constexpr int G = Fft<LOGN>::G;
    const int blocks = (2 * spec.n + G - 1) / G;
    timing_before("mt_xy_sigma", st);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kConvThreads), lds, st, x, y, n, spec, sigma);
    timing_after(st);
    return hipGetLastError();
}

// Max-convolution of long vectors through the buffer of ws: `slots` p of the
// whole batch per chunk.
template <typename T, int N2>
hipError_t launch_maxconv_long(const T* x, const T* y, int64_t b, int64_t n, int64_t m, const MaxconvSpec& spec,
                               T* z, uint8_t* pstar, const MaxconvWorkspace& w, hipStream_t st) {
    constexpr int N = 128 * N2;
    const int64_t L = n + m - 1;
    timing_before("mt_maxconv_long_setup", st);
    hipLaunchKernelGGL(mt_maxconv_long_setup_kernel<T>, dim3((unsigned)b + twiddle_blocks(N)),
                       dim3(kLongSetupThreads), 0, st, x, y, b, n, m, N, w.tw, w.rxy, w.inv, w.open_at);
    timing_after(st);
    hipError_t e = hipGetLastError();
    for (int chunk = 0, q_top = spec.n - 1; q_top >= 0 && e == hipSuccess; ++chunk, q_top -= w.slots) {
        const int q_end = q_top - w.slots + 1 > 0 ? q_top - w.slots + 1 : 0;
        const int64_t count = (int64_t)(q_top - q_end + 1) * b;
        const MaxconvLoad<T> ld{x, y, b, n, m, w.inv, w.open_at, chunk, q_top, spec};
        timing_before("mt_maxconv_long_columns", st);
        hipLaunchKernelGGL((mt_long_columns_kernel<N2, MaxconvLoad<T>>), dim3((unsigned)(count * (N2 / kF4Lines))),
                           dim3(kF4Threads), 0, st, ld, w.buf, w.tw);
        timing_after(st);
        timing_before("mt_maxconv_long_middle", st);
        hipLaunchKernelGGL(mt_long_middle_kernel<N2>, dim3((unsigned)(count * 16)), dim3(kF4Threads), 0, st, w.buf,
                           w.tw, w.open_at, b, chunk);
        timing_after(st);
        timing_before("mt_maxconv_long_rows", st);
        hipLaunchKernelGGL((mt_maxconv_long_rows_kernel<T, N2>), dim3((unsigned)(b * 16)), dim3(kF4Threads), 0, st,
                           w.buf, w.tw, b, L, spec, chunk, q_top, q_end, w.s_sel, w.code, w.open_at, w.rxy, z, pstar);
        timing_after(st);
        e = hipGetLastError();
    }
    return e;
}

// The ring results of long lists (N > kMaxConvN) through the global buffer.
template <typename T, int N2>
hipError_t launch_xy_long(const T* x, const T* y, int64_t n, const MaxconvSpec& spec, const XyWorkspace& w,
                          hipStream_t st) {
    constexpr int N = 128 * N2;
    const unsigned slots = 2 * (unsigned)spec.n;
    timing_before("mt_xy_sigma_setup", st);
    hipLaunchKernelGGL(mt_xy_long_setup_kernel<T>, dim3(1 + twiddle_blocks(N)), dim3(kLongSetupThreads), 0, st, x, y,
                       n, N, w.tw, w.mxy);
    timing_after(st);
    const XyLoad<T> ld{x, y, n, w.mxy, spec};
    timing_before("mt_xy_sigma_columns", st);
    hipLaunchKernelGGL((mt_long_columns_kernel<N2, XyLoad<T>>), dim3(slots * (N2 / kF4Lines)), dim3(kF4Threads), 0,
                       st, ld, w.buf, w.tw);
    timing_after(st);
    timing_before("mt_xy_sigma_middle", st);
    hipLaunchKernelGGL(mt_long_middle_kernel<N2>, dim3(slots * 16), dim3(kF4Threads), 0, st, w.buf, w.tw,
                       (const int*)nullptr, (int64_t)1, 0);
    timing_after(st);
    timing_before("mt_xy_sigma_rows", st);
    hipLaunchKernelGGL(mt_xy_long_rows_kernel<N2>, dim3(slots * 16), dim3(kF4Threads), 0, st, w.buf, w.tw, 2 * n - 1,
                       w.sigma);
    timing_after(st);
    return hipGetLastError();
}

// LDS bytes of the lockstep queue: log estimates and diagonals of 2K
// candidates; paired: the reported pairs and, when kept there, the log
// lengths; the 2 |P| K column cells when they are kept there.
size_t lockstep_lds(int K, int k, int np, bool paired, bool cols, bool lens) {
    return (size_t)2 * K * (sizeof(double) + sizeof(int)) +
           (paired ? (size_t)k * sizeof(int) + (lens ? (size_t)2 * K * sizeof(double) : 0) : 0) +
           (cols ? (size_t)2 * np * K * sizeof(double) : 0);
}
constexpr size_t kLdsBytes = 160 * 1024;

template <typename T, bool kPaired, bool kColsLds, int kRegS, bool kLenLds = true>
hipError_t launch_lockstep(const T* x, const T* y, int64_t n, int32_t k, int K, const MaxconvSpec& spec,
                           double* values, int32_t* diag, int32_t* ii, int32_t* jj, const XyWorkspace& w,
                           hipStream_t st) {
    auto queue = mt_xy_lockstep_kernel<T, kPaired, kColsLds, kRegS, kLenLds>;
    // at least the waves' maxima
    const size_t lds = std::max(lockstep_lds(K, k, spec.n, kPaired, kColsLds, kLenLds),
                                (size_t)(2 * kLockThreads / 64) * sizeof(double));
    if (lds > kLdsBytes) return hipErrorInvalidValue;
    static std::atomic<uint64_t> attr_set{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load() & bit)) {
        e = hipFuncSetAttribute((const void*)queue, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        if (e != hipSuccess) return e;
        attr_set.fetch_or(bit);
    }
    timing_before(kPaired ? "mt_xy_paired" : "mt_xy_queue", st);
    hipLaunchKernelGGL(queue, dim3(1), dim3(kLockThreads), lds, st, x, y, n, spec, w.cand_m,
                       w.cand_psi, w.cand_cols, K, k, values, diag, w.diag1, ii, jj);
    timing_after(st);
    return hipGetLastError();
}

// k <= kPairedMaxK: both runs in lockstep over their K = min(k, 2n - 1)
// candidates (plain or paired).
template <typename T>
hipError_t launch_xy_candidates(const T* x, const T* y, int64_t n, int32_t k, const MaxconvSpec& spec, bool paired,
                                double* values, int32_t* diag, int32_t* ii, int32_t* jj, const XyWorkspace& w,
                                hipStream_t st) {
    const int L = (int)(2 * n - 1), K = k < L ? k : L;
    if (k > kPairedMaxK || L >= kLongConvN || spec.n > 32) return hipErrorInvalidValue;
    timing_before("mt_xy_select", st);
    hipLaunchKernelGGL(mt_xy_select_kernel, dim3(2), dim3(kSelThreads), 0, st, w.psi, L, K, w.cand_m, w.cand_psi);
    hipLaunchKernelGGL(mt_xy_gather_kernel, dim3((unsigned)(2 * spec.n * K + 255) / 256), dim3(256), 0, st, w.sigma,
                       L, K, spec.n, w.cand_m, w.cand_cols);
    timing_after(st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // K <= 256: the columns always fit (at most 2 x 32 x 256 x 8 B plus
    // 40 K + 4 k bytes), and a lane's 8 slots of its run stay in registers.
    // The largest case, K = k = 4096, needs 40 K = 160 KiB plain and
    // 24 K + 4 k paired with the log lengths taken per rank.
    const bool cols = lockstep_lds(K, k, spec.n, paired, true, true) <= kLdsBytes;
    const bool regs = K <= 256 && cols;
    if (paired) {
        if (regs) return launch_lockstep<T, true, true, 8>(x, y, n, k, K, spec, values, diag, ii, jj, w, st);
        if (cols) return launch_lockstep<T, true, true, 0>(x, y, n, k, K, spec, values, diag, ii, jj, w, st);
        if (lockstep_lds(K, k, spec.n, true, false, true) <= kLdsBytes)
            return launch_lockstep<T, true, false, 0>(x, y, n, k, K, spec, values, diag, ii, jj, w, st);
        return launch_lockstep<T, true, false, 0, false>(x, y, n, k, K, spec, values, diag, ii, jj, w, st);
    }
    if (regs) return launch_lockstep<T, false, true, 8>(x, y, n, k, K, spec, values, diag, ii, jj, w, st);
    return cols ? launch_lockstep<T, false, true, 0>(x, y, n, k, K, spec, values, diag, ii, jj, w, st)
                : launch_lockstep<T, false, false, 0>(x, y, n, k, K, spec, values, diag, ii, jj, w, st);
}

template <typename T>
hipError_t launch_xy_t(const T* x, const T* y, int64_t n, int32_t k, const MaxconvSpec& spec, bool paired,
                       double* values, int32_t* diag, int32_t* ii, int32_t* jj, const XyWorkspace& w,
                       hipStream_t st) {
    hipError_t e = hipErrorInvalidValue;
    switch (maxconv_log_size(n, n)) {
        case 4: e = launch_xy_sigma_n<T, 4>(x, y, n, spec, w.sigma, st); break;
        case 5: e = launch_xy_sigma_n<T, 5>(x, y, n, spec, w.sigma, st); break;
        case 6: e = launch_xy_sigma_n<T, 6>(x, y, n, spec, w.sigma, st); break;
        case 7: e = launch_xy_sigma_n<T, 7>(x, y, n, spec, w.sigma, st); break;
        case 8: e = launch_xy_sigma_n<T, 8>(x, y, n, spec, w.sigma, st); break;
        case 9: e = launch_xy_sigma_n<T, 9>(x, y, n, spec, w.sigma, st); break;
        case 10: e = launch_xy_sigma_n<T, 10>(x, y, n, spec, w.sigma, st); break;
        case 11: e = launch_xy_sigma_n<T, 11>(x, y, n, spec, w.sigma, st); break;
        case 12: e = launch_xy_sigma_n<T, 12>(x, y, n, spec, w.sigma, st); break;
        case 13: e = launch_xy_long<T, 64>(x, y, n, spec, w, st); break;
        case 14: e = launch_xy_long<T, 128>(x, y, n, spec, w, st); break;
        default: break;
    }
    if (e != hipSuccess) return e;
    if (k <= 0) return hipSuccess;
    const int64_t L = 2 * n - 1;
    timing_before("mt_xy_psi", st);
    hipLaunchKernelGGL(mt_xy_psi_kernel, dim3((unsigned)((2 * L + 255) / 256)), dim3(256), 0, st, w.sigma, L, spec,
                       w.psi);
    timing_after(st);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (k <= kPairedMaxK) return launch_xy_candidates<T>(x, y, n, k, spec, paired, values, diag, ii, jj, w, st);
    if (paired) return hipErrorInvalidValue;
    // psi of one run in LDS: up to 8 (kLongConvN - 1) bytes
    auto queue = mt_xy_queue_kernel<T>;
    static std::atomic<uint64_t> attr_set{0};
    int dev = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load() & bit)) {
        e = hipFuncSetAttribute((const void*)queue, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLongConvN * (int)sizeof(double));
        if (e != hipSuccess) return e;
        attr_set.fetch_or(bit);
    }
    timing_before("mt_xy_queue", st);
    hipLaunchKernelGGL(queue, dim3(2), dim3(64), (size_t)L * sizeof(double), st, x, y, n, spec, w.sigma, w.psi, k,
                       values, w.values1, w.diag0, w.diag1);
    timing_after(st);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    timing_before("mt_xy_index", st);
    hipLaunchKernelGGL(mt_xy_index_kernel, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, st, w.diag0, w.diag1, k,
                       n, diag, ii, jj);
    timing_after(st);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_maxconv(const void* x, const void* y, int f64, int64_t b, int64_t n, int64_t m,
                          const MaxconvSpec& spec, void* z, uint8_t* pstar, const MaxconvWorkspace& w,
                          hipStream_t st) {
    if (b <= 0 || n <= 0 || m <= 0) return hipSuccess;
    const int logN = maxconv_log_size(n, m);
    if (logN > kLongConvLog) return hipErrorInvalidValue;
    if (logN > kMaxConvLog) {
        auto run = [&](auto one, auto n2) {
            using T = decltype(one);
            return launch_maxconv_long<T, decltype(n2)::value>((const T*)x, (const T*)y, b, n, m, spec, (T*)z, pstar,
                                                               w, st);
        };
        using N64 = std::integral_constant<int, 64>;
        using N128 = std::integral_constant<int, 128>;
        if (logN == 13) return f64 ? run(0.0, N64{}) : run(0.0f, N64{});
        return f64 ? run(0.0, N128{}) : run(0.0f, N128{});
    }
    if (f64)
        return launch_maxconv_t<double>((const double*)x, (const double*)y, b, n, m, spec, (double*)z, pstar, st);
    return launch_maxconv_t<float>((const float*)x, (const float*)y, b, n, m, spec, (float*)z, pstar, st);
}

hipError_t launch_xy_topk(const void* x, const void* y, int f64, int64_t n, int32_t k, const MaxconvSpec& spec,
                          bool paired, double* values, int32_t* diag, int32_t* ii, int32_t* jj,
                          const XyWorkspace& w, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (maxconv_log_size(n, n) > kLongConvLog) return hipErrorInvalidValue;
    if (f64)
        return launch_xy_t<double>((const double*)x, (const double*)y, n, k, spec, paired, values, diag, ii, jj, w,
                                   st);
    return launch_xy_t<float>((const float*)x, (const float*)y, n, k, spec, paired, values, diag, ii, jj, w, st);
}

hipError_t launch_maxconv_exact(const void* x, const void* y, int f64, int64_t b, int64_t n, int64_t m,
                                void* z, hipStream_t st) {
    const int64_t total = b * (n + m - 1);
    if (b <= 0 || n <= 0 || m <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    timing_before("mt_exact_maxconv", st);
    if (f64)
        hipLaunchKernelGGL(mt_maxconv_exact_kernel<double>, dim3(blocks), dim3(256), 0, st, (const double*)x,
                           (const double*)y, b, n, m, (double*)z);
    else
        hipLaunchKernelGGL(mt_maxconv_exact_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float*)x,
                           (const float*)y, b, n, m, (float*)z);
    timing_after(st);
    return hipGetLastError();
}

}  // namespace mt
