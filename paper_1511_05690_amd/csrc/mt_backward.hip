// Adjoint of the p-norm estimate with p* held fixed per entry: the per-entry
// weights that enter the two gradient products, and the p* histogram that
// lets the adjoint GEMMs skip the p no entry uses.
//
// With C' = C / (r_i c_j) and p = p*_ij (the smallest p of the family where
// no p was stable), the derivative of C_ij = (sum_k A_ik^p B_kj^p)^(1/p) gives
//   dL/dA = sum_p A'^(p-1) .* (Gt_p  B'^p^T),  Gt_p  = [p* = p] G c_j C'^(1-p)
//   dL/dB = sum_p B'^(p-1) .* (A'^p^T Gt'_p),  Gt'_p = [p* = p] G r_i C'^(1-p)
// (the paper notes the p-norm rings are continuous and differentiable,
// Sec. 4).  Entries with C = 0 contribute nothing.
#include <cfloat>
#include <cmath>

#include "mt_internal.h"

namespace mt {
namespace {

constexpr int kThreads = 256;

__device__ inline uint16_t bf16_rne(float x) {
    // Round to nearest even on the bit pattern (finite x).
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline float bf16_to_float(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// g x^-e for x > 0 by binary powering of 1 / x as an unevaluated sum h + l
// (l holds what the product h rounded off), so that the result is good to
// about one rounding whatever e: at e = 63 some 60 FP64 operations, where
// exp(-e log x), whose error grows as |e log x| 2^-53, took about 200.
// Beyond the FP64 range the power is infinite, and it is 0 at an infinite x
// (an entry of C that overflowed its type); an infinite g stays infinite.
__device__ inline double times_pow_neg(double g, double x, int e) {
    if (!(x <= DBL_MAX)) return e > 0 ? g * 0.0 : g;
    double xh = 1.0 / x;
    double xl = fma(-x, xh, 1.0) * xh;
    double yh = 1.0, yl = 0.0;
    while (true) {
        if (e & 1) {
            const double h = yh * xh;
            yl = fma(yh, xl, fma(yl, xh, fma(yh, xh, -h)));
            yh = h;
        }
        e >>= 1;
        if (e == 0) break;
        const double h = xh * xh;
        xl = fma(2.0 * xh, xl, fma(xh, xh, -h));
        xh = h;
    }
    if (!(yh <= DBL_MAX)) return g * HUGE_VAL;
    if (!(fabs(g) <= DBL_MAX)) return g * yh;
    return fma(g, yh, g * yl);
}

// hist[q] = number of entries whose p is family index q (MT_PSTAR_NONE -> 0).
// Almost every entry of a product often has the same p, so one counter per p
// and block serialised the LDS atomics of a wave (64 x 512^2 codes: 59 us;
// 12 us now, the 17 MB read take 3 us).  Each lane counts into a column of
// its own (64 columns, shared by the block's waves: one bank each), 16 codes
// a load, and a block adds each p once.
constexpr int kHistBytes = 16;
__global__ __launch_bounds__(kThreads) void mt_pstar_hist_kernel(const uint8_t* __restrict__ ps,
                                                                 int64_t total, int n_p,
                                                                 int32_t* __restrict__ hist) {
    __shared__ int32_t h[MT_MAX_P][64];
    const int lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < MT_MAX_P * 64; i += kThreads) ((int32_t*)h)[i] = 0;
    __syncthreads();
    auto count = [&](int q) { atomicAdd(&h[q == MT_PSTAR_NONE || q >= n_p ? 0 : q][lane], 1); };
    // p_star may start at any byte: the loads are 16 bytes wide, not aligned
    typedef uint32_t codes __attribute__((ext_vector_type(4), aligned(1)));
    const int64_t chunks = total / kHistBytes;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    const int64_t first = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t v = first; v < chunks; v += stride) {
        const codes w = *(const codes*)(ps + v * kHistBytes);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // four equal codes (the common case) are one add
            const int q = (int)(w[i] & 255u);
            if (w[i] == (uint32_t)q * 0x01010101u) {
                atomicAdd(&h[q == MT_PSTAR_NONE || q >= n_p ? 0 : q][lane], 4);
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) count((int)((w[i] >> (8 * t)) & 255u));
            }
        }
    }
    for (int64_t e = chunks * kHistBytes + first; e < total; e += stride) count(ps[e]);
    __syncthreads();
    for (int q = threadIdx.x >> 6; q < n_p; q += kThreads / 64) {
        int32_t v = h[q][lane];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0 && v) atomicAdd(&hist[q], v);
    }
}

// Per batch item, the binary exponents of the largest row scale and of the
// largest column scale: ex[bi] = e with max_i r_i < 2^e, ex[b + bi] the
// same for c.  The BF16 adjoint planes carry r_i / 2^ex and c_j / 2^ex, which
// lie in (0, 1] whatever the range of the inputs, and the adjoint GEMMs
// multiply their sums back by 2^ex.
__global__ __launch_bounds__(kThreads) void mt_scale_exp_kernel(const double* __restrict__ r,
                                                                const double* __restrict__ c, int64_t m,
                                                                int64_t n, int32_t* __restrict__ ex) {
    __shared__ double red[2][kThreads / 64];
    const int64_t bi = blockIdx.x;
    double mr = 0.0, mc = 0.0;
    for (int64_t i = threadIdx.x; i < m; i += kThreads) mr = fmax(mr, r[bi * m + i]);
    for (int64_t j = threadIdx.x; j < n; j += kThreads) mc = fmax(mc, c[bi * n + j]);
    for (int off = 32; off > 0; off >>= 1) {
        mr = fmax(mr, __shfl_xor(mr, off, 64));
        mc = fmax(mc, __shfl_xor(mc, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = mr;
        red[1][threadIdx.x >> 6] = mc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) {
            mr = fmax(mr, red[0][w]);
            mc = fmax(mc, red[1][w]);
        }
        int er = 0, ec = 0;
        if (mr > 0.0) (void)frexp(mr, &er);
        if (mc > 0.0) (void)frexp(mc, &ec);
        ex[bi] = er;
        ex[gridDim.x + bi] = ec;
    }
}

// 8 consecutive values as BF16 hi and lo planes (kBf16) or as doubles.
template <bool kBf16>
__device__ __forceinline__ void store_adjoint8(void* planes, int64_t pos, int64_t plane_elems, const double (&v)[8]) {
    if (kBf16) {
        uint16_t* pl = (uint16_t*)planes + pos;
        u32x4 hi, lo;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float f0 = (float)v[2 * t], f1 = (float)v[2 * t + 1];
            const uint16_t h0 = bf16_rne(f0), h1 = bf16_rne(f1);
            hi[t] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            lo[t] = (uint32_t)bf16_rne(f0 - bf16_to_float(h0)) | ((uint32_t)bf16_rne(f1 - bf16_to_float(h1)) << 16);
        }
        *(u32x4*)pl = hi;
        *(u32x4*)(pl + plane_elems) = lo;
    } else {
        double* pl = (double*)planes + pos;
#pragma unroll
        for (int t = 0; t < 8; t += 2) *(double2*)(pl + t) = double2{v[t], v[t + 1]};
    }
}

// Adjoint planes for one 64 x 64 (i, j) tile of one batch item.
//   XA: [b][plane][m_pad][n_kpad]  Gt_p   (rows i, inner j)  -> dA product
//   YB: [b][plane][n_pad][m_kpad]  Gt'_p^T (rows j, inner i) -> dB product
// For the BF16 path each p has a hi and a lo plane (planes 2q, 2q + 1);
// for FP64 one plane (q).  Planes of p that no entry uses are not written.
// Bound by the latency of its loads and of the weights' FP64 chain: a thread
// owns 8 consecutive j of two rows, so that all its loads are in flight at
// once (16 rounds of one element each, with the family's p looked up in the
// arguments, ran at 1.9 TB/s: 152 us at 64 x 512^2, 117 us now), and its XA
// chunks go out from registers; only YB takes the LDS transpose.
template <typename T, bool kBf16>
__global__ __launch_bounds__(kThreads) void mt_adjoint_prep_kernel(
    const T* __restrict__ G, const T* __restrict__ C, const uint8_t* __restrict__ pstar,
    const double* __restrict__ r, const double* __restrict__ c, const int32_t* __restrict__ ex, int64_t m,
    int64_t n, AdjPrepSpec spec, const int32_t* __restrict__ hist, void* __restrict__ XA,
    void* __restrict__ YB) {
    __shared__ double gw[64][65];  // G * C'^(1-p), 0 where C = 0 or outside
    __shared__ uint8_t qq[64][68];  // family index of p*
    __shared__ double rsh[64], csh[64];  // r_i and c_j as the planes take them (/ 2^ex on the BF16 path)
    __shared__ double rm[64], cm[64];    // mantissas of r_i and c_j
    __shared__ int re[64], ce[64];       // and their exponents
    __shared__ int pt[MT_MAX_P];         // the family
    const int64_t bi = blockIdx.z;
    const int64_t i0 = (int64_t)blockIdx.y * 64, j0 = (int64_t)blockIdx.x * 64;
    const int64_t base = bi * m * n;

    // this thread's tasks: row tid / 8 + 32 t, columns 8 (tid % 8) .. + 7
    constexpr int kTasks = 64 * 8 / kThreads;
    typedef T vec8 __attribute__((ext_vector_type(8), aligned(sizeof(T))));
    typedef uint8_t code8 __attribute__((ext_vector_type(8), aligned(1)));
    const int ch = threadIdx.x & 7;
    const int64_t j = j0 + ch * 8;
    vec8 gv[kTasks], cv[kTasks];
    code8 pv[kTasks];
#pragma unroll
    for (int t = 0; t < kTasks; ++t) {
        const int64_t i = i0 + (threadIdx.x >> 3) + t * (kThreads / 8);
        const int64_t o = base + i * n + j;
        if (i < m && j + 8 <= n) {
            gv[t] = *(const vec8*)(G + o);
            cv[t] = *(const vec8*)(C + o);
            pv[t] = *(const code8*)(pstar + o);
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool in = i < m && j + u < n;
                gv[t][u] = in ? G[o + u] : T(0);
                cv[t][u] = in ? C[o + u] : T(0);
                pv[t][u] = in ? pstar[o + u] : 0;
            }
        }
    }
    uint32_t used = 0;
    for (int q = 0; q < spec.n_p; ++q) used |= (hist[q] != 0 ? 1u : 0u) << q;
    if (threadIdx.x < 128) {
        const bool is_r = threadIdx.x < 64;
        const int t = threadIdx.x & 63;
        const int64_t idx = (is_r ? i0 : j0) + t;
        const double v = is_r ? (idx < m ? r[bi * m + idx] : 0.0) : (idx < n ? c[bi * n + idx] : 0.0);
        int e = 0;
        const double mv = v > 0.0 ? frexp(v, &e) : 0.0;
        const double vs = ex ? ldexp(v, -ex[(is_r ? 0 : gridDim.z) + bi]) : v;
        if (is_r) {
            rsh[t] = vs;
            rm[t] = mv;
            re[t] = e;
        } else {
            csh[t] = vs;
            cm[t] = mv;
            ce[t] = e;
        }
    }
    for (int q = threadIdx.x; q < spec.n_p; q += kThreads) pt[q] = spec.p[q];
    __syncthreads();

#pragma unroll
    for (int t = 0; t < kTasks; ++t) {
        // 1. per-entry weights (FP64)
        const int ii = (threadIdx.x >> 3) + t * (kThreads / 8);
        const int64_t i = i0 + ii;
        double w[8];
        int q8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int jj = ch * 8 + u;
            const int code = pv[t][u];
            const int q = (code == MT_PSTAR_NONE || code >= spec.n_p) ? 0 : code;
            // C' = C / (r_i c_j), formed as (C 2^-(e_r + e_c)) / (m_r m_c)
            // so that r_i c_j itself never has to be representable
            const double mrc = rm[ii] * cm[jj];
            const double cs = mrc > 0.0 ? ldexp((double)cv[t][u], -(re[ii] + ce[jj])) / mrc : 0.0;
            w[u] = cs > 0.0 ? times_pow_neg((double)gv[t][u], cs, pt[q] - 1) : 0.0;  // G C'^(1-p)
            q8[u] = q;
            gw[ii][jj] = w[u];
            qq[ii][jj] = (uint8_t)q;
        }
        // 2. XA planes (rows i, inner j)
        if (i < spec.xa_rows_pad && j < spec.xa_cols_pad) {
            for (uint32_t left = used; left != 0u; left &= left - 1u) {
                const int q = __builtin_ctz(left);
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = q8[u] == q ? w[u] * csh[ch * 8 + u] : 0.0;
                const int64_t plane = bi * spec.planes + (kBf16 ? 2 * q : q);
                const int64_t elems = spec.xa_rows_pad * spec.xa_cols_pad;
                store_adjoint8<kBf16>(XA, plane * elems + i * spec.xa_cols_pad + j, elems, v);
            }
        }
    }
    __syncthreads();

    // 3. YB planes (rows j, inner i): 8 consecutive i per task (transposed)
    for (int task = threadIdx.x; task < 64 * 8; task += kThreads) {
        const int jj = task >> 3, ci = task & 7;
        const int64_t jr = j0 + jj, i = i0 + ci * 8;
        if (jr >= spec.yb_rows_pad || i >= spec.yb_cols_pad) continue;
        double w[8];
        int q8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            w[u] = gw[ci * 8 + u][jj] * rsh[ci * 8 + u];
            q8[u] = qq[ci * 8 + u][jj];
        }
        for (uint32_t left = used; left != 0u; left &= left - 1u) {
            const int q = __builtin_ctz(left);
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = q8[u] == q ? w[u] : 0.0;
            const int64_t plane = bi * spec.planes + (kBf16 ? 2 * q : q);
            const int64_t elems = spec.yb_rows_pad * spec.yb_cols_pad;
            store_adjoint8<kBf16>(YB, plane * elems + jr * spec.yb_cols_pad + i, elems, v);
        }
    }
}

}  // namespace

hipError_t launch_pstar_hist(const uint8_t* ps, int64_t total, int n_p, int32_t* hist,
                             hipStream_t st) {
    if (total <= 0) return hipSuccess;
    // at most two blocks per CU: their adds to the same few counters queue
    int64_t g = (total + kThreads * kHistBytes - 1) / (kThreads * kHistBytes);
    if (g > 512) g = 512;
    timing_before("mt_pstar_hist", st);
    hipLaunchKernelGGL(mt_pstar_hist_kernel, dim3((unsigned)g), dim3(kThreads), 0, st, ps, total, n_p, hist);
    timing_after(st);
    return hipGetLastError();
}

hipError_t launch_scale_exp(const double* r, const double* c, int64_t b, int64_t m, int64_t n, int32_t* ex,
                            hipStream_t st) {
    if (b <= 0) return hipSuccess;
    timing_before("mt_scale_exp", st);
    hipLaunchKernelGGL(mt_scale_exp_kernel, dim3((unsigned)b), dim3(kThreads), 0, st, r, c, m, n, ex);
    timing_after(st);
    return hipGetLastError();
}

hipError_t launch_adjoint_prep(const void* G, const void* C, const uint8_t* pstar, int io_f64,
                               const double* r, const double* c, const int32_t* ex, int64_t b, int64_t m,
                               int64_t n, const AdjPrepSpec& spec, const int32_t* hist, int bf16, void* XA,
                               void* YB, hipStream_t st) {
    const int64_t rows_cover = spec.xa_rows_pad > spec.yb_cols_pad ? spec.xa_rows_pad : spec.yb_cols_pad;
    const int64_t cols_cover = spec.xa_cols_pad > spec.yb_rows_pad ? spec.xa_cols_pad : spec.yb_rows_pad;
    const dim3 grid((unsigned)((cols_cover + 63) / 64), (unsigned)((rows_cover + 63) / 64), (unsigned)b);
#define MT_PREP(T, BF)                                                                              \
    hipLaunchKernelGGL((mt_adjoint_prep_kernel<T, BF>), grid, dim3(kThreads), 0, st, (const T*)G,  \
                       (const T*)C, pstar, r, c, ex, m, n, spec, hist, XA, YB)
    timing_before("mt_adjoint_prep", st);
    if (io_f64) {
        if (bf16) MT_PREP(double, true); else MT_PREP(double, false);
    } else {
        if (bf16) MT_PREP(float, true); else MT_PREP(float, false);
    }
#undef MT_PREP
    timing_after(st);
    return hipGetLastError();
}

}  // namespace mt
