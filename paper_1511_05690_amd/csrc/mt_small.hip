// One-kernel product estimate on the FP64 path for small products: the row
// and column scales of the scaled ring call H' (Sec. 2.1), the powers, the
// ring products S_p = A'^p B'^p (Alg. 3 / Alg. 5) and the selection of the
// largest stable p with its 1/p root (Sec. 1, Alg. 5) in one launch.
//
// A workgroup of W waves owns a 16 x 16 output tile of one batch item, each
// wave 32 inner indices of it.  A lane holds 8 inner indices of one row of A
// and of one column of B in registers, as v_mfma_f64_16x16x4f64 takes its
// operands; the row and column maxima come from the same registers.  For each
// p, from the largest down, a lane raises its 16 values, the wave multiplies
// them (8 MFMAs) and the waves' sums are added through LDS.  An entry takes
// the first p with S_p >= tau (at the smallest p: whatever S is, with no
// stable p marked); the tile stops once every entry has its p, and the roots
// are taken once at the end.  For the small products it serves (b m k n up to
// a few times 256^3) this replaces the general path's seven to fourteen
// launches (maxima, planes, MFMA GEMM, sparse tail, root) whose fixed costs
// exceed the arithmetic.  The numbers are those of the general FP64 path up
// to the order of the FP64 sums.
//
// Bound by latencies (launch, first loads, one barrier pair per p), so the
// tile is the smallest MFMA tile and the inner dimension is split over waves:
// 256 x 256 x 256 is 256 workgroups, one per compute unit.  With 32 x 32
// tiles on the vector ALUs, operands and powers in LDS, it was 64 workgroups
// and 33 us a call; now 13 (kernel 9.6).  Elsewhere: 320^3 48 -> 25,
// 4000 x 16^3 343 -> 17, 2048 x 8 x 2048 278 -> 50, 16 x 20000 x 16 2421 -> 370.
#include <cfloat>
#include <cmath>

#include "mt_internal.h"

namespace mt {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kSmTile = 16;   // output tile edge
constexpr int kSmLane = 8;    // inner indices of a lane
constexpr int kSmWaveK = 32;  // inner indices of a wave: 4 lanes per row or column

// the scaled input a / s of H': one reciprocal per line when s is normal
// (inv > 0), a division when s is subnormal, 0 for a zero line
__device__ inline double sm_scaled(double a, double s, double inv) {
    if (__builtin_expect(inv > 0.0, 1)) return a * inv;
    return s > 0.0 ? a / s : 0.0;
}

template <typename T, int W>
__global__ __launch_bounds__(64 * W) void mt_small_product_f64_kernel(const T* __restrict__ A,
                                                                     const T* __restrict__ B, int64_t m, int64_t k,
                                                                     int64_t n, SmallSpec spec, T* __restrict__ C,
                                                                     uint8_t* __restrict__ pstar,
                                                                     unsigned long long* work) {
    __shared__ double part[W * 256];
    __shared__ double rmax[W * kSmTile], cmax[W * kSmTile];
    constexpr int kChunk = W * kSmWaveK;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (work && tid == 0) timing_span_begin(work);
    const int64_t bi = blockIdx.y;
    const unsigned tiles_n = (unsigned)((n + kSmTile - 1) / kSmTile);
    const int64_t row0 = (int64_t)(blockIdx.x / tiles_n) * kSmTile;
    const int64_t col0 = (int64_t)(blockIdx.x % tiles_n) * kSmTile;
    const int li = lane & 15, lk = wave * kSmWaveK + (lane >> 4) * kSmLane;
    const bool row_in = row0 + li < m, col_in = col0 + li < n;
    const T* a = A + (bi * m + (row_in ? row0 + li : m - 1)) * k;
    const T* b = B + bi * k * n + (col_in ? col0 + li : n - 1);

    // this lane's 8 inner indices of the chunk from kr0 on, 0 outside.  Every
    // load is issued (indices outside are clamped and the value dropped), so
    // that they are all in flight at once.
    double xa[kSmLane], xb[kSmLane];
    auto load = [&](int64_t kr0) {
        const int64_t q0 = kr0 + lk;
        T va[kSmLane], vb[kSmLane];
#pragma unroll
        for (int s = 0; s < kSmLane; ++s) {
            const int64_t q = min(q0 + s, k - 1);
            va[s] = a[q];
            vb[s] = b[q * n];
        }
#pragma unroll
        for (int s = 0; s < kSmLane; ++s) {
            const bool in = q0 + s < k;
            xa[s] = in && row_in ? (double)va[s] : 0.0;
            xb[s] = in && col_in ? (double)vb[s] : 0.0;
        }
    };

    // r_i = max_k A_ik and c_j = max_k B_kj of the tile
    double r = 0.0, c = 0.0;
    for (int64_t kr0 = 0; kr0 < k; kr0 += kChunk) {
        load(kr0);
#pragma unroll
        for (int s = 0; s < kSmLane; ++s) {
            r = fmax(r, xa[s]);
            c = fmax(c, xb[s]);
        }
    }
    for (int off = 16; off < 64; off <<= 1) {
        r = fmax(r, __shfl_xor(r, off));
        c = fmax(c, __shfl_xor(c, off));
    }
    if (lane < kSmTile) {
        rmax[wave * kSmTile + lane] = r;
        cmax[wave * kSmTile + lane] = c;
    }
    __syncthreads();
    auto line_max = [](const double* mx, int i) {
        double v = mx[i];
#pragma unroll
        for (int w = 1; w < W; ++w) v = fmax(v, mx[w * kSmTile + i]);
        return v;
    };
    r = line_max(rmax, li);
    c = line_max(cmax, li);
    const double rinv = r >= DBL_MIN ? 1.0 / r : 0.0, cinv = c >= DBL_MIN ? 1.0 / c : 0.0;
    auto scale = [&]() {
#pragma unroll
        for (int s = 0; s < kSmLane; ++s) {
            xa[s] = sm_scaled(xa[s], r, rinv);
            xb[s] = sm_scaled(xb[s], c, cinv);
        }
    };
    // the operands stay in registers for every p when the inner dimension fits
    const bool resident = k <= kChunk;
    if (resident) scale();

    // this thread's entries e = tid + 64 W u of the tile (row e / 16, column
    // e % 16); bit u of `open` is set while the entry has no p yet
    constexpr int kOwn = W >= 4 ? 1 : 4 / W;
    uint32_t open = 0;
    double S[kOwn], corr[kOwn];
    int ps[kOwn], qs[kOwn];
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
        const int e = tid + 64 * W * u;
        if (e < 256 && row0 + e / kSmTile < m && col0 + e % kSmTile < n) open |= 1u << u;
        S[u] = 0.0;
        corr[u] = 1.0;
        ps[u] = 1;
        qs[u] = MT_PSTAR_NONE;
    }
    const uint32_t mine = open;
    int visited = 0;
    for (int q = spec.n - 1; q >= 0; --q) {  // the largest p first
        ++visited;
        const int p = spec.p[q];
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int64_t kr0 = 0; kr0 < k; kr0 += kChunk) {
            if (!resident) {
                load(kr0);
                scale();
            }
            // (a / r)^p and (b / c)^p by binary powering
            double ta[kSmLane], tb[kSmLane], ya[kSmLane], yb[kSmLane];
#pragma unroll
            for (int s = 0; s < kSmLane; ++s) {
                ta[s] = xa[s];
                tb[s] = xb[s];
                ya[s] = 1.0;
                yb[s] = 1.0;
            }
            for (int pp = p; pp; pp >>= 1) {
                if (pp & 1) {
#pragma unroll
                    for (int s = 0; s < kSmLane; ++s) {
                        ya[s] *= ta[s];
                        yb[s] *= tb[s];
                    }
                }
#pragma unroll
                for (int s = 0; s < kSmLane; ++s) {
                    ta[s] *= ta[s];
                    tb[s] *= tb[s];
                }
            }
#pragma unroll
            for (int s = 0; s < kSmLane; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ya[s], yb[s], acc, 0, 0, 0);
        }
        // accumulator t of a lane: row lane / 16 + 4 t, column lane % 16
#pragma unroll
        for (int t = 0; t < 4; ++t) part[wave * 256 + 64 * t + lane] = acc[t];
        __syncthreads();
        const bool last = q == 0;
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            if (!(open & (1u << u))) continue;
            const int e = tid + 64 * W * u;
            double s = part[e];
#pragma unroll
            for (int w = 1; w < W; ++w) s += part[w * 256 + e];
            const bool stable = s >= spec.tau;
            if (!stable && !last) continue;
            open &= ~(1u << u);
            S[u] = s;
            ps[u] = p;
            corr[u] = spec.corr[q];
            if (stable) qs[u] = q;
        }
        if (!__syncthreads_or(open != 0)) break;
    }
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
        if (!(mine & (1u << u))) continue;
        const int e = tid + 64 * W * u, i = e / kSmTile, j = e % kSmTile;
        const double root = ps[u] == 1 ? S[u] : (S[u] > 0.0 ? exp(log(S[u]) / (double)ps[u]) : 0.0);
        double v = line_max(rmax, i) * line_max(cmax, j) * root * corr[u];
        if (spec.clamp) v = fmin(v, 1.0);
        const int64_t o = (bi * m + row0 + i) * n + col0 + j;
        C[o] = (T)v;
        if (pstar) pstar[o] = (uint8_t)qs[u];
    }
    if (work) {
        // timed launch: 2 k flops per output entry of the tile and p visited,
        // and the end
        __syncthreads();
        if (tid == 0) {
            const int64_t rows = m - row0 < kSmTile ? m - row0 : kSmTile;
            const int64_t cols = n - col0 < kSmTile ? n - col0 : kSmTile;
            atomicAdd(work, (unsigned long long)(2 * rows * cols * k * visited));
            timing_span_end(work);
        }
    }
}

}  // namespace

bool small_product_fits(int64_t b, int64_t m, int64_t n) {
    // a launch has fewer than 2^32 threads in x, at most 1024 per tile
    return b <= 65535 && ((m + kSmTile - 1) / kSmTile) * ((n + kSmTile - 1) / kSmTile) < ((int64_t)1 << 22);
}

hipError_t launch_small_product_f64(const void* A, const void* B, int f64, int64_t b, int64_t m, int64_t k,
                                    int64_t n, const SmallSpec& spec, void* C, uint8_t* pstar, hipStream_t st) {
    if (b <= 0 || m <= 0 || n <= 0) return hipSuccess;
    const dim3 grid((unsigned)(((m + kSmTile - 1) / kSmTile) * ((n + kSmTile - 1) / kSmTile)), (unsigned)b);
    timing_before("mt_small_product_f64", st);
    unsigned long long* work = timing_work_slot();
    // waves: one per 32 inner indices, up to 16 (512 indices in registers;
    // longer inner dimensions go round in chunks of 512: fewer waves would
    // only have fewer loads on their way)
#define MT_SMALL(T, W)                                                                                         \
    hipLaunchKernelGGL((mt_small_product_f64_kernel<T, W>), grid, dim3(64 * W), 0, st, (const T*)A, (const T*)B, \
                       m, k, n, spec, (T*)C, pstar, work)
#define MT_SMALL_K(T)                 \
    if (k <= 32) MT_SMALL(T, 1);       \
    else if (k <= 64) MT_SMALL(T, 2);  \
    else if (k <= 128) MT_SMALL(T, 4); \
    else if (k <= 256) MT_SMALL(T, 8); \
    else MT_SMALL(T, 16)
    if (f64) {
        MT_SMALL_K(double);
    } else {
        MT_SMALL_K(float);
    }
#undef MT_SMALL_K
#undef MT_SMALL
    timing_after(st);
    return hipGetLastError();
}

}  // namespace mt
