// p-family GEMMs on FP64 MFMA (gfx950): the plain-precision path.  Same
// scheme as the BF16 kernels (one main loop, two epilogues), with FP64 planes
// and v_mfma_f64_16x16x4f64.
//
// Forward (selection-record epilogue).  Ring products of every p of the
// family per output tile, largest p first (Alg. 5 and Sec. 1).  Once per
// entry the epilogue records the ring result S at the largest p with
// S_p >= tau (FP64 test) and that p's index; the FP64 root C = r c S^(1/p) is
// taken by the select-root pass (mt_elementwise.hip), which keeps the
// library's log / exp out of the unrolled epilogue.  A tile whose entries all
// have their p stops: the smaller p cannot change the result.
//
// Adjoint (accumulating epilogue).  As in the BF16 kernel: sum over the p
// some entry uses of (scaled input)^(p-1) .* (X_p Y_p^T), written once.
//
// Tiling: 256 threads = 4 waves in 2 x 2; each wave owns WT x WT MFMA tiles of
// 16 x 16.  K step 16 doubles = 128-byte LDS rows, loaded by
// global_load_lds_dwordx4 and double buffered; 16-byte chunk index
// XOR-swizzled with (row >> 1) & 7.  At most 256 registers per lane, so two
// workgroups share a CU and one hides the other's barrier waits.
#include <atomic>
#include <cfloat>
#include <cmath>

#include "mt_internal.h"

namespace mt {
namespace {

constexpr int kThreads = 256;

struct GemmGeomF64 {
    const double* X;
    const double* Y;
    int64_t x_plane_elems;
    int64_t y_plane_elems;
    int64_t x_batch_elems;
    int64_t y_batch_elems;
    int64_t kp;
    int64_t rows, cols;
    int32_t tiles_m, tiles_n;
    int32_t bm;                // output tile side
    unsigned long long* work;  // if set: MFMA flops executed, summed over workgroups
};

template <int WT_>
struct CfgF64 {
    static constexpr int WT = WT_;
    static constexpr int BM = 2 * WT * 16;
    static constexpr int A_BYTES = BM * 128;
    static constexpr int BUF_BYTES = 2 * A_BYTES;
    static constexpr int PIPE_BYTES = 2 * BUF_BYTES;
    static_assert((BM / 32) % 2 == 0, "row groups per wave must be even");
};

struct TileCtx {
    int lane, wave, wm, wn, bi;
    int64_t row0, col0;
};

// ------------------------------------------------------------ selection record
template <class C, bool R1, bool RERUN = false>
struct RecordEpi {
    static constexpr int WT = C::WT;
    static constexpr int NDEC = (WT * WT * 4 + 31) / 32;
    static constexpr int LDS_BYTES = 0;
    using Args = EpiArgs;
    EpiArgs a;
    int64_t n;
    uint32_t decided[NDEC];
    // r = 1 projection: S_{p*} recorded, S at the next smaller p still due;
    // otherwise: parked, i.e. stable at the p recorded and a larger p may be
    // stable too
    uint32_t pending[NDEC];
    int lr0, lc0;
    int64_t out_lane;
    int32_t rows_left, cols_left;
    int32_t n_eval;  // plan entries whose planes this launch may read

    static constexpr bool kCanStop = true;
    __device__ bool active(int, const FamilyPlan&) const { return true; }
    // Deferred planes: the planes of plan entries n_eval and below are not
    // written (yet), so the way down ends above them.  The rerun launch runs
    // only the tiles marked for it, with every plane written, densely to the
    // end.
    __device__ int down_end(const FamilyPlan& plan) const { return min(plan.n, n_eval); }
    static __device__ bool skip_tile(const Args& a, int64_t tile) { return RERUN && a.missed_tile[tile] == 0u; }
    // The tile's number of handed-over entries (0 first).
    __device__ void record_count(int64_t tile, uint32_t n) const {
        if (!RERUN && a.tile_count != nullptr) a.tile_count[tile] = n;
    }
    // Where this tile's `total` entries go in the tail list (one thread).
    __device__ uint32_t take_slots(int64_t tile, int total) const {
        if (a.tile_count == nullptr) return atomicAdd(a.tail_count, (uint32_t)total);
        a.tile_count[tile] = (uint32_t)total;
        return (uint32_t)(tile * a.tail_max);
    }
    __device__ void record_tile(int64_t tile, bool missed) const {
        if (RERUN || a.missed_tile == nullptr) return;
        a.missed_tile[tile] = missed ? 1u : 0u;
        if (missed) *a.low_missed = 1;
    }

    // Entries of this lane without their final record yet: `open` ones have
    // no stable p so far, `parked` ones wait for the way up (with the r = 1
    // projection, whose search starts at the largest p, all count as open).
    __device__ void counts(int& open, int& parked) const {
        constexpr int TOT = WT * WT * 4;
        open = parked = 0;
#pragma unroll
        for (int i = 0; i < NDEC; ++i) {
            const uint32_t full = (TOT - 32 * i >= 32) ? 0xFFFFFFFFu : ((1u << (TOT - 32 * i)) - 1u);
            const uint32_t und = ~decided[i] & full;
            if (R1) {
                open += __builtin_popcount(und);
            } else {
                parked += __builtin_popcount(und & pending[i]);
                open += __builtin_popcount(und & ~pending[i]);
            }
        }
    }
    __device__ int32_t start_index() const { return (!R1 && a.start) ? *a.start : 0; }
    __device__ bool can_hand_over(int total) const { return !RERUN && a.tail != nullptr && total <= a.tail_max; }
    // Write this lane's undecided entries to the sparse-tail list from `pos`
    // on, after plan entry e of a search that started at plan entry s.
    __device__ void hand_over(uint32_t pos, int e, int s, const TileCtx& t) const {
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                const int tix = i * WT + j;
                const int sh = (tix & 7) * 4;
#pragma unroll 1
                for (int r = 0; r < 4; ++r) {
                    const uint32_t mask = 1u << (sh + r);
                    if (decided[tix >> 3] & mask) continue;
                    TailEntry te;
                    te.bi = t.bi;
                    te.i = (int32_t)(t.row0 + lr0 + i * 16 + 4 * r);
                    te.j = (int32_t)(t.col0 + lc0 + j * 16);
                    if (pending[tix >> 3] & mask) {
                        te.state = R1 ? kTailR1 : kTailRise;
                        te.e_next = (int16_t)(R1 ? e + 1 : (e < s ? e - 1 : s - 1));
                    } else {
                        te.state = kTailOpen;
                        te.e_next = (int16_t)(e + 1);
                    }
                    a.tail[pos++] = te;
                }
            }
    }

    __device__ void setup(const TileCtx& t, const GemmGeomF64& g, uint8_t*, int) {
        n = g.cols;
        n_eval = MT_MAX_P;
        if (!RERUN && a.low_need != nullptr && __builtin_amdgcn_readfirstlane(*a.low_need) == 0) n_eval = a.n_eval;
#pragma unroll
        for (int i = 0; i < NDEC; ++i) decided[i] = pending[i] = 0u;
        // Entry (i, j, r) of this lane: tile row wm*WT*16 + i*16 + l/16 + 4r,
        // tile column wn*WT*16 + j*16 + l%16.
        lr0 = t.wm * WT * 16 + (t.lane >> 4);
        lc0 = t.wn * WT * 16 + (t.lane & 15);
        out_lane = ((int64_t)t.bi * g.rows + t.row0 + lr0) * n + t.col0 + lc0;
        rows_left = (int32_t)min<int64_t>(g.rows - (t.row0 + lr0), 1 << 30);
        cols_left = (int32_t)min<int64_t>(n - (t.col0 + lc0), 1 << 30);
        // Entries outside the matrix count as decided from the start.
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int tix = i * WT + j;
                    if (!(j * 16 < cols_left && i * 16 + 4 * r < rows_left))
                        decided[tix >> 3] |= 1u << ((tix & 7) * 4 + r);
                }
    }

    // stage: a free pipeline buffer; each wave stages one 16 x 16 tile
    // (lane-major) and walks its four entries per lane in a rolled loop.
    // Plan entry e of a p search that started at plan entry s: entries e >= s
    // go down from the start (smaller p), entries e < s up (larger p).
    __device__ void entry(int e, int s, const FamilyPlan& plan, f64x4 (&acc)[WT][WT], const TileCtx& t,
                          uint8_t* stage) {
        const bool last = (e == plan.n - 1);
        const bool up = e < s;  // only parked entries are left
        const bool park_here = !up && e == s && s > 0;
        const double rise_thr = plan.e[e].rise_thr;
        const double tau = plan.tau;
        const uint8_t pcode = (uint8_t)plan.e[e].pidx;
        // r = 1 projection: S_{p*} goes to `out`, S at the next smaller p to
        // `out2`; the select-root pass combines them
        const bool defer = R1 && plan.e[e].inv_dp > 0.f;
        double* out = (double*)a.out + out_lane;
        double* out2 = a.out2 ? (double*)a.out2 + out_lane : nullptr;
        uint8_t* ps = a.pstar + out_lane;
        double* stg = (double*)stage + t.wave * 256;
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
#pragma unroll
                for (int r = 0; r < 4; ++r) stg[r * 64 + t.lane] = acc[i][j][r];
                __builtin_amdgcn_wave_barrier();
                const bool col_ok = j * 16 < cols_left;
                const int tix = i * WT + j;
                uint32_t dec = decided[tix >> 3];
                uint32_t pnd = pending[tix >> 3];
                const int sh = (tix & 7) * 4;
#pragma unroll 1
                for (int r = 0; r < 4; ++r) {
                    const uint32_t mask = 1u << (sh + r);
                    const int roff = i * 16 + 4 * r;
                    const double S = stg[r * 64 + t.lane];
                    const bool stable = S >= tau;
                    const int64_t o = (int64_t)roff * n + j * 16;
                    if constexpr (!R1) {
                        // entries outside the matrix are decided from the start
                        if (dec & mask) continue;
                        if (!up) {
                            if (pnd & mask) continue;  // parked at the start: waits for the way up
                            if (!(stable || last)) continue;
                            out[o] = S;
                            ps[o] = stable ? pcode : (uint8_t)MT_PSTAR_NONE;
                            // S_q <= S^(q/p): the next larger q may still pass
                            if (stable && park_here && S >= rise_thr)
                                pnd |= mask;
                            else
                                dec |= mask;
                        } else {
                            // not stable here: the record of the p below stands
                            if (stable) {
                                out[o] = S;
                                ps[o] = pcode;
                                if (e > 0 && S >= rise_thr) continue;
                            }
                            pnd &= ~mask;
                            dec |= mask;
                        }
                        continue;
                    }
                    if (pnd & mask) {
                        out2[o] = S;
                        pnd &= ~mask;
                        dec |= mask;
                    } else if (col_ok && roff < rows_left && !(dec & mask) && (stable || last)) {
                        out[o] = S;
                        ps[o] = stable ? pcode : (uint8_t)MT_PSTAR_NONE;
                        if (stable && defer)
                            pnd |= mask;
                        else
                            dec |= mask;
                    }
                }
                decided[tix >> 3] = dec;
                pending[tix >> 3] = pnd;
                __builtin_amdgcn_wave_barrier();
            }
    }

    __device__ void finish(const TileCtx&) {}
};

// ------------------------------------------------------------ store-all epilogue
// S of plan entry e to plane pidx of the stack out (planes of b x rows x n),
// every entry of the tile, every entry of the plan: the r = 2 projection
// needs four ring results per entry, chosen after p* is known.
template <class C>
struct StoreAllEpi {
    static constexpr int WT = C::WT;
    static constexpr int LDS_BYTES = 0;
    using Args = EpiArgs;
    static constexpr bool kCanStop = false;
    EpiArgs a;
    int64_t n, out_lane;
    int32_t rows_left, cols_left;

    __device__ bool active(int, const FamilyPlan&) const { return true; }
    __device__ int down_end(const FamilyPlan& plan) const { return plan.n; }
    static __device__ bool skip_tile(const Args&, int64_t) { return false; }
    __device__ void record_tile(int64_t, bool) const {}
    __device__ void counts(int& open, int& parked) const { open = parked = 0; }
    __device__ int32_t start_index() const { return 0; }
    __device__ bool can_hand_over(int) const { return false; }
    __device__ uint32_t take_slots(int64_t, int) const { return 0u; }
    __device__ void record_count(int64_t, uint32_t) const {}
    __device__ void hand_over(uint32_t, int, int, const TileCtx&) const {}

    __device__ void setup(const TileCtx& t, const GemmGeomF64& g, uint8_t*, int) {
        n = g.cols;
        const int lr0 = t.wm * WT * 16 + (t.lane >> 4);
        const int lc0 = t.wn * WT * 16 + (t.lane & 15);
        out_lane = ((int64_t)t.bi * g.rows + t.row0 + lr0) * n + t.col0 + lc0;
        rows_left = (int32_t)min<int64_t>(g.rows - (t.row0 + lr0), 1 << 30);
        cols_left = (int32_t)min<int64_t>(n - (t.col0 + lc0), 1 << 30);
    }

    // accumulator (i, j, r) of this lane: tile row i*16 + l/16 + 4r, column
    // j*16 + l%16 (the v_mfma_f64_16x16x4f64 layout)
    __device__ void entry(int e, int, const FamilyPlan& plan, f64x4 (&acc)[WT][WT], const TileCtx&, uint8_t*) {
        double* out = (double*)a.out + (int64_t)plan.e[e].pidx * a.stack_stride + out_lane;
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j * 16 < cols_left && i * 16 + 4 * r < rows_left)
                        out[(int64_t)(i * 16 + 4 * r) * n + j * 16] = acc[i][j][r];
    }

    __device__ void finish(const TileCtx&) {}
};

// ------------------------------------------------------------ adjoint epilogue
template <class C, typename TM>
struct AdjointEpiF64 {
    static constexpr int WT = C::WT;
    // inverse mantissas of the row and column scales, then their exponents
    static constexpr int LDS_BYTES = 2 * C::BM * 8 + 2 * C::BM * 4;
    using Args = AdjArgs;
    static constexpr bool kCanStop = false;
    AdjArgs a;
    int64_t rows, cols;
    f64x4 tot[WT][WT];
    __device__ int down_end(const FamilyPlan& plan) const { return plan.n; }
    static __device__ bool skip_tile(const Args&, int64_t) { return false; }
    __device__ void record_tile(int64_t, bool) const {}
    double* rs;
    double* cs;
    int* res;
    int* ces;
    int lr0, lc0;
    int64_t lane_off;
    int32_t rows_left, cols_left;

    __device__ bool active(int e, const FamilyPlan& plan) const { return a.hist[plan.e[e].pidx] > 0; }
    __device__ void counts(int& open, int& parked) const { open = parked = 0; }
    __device__ int32_t start_index() const { return 0; }
    __device__ bool can_hand_over(int) const { return false; }
    __device__ uint32_t take_slots(int64_t, int) const { return 0u; }
    __device__ void record_count(int64_t, uint32_t) const {}
    __device__ void hand_over(uint32_t, int, int, const TileCtx&) const {}

    __device__ void setup(const TileCtx& t, const GemmGeomF64& g, uint8_t* lds, int tid) {
        rows = g.rows;
        cols = g.cols;
        rs = (double*)lds;
        cs = rs + C::BM;
        res = (int*)(rs + 2 * C::BM);
        ces = res + C::BM;
        // scale v = m 2^e: M / v is formed as (M 2^-e) / m, finite also for
        // a subnormal scale (whose reciprocal is not)
        for (int i = tid; i < 2 * C::BM; i += kThreads) {
            double v = 1.0;
            if (i < C::BM) {
                if (a.scale_rows && t.row0 + i < rows) v = a.scale_rows[(int64_t)t.bi * rows + t.row0 + i];
            } else {
                const int64_t cc = t.col0 + (i - C::BM);
                if (a.scale_cols && cc < cols) v = a.scale_cols[(int64_t)t.bi * cols + cc];
            }
            int e = 0;
            const double m = v > 0.0 ? frexp(v, &e) : 0.0;
            rs[i] = m > 0.0 ? 1.0 / m : 0.0;
            res[i] = e;
        }
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) tot[i][j] = f64x4{};
        lr0 = t.wm * WT * 16 + (t.lane >> 4);
        lc0 = t.wn * WT * 16 + (t.lane & 15);
        lane_off = ((int64_t)t.bi * rows + t.row0 + lr0) * cols + t.col0 + lc0;
        rows_left = (int32_t)min<int64_t>(rows - (t.row0 + lr0), 1 << 30);
        cols_left = (int32_t)min<int64_t>(cols - (t.col0 + lc0), 1 << 30);
    }

    __device__ void entry(int e, int, const FamilyPlan& plan, f64x4 (&acc)[WT][WT], const TileCtx&, uint8_t*) {
        const int pm1 = plan.e[e].p - 1;
        const TM* src = (const TM*)a.M + lane_off;
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                const bool col_ok = j * 16 < cols_left;
                const double cinv = cs[lc0 + j * 16];
                const int cexp = ces[lc0 + j * 16];
                double x[4], pw[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int roff = i * 16 + 4 * r;
                    x[r] = (col_ok && roff < rows_left)
                               ? __builtin_amdgcn_ldexp((double)src[(int64_t)roff * cols + j * 16],
                                                        -(res[lr0 + roff] + cexp)) *
                                     rs[lr0 + roff] * cinv
                               : 0.0;
                    pw[r] = 1.0;
                }
                for (int ex = pm1; ex; ex >>= 1) {
                    if (ex & 1) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) pw[r] *= x[r];
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] *= x[r];
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) tot[i][j][r] += pw[r] * acc[i][j][r];
            }
    }

    __device__ void finish(const TileCtx& t) {
        const int64_t row_base = (int64_t)t.bi * rows + t.row0 + lr0;
        const int64_t col_base = (int64_t)t.bi * cols + t.col0 + lc0;
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                if (!(j * 16 < cols_left)) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int roff = i * 16 + 4 * r;
                    if (roff < rows_left) {
                        const int64_t o = lane_off + (int64_t)roff * cols + j * 16;
                        double w = tot[i][j][r];
                        // chain factors of a balanced forward
                        if (a.out_row_mul) w *= a.out_row_mul[row_base + roff];
                        if (a.out_col_mul) w *= a.out_col_mul[col_base + j * 16];
                        if (a.out_f64)
                            ((double*)a.out)[o] = w;
                        else
                            ((float*)a.out)[o] = (float)w;
                    }
                }
            }
    }
};

// ------------------------------------------------------------ the main loop
template <class C, class Epi>
__global__ __launch_bounds__(kThreads, 2) void mt_pfamily_gemm_f64_kernel(GemmGeomF64 g,
                                                                         FamilyPlan plan,
                                                                         typename Epi::Args args) {
    constexpr int WT = C::WT;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    __shared__ int s_act[MT_MAX_P + 1];
    __shared__ int s_done[2][4];  // per wave: undecided entries (entry parity)
    __shared__ int s_open[2][4];  // per wave: of which open (entry parity)
    __shared__ uint32_t s_tail_base;

    const int tid = threadIdx.x;
    if (g.work && tid == 0) timing_span_begin(g.work);
    TileCtx t;
    t.lane = tid & 63;
    t.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    t.wm = t.wave >> 1;
    t.wn = t.wave & 1;
    const int lane = t.lane;
    const int wave = t.wave;

    int id = blockIdx.x;
    const int nwg = gridDim.x;
    if ((nwg & 7) == 0) id = (id & 7) * (nwg >> 3) + (id >> 3);
    const int per_batch = g.tiles_m * g.tiles_n;
    t.bi = id / per_batch;
    const int tt = id - t.bi * per_batch;
    constexpr int GROUP = 8;
    const int group = tt / (GROUP * g.tiles_n);
    const int first_m = group * GROUP;
    const int gsz = min(GROUP, g.tiles_m - first_m);
    const int in_g = tt - group * GROUP * g.tiles_n;
    const int tm = first_m + in_g % gsz;
    const int tn = in_g / gsz;
    t.row0 = (int64_t)tm * C::BM;
    t.col0 = (int64_t)tn * C::BM;
    const int64_t tile_id = (int64_t)t.bi * per_batch + (int64_t)tm * g.tiles_n + tn;
    if (Epi::skip_tile(args, tile_id)) return;

    Epi epi;
    epi.a = args;
    epi.setup(t, g, smem + C::PIPE_BYTES, tid);
    if (tid == 0) {
        epi.record_tile(tile_id, false);
        epi.record_count(tile_id, 0u);
    }
    // The p search starts at plan entry e0 (0: the largest p), goes down to
    // the smallest p and then up from e0 - 1 to the largest; s_act holds the
    // active plan entries in that order.
    const int e0_req = __builtin_amdgcn_readfirstlane(epi.start_index());
    const int e0 = e0_req < 0 ? 0 : (e0_req >= plan.n ? plan.n - 1 : e0_req);
    // deferred planes not written: the way down ends above them
    const int e_end = epi.down_end(plan);
    if (tid == 0) {
        int na = 0;
        for (int e = e0; e < e_end; ++e)
            if (epi.active(e, plan)) s_act[1 + na++] = e;
        for (int e = e0 - 1; e >= 0; --e)
            if (epi.active(e, plan)) s_act[1 + na++] = e;
        s_act[0] = na;
    }

    const double* Xbase = g.X + (int64_t)t.bi * g.x_batch_elems + t.row0 * g.kp;
    const double* Ybase = g.Y + (int64_t)t.bi * g.y_batch_elems + t.col0 * g.kp;
    const int nkt = (int)(g.kp / 16);

    // Operand reads: row l%16 of a 16-row block, k = 4*kk + l/16, i.e.
    // logical chunk 2*kk + l/32, half (l/16)&1; swizzle (l >> 1) & 7.
    const int32_t rd_base = (lane & 15) * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) * 16) + ((lane >> 4) & 1) * 8;

    __syncthreads();
    const int nact = __builtin_amdgcn_readfirstlane(s_act[0]);

    // Loads: instruction i of this wave fills rows R0 .. R0 + 7, R0 = (wave *
    // G + i) * 8; lane l fills row R0 + l/8, physical 16-byte chunk l%8 holding
    // logical chunk (l%8) ^ swz(row) = (l%8) ^ ((i&1)*4 + l/16).  The lane's
    // addresses are set when the loads move to the next entry and advance by
    // one K step per issue (looking the entry up for every step put an LDS
    // read and a dependent scalar load in front of each step's MFMAs).
    constexpr int G = C::BM / 32;
    int la_ = 0, ls = 0, lkt = 0, lseg = 1;
    const double *lx[G], *ly[G];
    auto set_cursor = [&]() {
        if (la_ >= nact) return;
        const PlanEntry& pe = plan.e[__builtin_amdgcn_readfirstlane(s_act[1 + la_])];
        lseg = pe.nseg;
        const double* x = Xbase + (int64_t)pe.a_plane[ls] * g.x_plane_elems;
        const double* y = Ybase + (int64_t)pe.b_plane[ls] * g.y_plane_elems;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int64_t o = (int64_t)((wave * G + i) * 8 + (lane >> 3)) * g.kp +
                              (((lane & 7) ^ ((i & 1) * 4 + (lane >> 4))) * 2);
            lx[i] = x + o;
            ly[i] = y + o;
        }
    };
    // the next K step's loads into buffer b, and the cursor one step on
    auto issue = [&](int b) {
        uint8_t* la = smem + b * C::BUF_BYTES;
        uint8_t* lb = la + C::A_BYTES;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int R0 = (wave * G + i) * 8;
            __builtin_amdgcn_global_load_lds((glb_cvoid*)lx[i], (lds_void*)(la + R0 * 128), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((glb_cvoid*)ly[i], (lds_void*)(lb + R0 * 128), 16, 0, 0);
            lx[i] += 16;
            ly[i] += 16;
        }
        if (++lkt == nkt) {
            lkt = 0;
            if (++ls == lseg) {
                ls = 0;
                ++la_;
            }
            set_cursor();
        }
    };

    set_cursor();
    if (nkt > 0 && nact > 0) issue(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    int buf = 0;
    int64_t steps_done = 0;
    for (int ai = 0; ai < nact; ++ai) {
        const int e = __builtin_amdgcn_readfirstlane(s_act[1 + ai]);
        f64x4 acc[WT][WT];
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) acc[i][j] = f64x4{};

        const int ntiles = plan.e[e].nseg * nkt;
        for (int st = 0; st < ntiles; ++st) {
            if (la_ < nact) issue(buf ^ 1);
            __builtin_amdgcn_s_setprio(1);
            const uint8_t* pa = smem + buf * C::BUF_BYTES + t.wm * WT * 16 * 128;
            const uint8_t* pb = smem + buf * C::BUF_BYTES + C::A_BYTES + t.wn * WT * 16 * 128;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int32_t ro = rd_base ^ (kk << 5);
                double a[WT], b[WT];
#pragma unroll
                for (int i = 0; i < WT; ++i) a[i] = *(const double*)(pa + i * 16 * 128 + ro);
#pragma unroll
                for (int j = 0; j < WT; ++j) b[j] = *(const double*)(pb + j * 16 * 128 + ro);
#pragma unroll
                for (int i = 0; i < WT; ++i)
#pragma unroll
                    for (int j = 0; j < WT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
            }

            __builtin_amdgcn_s_setprio(0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            buf ^= 1;
        }
        steps_done += ntiles;
        // the buffer the last step read is free until the next step's loads,
        // which wait for the barrier below
        epi.entry(e, e0, plan, acc, t, smem + (buf ^ 1) * C::BUF_BYTES);
        int lane_pre = 0;
        if (Epi::kCanStop) {
            int n_open, n_parked;
            epi.counts(n_open, n_parked);
            const int cnt = n_open + n_parked;
            int incl = cnt, incl_open = n_open;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(incl, d);
                const int yo = __shfl_up(incl_open, d);
                if (lane >= d) {
                    incl += y;
                    incl_open += yo;
                }
            }
            lane_pre = incl - cnt;
            const int wtot = __shfl(incl, 63);
            const int wopen = __shfl(incl_open, 63);
            if (lane == 0) {
                s_done[ai & 1][wave] = wtot;
                s_open[ai & 1][wave] = wopen;
            }
        }
        __syncthreads();
        if (Epi::kCanStop) {
            int total = 0, open = 0, wave_pre = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int x = s_done[ai & 1][w];
                total += x;
                open += s_open[ai & 1][w];
                wave_pre += w < wave ? x : 0;
            }
            total = __builtin_amdgcn_readfirstlane(total);
            open = __builtin_amdgcn_readfirstlane(open);
            // every entry has its p; the next entry's loads have landed
            // (vmcnt(0) above) and are left unused
            if (total == 0) break;
            // a few left: the sparse tail finishes them
            if (ai + 1 < nact && epi.can_hand_over(total)) {
                if (tid == 0) s_tail_base = epi.take_slots(tile_id, total);
                __syncthreads();
                epi.hand_over(s_tail_base + (uint32_t)(wave_pre + lane_pre), e, e0, t);
                break;
            }
            // deferred planes: entries still open after the way down (which
            // ends above the deferred p) and not handed to the tail need
            // those p; the tile runs again once their planes are written
            // (what it records meanwhile is overwritten then)
            if (e_end < plan.n && e == e_end - 1 && open > 0 && tid == 0) epi.record_tile(tile_id, true);
            // going down with nothing open left: only the entries parked at
            // the start wait, for larger p; skip to the way up (plan entry
            // e0 - 1) and reload its first K step in place of the prefetched one
            const int n_down = e_end - e0;
            if (open == 0 && e >= e0 && e0 > 0 && ai + 1 < n_down) {
                ai = n_down - 1;  // ++ai below -> first entry of the way up
                la_ = n_down;
                ls = 0;
                lkt = 0;
                set_cursor();
                if (nkt > 0) issue(buf);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
            }
        }
    }
    epi.finish(t);
    if (g.work) {
        // timed launch: the work, and the end once every wave is done
        __syncthreads();
        if (tid == 0) {
            atomicAdd(g.work, (unsigned long long)steps_done * (2ull * C::BM * C::BM * 16));
            timing_span_end(g.work);
        }
    }
}

// ------------------------------------------------------------ the sparse tail
// Handed-over entries: S_p as an FP64 dot product of the entry's X and Y plane
// rows for the plan entries from e_next on, recorded exactly as the record
// epilogue does (S, p* index; with the r = 1 projection S at the next smaller
// p in out2) for the select-root pass.
//
// Bound by the plane rows' bytes, mostly from the caches: a wave takes up to
// kTailGroup entries of one row and state together and loads the row's X
// chunks once for them (2048-vertex APSP, 11 squarings: 2.58 ms one entry at
// a time, 1.72 ms in groups of four).  Lane l sums the 2-element chunks l, l + 64,
// ... in order, U chunks loaded before any is used.
constexpr int kTailGroup = 4;
template <int N>
__device__ __forceinline__ void tail_dot_n_f64(const double* xp, const double* const (&yp)[N], int64_t kp, int lane,
                                               double (&S)[N]) {
    constexpr int U = N == 1 ? 8 : 4;
    double acc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = 0.0;
    int64_t k0 = lane * 2;
    for (; k0 + (U - 1) * 128 < kp; k0 += U * 128) {
        double2 vx[U], vy[N][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vx[u] = *(const double2*)(xp + k0 + u * 128);
#pragma unroll
            for (int q = 0; q < N; ++q) vy[q][u] = *(const double2*)(yp[q] + k0 + u * 128);
        }
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                acc[q] = fma(vx[u].x, vy[q][u].x, acc[q]);
                acc[q] = fma(vx[u].y, vy[q][u].y, acc[q]);
            }
    }
    for (; k0 < kp; k0 += 128) {
        const double2 vx = *(const double2*)(xp + k0);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const double2 vy = *(const double2*)(yp[q] + k0);
            acc[q] = fma(vx.x, vy.x, acc[q]);
            acc[q] = fma(vx.y, vy.y, acc[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) acc[q] += __shfl_xor(acc[q], d);
        S[q] = acc[q];
    }
}
// S of the active entries of a group at plan entry pe (the others' S is left).
__device__ void tail_dot_group_f64(const double* xr, const double* const (&yr)[kTailGroup],
                                   const bool (&act)[kTailGroup], const PlanEntry& pe, const GemmGeomF64& g, int lane,
                                   double (&S)[kTailGroup]) {
    const double* xp = xr + (int64_t)pe.a_plane[0] * g.x_plane_elems;
    const int64_t oy = (int64_t)pe.b_plane[0] * g.y_plane_elems;
    int n_act = 0, only = 0;
#pragma unroll
    for (int q = 0; q < kTailGroup; ++q)
        if (act[q]) {
            ++n_act;
            only = q;
        }
    if (n_act == 1) {
        const double* y = yr[0];
#pragma unroll
        for (int q = 1; q < kTailGroup; ++q)
            if (only == q) y = yr[q];
        const double* const y1[1] = {y + oy};
        double s1[1];
        tail_dot_n_f64<1>(xp, y1, g.kp, lane, s1);
#pragma unroll
        for (int q = 0; q < kTailGroup; ++q)
            if (only == q) S[q] = s1[0];
        return;
    }
    // an inactive entry repeats an active one's row (its loads hit the same
    // lines) and its sum is dropped
    const double* yp[kTailGroup];
#pragma unroll
    for (int q = 0; q < kTailGroup; ++q) {
        const double* y = yr[0];
#pragma unroll
        for (int t = 0; t < kTailGroup; ++t)
            if ((act[q] ? q : only) == t) y = yr[t];
        yp[q] = y + oy;
    }
    double Sg[kTailGroup];
    tail_dot_n_f64<kTailGroup>(xp, yp, g.kp, lane, Sg);
#pragma unroll
    for (int q = 0; q < kTailGroup; ++q)
        if (act[q]) S[q] = Sg[q];
}

template <bool R1>
__global__ __launch_bounds__(256) void mt_tail_f64_kernel(GemmGeomF64 g, FamilyPlan plan, EpiArgs a) {
    constexpr int G = kTailGroup;
    const int lane = threadIdx.x & 63;
    const uint32_t count = __builtin_amdgcn_readfirstlane(*a.tail_count);
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    // each wave takes a contiguous run of the row-sorted list
    const int64_t run = ((int64_t)count + waves - 1) / waves;
    const int64_t w0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * run;
    const int64_t w1 = min<int64_t>(w0 + run, (int64_t)count);
    double* out = (double*)a.out;
    double* out2 = (double*)a.out2;
    // deferred planes not written: an entry that reaches them marks its tile
    // for the rerun launch instead
    int n_eval = MT_MAX_P;
    if (a.low_need != nullptr && __builtin_amdgcn_readfirstlane(*a.low_need) == 0) n_eval = a.n_eval;
    const int last = plan.n - 1;
    for (int64_t w = w0; w < w1;) {
        // up to G entries of one row and state, each with the plan entry it
        // runs next (nxt, -1: done)
        const TailEntry t0 = a.tail_sorted[w];
        const int64_t row = (int64_t)t0.bi * g.rows + t0.i;
        const double* xr = g.X + (int64_t)t0.bi * g.x_batch_elems + (int64_t)t0.i * g.kp;
        const double* yr[G];
        int64_t o[G];
        int nxt[G], col[G];
        int gn = 0;
#pragma unroll
        for (int q = 0; q < G; ++q) {
            nxt[q] = -1;
            col[q] = t0.j;
            bool in = q == 0;
            if (q > 0 && gn == q && w + q < w1) {
                const TailEntry t = a.tail_sorted[w + q];
                in = t.bi == t0.bi && t.i == t0.i && t.state == t0.state;
                if (in) {
                    col[q] = t.j;
                    nxt[q] = t.e_next;
                }
            }
            if (q == 0) nxt[q] = t0.e_next;
            if (in) ++gn;
            yr[q] = g.Y + (int64_t)t0.bi * g.y_batch_elems + (int64_t)col[q] * g.kp;
            o[q] = row * g.cols + col[q];
        }
        w += gn;
        auto mark = [&](int q) {
            if (lane == 0) {
                a.missed_tile[((int64_t)t0.bi * g.tiles_m + t0.i / g.bm) * g.tiles_n + col[q] / g.bm] = 1u;
                *a.low_missed = 1;
            }
        };
        bool act[G];
        double S[G];
        if (!R1 && t0.state == kTailRise) {
            // stable at e_next + 1 (recorded): go up while a larger p may be
            // stable too; an unstable p leaves the record below standing
            while (true) {
                int e = -1;
#pragma unroll
                for (int q = 0; q < G; ++q) e = max(e, nxt[q]);
                if (e < 0) break;
#pragma unroll
                for (int q = 0; q < G; ++q) act[q] = nxt[q] == e;
                const PlanEntry& pe = plan.e[e];
                tail_dot_group_f64(xr, yr, act, pe, g, lane, S);
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    if (!act[q]) continue;
                    nxt[q] = -1;
                    if (!(S[q] >= plan.tau)) continue;
                    if (lane == 0) {
                        out[o[q]] = S[q];
                        a.pstar[o[q]] = (uint8_t)pe.pidx;
                    }
                    if (S[q] >= pe.rise_thr) nxt[q] = e - 1;
                }
            }
            continue;
        }
        // going down from e_next.  An entry whose S is exactly 0 (every term 0
        // or underflowed: pairs a sparse APSP operand does not connect) looks
        // at the smallest p, once and where its planes are written: if S is
        // below tau there too, no p between them is stable, since S_p does not
        // grow with p for terms in [0, 1]; otherwise it goes on from where it
        // was (back).
        constexpr int kNotLooked = -1, kLooked = -2;
        bool pend[G];
        int back[G];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            pend[q] = R1 && t0.state == kTailR1;
            back[q] = kNotLooked;
        }
        while (true) {
            int e = MT_MAX_P;
#pragma unroll
            for (int q = 0; q < G; ++q)
                if (nxt[q] >= 0) e = min(e, nxt[q]);
            if (e >= MT_MAX_P) break;
#pragma unroll
            for (int q = 0; q < G; ++q) act[q] = nxt[q] == e;
            if (e >= n_eval) {
#pragma unroll
                for (int q = 0; q < G; ++q)
                    if (act[q]) {
                        mark(q);
                        nxt[q] = -1;
                    }
                continue;
            }
            const PlanEntry& pe = plan.e[e];
            tail_dot_group_f64(xr, yr, act, pe, g, lane, S);
#pragma unroll
            for (int q = 0; q < G; ++q) {
                if (!act[q]) continue;
                if (R1 && pend[q]) {
                    if (lane == 0) out2[o[q]] = S[q];
                    nxt[q] = -1;
                    continue;
                }
                const bool stable = S[q] >= plan.tau;
                if (back[q] >= 0 && stable) {
                    // stable at the smallest p after all: the p in between
                    nxt[q] = back[q] + 1;
                    back[q] = kLooked;
                    continue;
                }
                if (!(stable || e == last)) {
                    nxt[q] = e + 1;
                    if (!R1 && S[q] == 0.0 && back[q] == kNotLooked && e + 1 < last && last < n_eval) {
                        back[q] = e;
                        nxt[q] = last;
                    }
                    continue;
                }
                if (lane == 0) {
                    out[o[q]] = S[q];
                    a.pstar[o[q]] = stable ? (uint8_t)pe.pidx : (uint8_t)MT_PSTAR_NONE;
                }
                nxt[q] = -1;
                if (R1 && stable && pe.inv_dp > 0.f) {
                    pend[q] = true;
                    nxt[q] = e + 1;
                }
            }
        }
    }
}

template <class C, class Epi>
hipError_t launch_gemm(const GemmGeomF64& g, int64_t b, const FamilyPlan& plan,
                       const typename Epi::Args& args, const char* name, hipStream_t st) {
    const int lds = C::PIPE_BYTES + Epi::LDS_BYTES;
    auto kern = mt_pfamily_gemm_f64_kernel<C, Epi>;
    // the dynamic-LDS limit is a per-device attribute of the kernel
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
    const int64_t nwg = b * (int64_t)g.tiles_m * g.tiles_n;
    timing_before(name, st);
    GemmGeomF64 gw = g;
    gw.work = timing_work_slot();
    hipLaunchKernelGGL(kern, dim3((unsigned)nwg), dim3(kThreads), lds, st, gw, plan, args);
    timing_after(st);
    return hipGetLastError();
}

GemmGeomF64 make_geom(const double* X, const double* Y, int64_t rows, int64_t cols, int64_t rows_pad,
                      int64_t cols_pad, int64_t kp, int32_t x_planes, int32_t y_planes, int bm) {
    GemmGeomF64 g;
    g.X = X;
    g.Y = Y;
    g.x_plane_elems = rows_pad * kp;
    g.y_plane_elems = cols_pad * kp;
    g.x_batch_elems = g.x_plane_elems * x_planes;
    g.y_batch_elems = g.y_plane_elems * y_planes;
    g.kp = kp;
    g.rows = rows;
    g.cols = cols;
    g.tiles_m = (int32_t)(rows_pad / bm);
    g.tiles_n = (int32_t)(cols_pad / bm);
    g.bm = bm;
    g.work = nullptr;
    return g;
}

}  // namespace

hipError_t launch_pfamily_gemm_f64(const double* Ap, const double* Bp, int64_t b, int64_t m,
                                   int64_t n, int64_t mp, int64_t np, int64_t kp, int32_t n_planes,
                                   int bm, const FamilyPlan& plan, const EpiArgs& epi,
                                   hipStream_t st) {
    const GemmGeomF64 g = make_geom(Ap, Bp, m, n, mp, np, kp, n_planes, n_planes, bm);
    const char* name = "mt_pfamily_gemm_f64";
    hipError_t e = hipErrorInvalidValue;
    if (epi.mode == EPI_STORE_ALL) {
        if (bm == 128) return launch_gemm<CfgF64<4>, StoreAllEpi<CfgF64<4>>>(g, b, plan, epi, name, st);
        if (bm == 64) return launch_gemm<CfgF64<2>, StoreAllEpi<CfgF64<2>>>(g, b, plan, epi, name, st);
        return e;
    }
    if (bm == 128)
        e = plan.r1 ? launch_gemm<CfgF64<4>, RecordEpi<CfgF64<4>, true>>(g, b, plan, epi, name, st)
                    : launch_gemm<CfgF64<4>, RecordEpi<CfgF64<4>, false>>(g, b, plan, epi, name, st);
    else if (bm == 64)
        e = plan.r1 ? launch_gemm<CfgF64<2>, RecordEpi<CfgF64<2>, true>>(g, b, plan, epi, name, st)
                    : launch_gemm<CfgF64<2>, RecordEpi<CfgF64<2>, false>>(g, b, plan, epi, name, st);
    if (e != hipSuccess || !epi.tail) return e;
    // the sparse tail for the entries the tiles handed over
    const int64_t cap = (int64_t)epi.tail_max * b * g.tiles_m * g.tiles_n;
    e = launch_tail_sort(epi, b * g.tiles_m, g.tiles_n, bm, st);
    if (e != hipSuccess) return e;
    int64_t blocks = (cap + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    timing_before("mt_tail_f64", st);
    if (plan.r1)
        hipLaunchKernelGGL(mt_tail_f64_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, g, plan, epi);
    else
        hipLaunchKernelGGL(mt_tail_f64_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, g, plan, epi);
    timing_after(st);
    return hipGetLastError();
}

hipError_t launch_rerun_gemm_f64(const double* Ap, const double* Bp, int64_t b, int64_t m, int64_t n, int64_t mp,
                                 int64_t np, int64_t kp, int32_t n_planes, int bm, const FamilyPlan& plan,
                                 const EpiArgs& epi, hipStream_t st) {
    if (epi.missed_tile == nullptr || plan.r1 || epi.mode == EPI_STORE_ALL) return hipErrorInvalidValue;
    const GemmGeomF64 g = make_geom(Ap, Bp, m, n, mp, np, kp, n_planes, n_planes, bm);
    // a launch of its own name: the forward GEMM's timing and work stay apart
    // (a tile that is not marked adds no work and ends no span)
    const char* name = "mt_rerun_gemm_f64";
    if (bm == 128) return launch_gemm<CfgF64<4>, RecordEpi<CfgF64<4>, false, true>>(g, b, plan, epi, name, st);
    if (bm == 64) return launch_gemm<CfgF64<2>, RecordEpi<CfgF64<2>, false, true>>(g, b, plan, epi, name, st);
    return hipErrorInvalidValue;
}

hipError_t launch_adjoint_gemm_f64(const double* Xp, const double* Yp, int64_t b, int64_t rows,
                                   int64_t cols, int64_t rows_pad, int64_t cols_pad, int64_t kp,
                                   int32_t x_planes, int32_t y_planes, const FamilyPlan& plan,
                                   const AdjArgs& adj, hipStream_t st) {
    using CA = CfgF64<2>;
    static_assert(CA::BM == kAdjF64BM, "adjoint tile");
    const GemmGeomF64 g = make_geom(Xp, Yp, rows, cols, rows_pad, cols_pad, kp, x_planes, y_planes, CA::BM);
    const char* name = "mt_adjoint_gemm_f64";
    if (adj.m_f64) return launch_gemm<CA, AdjointEpiF64<CA, double>>(g, b, plan, adj, name, st);
    return launch_gemm<CA, AdjointEpiF64<CA, float>>(g, b, plan, adj, name, st);
}

}  // namespace mt
