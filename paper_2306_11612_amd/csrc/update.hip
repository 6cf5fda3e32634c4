// Per-update kernels of dynamic volume lines (Eqs. 1-4 and section
// "Projecting Cells to 1D" of Zellmann et al., arXiv 2306.11612), over a
// batch of requests (a request = one volume, its TFs and parameters).
//
//   K0 k_vmax_exact   (DVL_VMAX_EXACT requests only) max over cells of V_h
//   K1 k_tile_sums    TF lookup, V_h (Eq. 1) and importance f (Eq. 3) of every
//                     cell; fp64 sum of f per tile; each wave owns a run of
//                     consecutive tiles and records their prefix inside it
//   K2 + K3a k_carry_classify (one kernel)
//                     K2: exclusive scan of the run totals (Eq. 4 across runs;
//                     fp64 or compensated fp32), made monotone; K3a, per
//                     tile, one lane each: its pixel position; if its pixel
//                     interval lies inside one bin, the whole tile is that
//                     bin's part
//   K3b k_bin         per tile holding a bin edge: recompute f, monotone
//                     in-tile prefix, pixel interval of every cell; the cell
//                     range of every bin that starts and ends inside the
//                     tile, and of the tile's first and last bin (per-tile
//                     records)
//   K4 k_bin_stats    per (request, bin): the bin's cell range (merged from
//                     the records of the tiles it touches), then its mean,
//                     min and max per field from the values of its partial
//                     end segments and the statistics of the segments and
//                     tiles it covers whole; the height
//
// The paper's GPU version runs the projection once per field with global
// atomics on the W bins (its Table 1 bottleneck).  Here the projection is
// hierarchical over tiles (the paper's future-work suggestion): only tiles
// that contain a bin edge are read again, to find where bins start and end;
// no atomics on bins, and the statistics of a bin cost work in proportion to
// its two ends, not to its cells.  Results are bitwise deterministic and do
// not depend on what else is in the batch.
//
// K0, K1, K3b and K4 depend on the field storage type and the field count;
// they live in update_kernels.hpp and are instantiated once per (type,
// count) in translation units the build generates.  This file holds K2, K3a,
// the TF entry cache builder and the launcher.
#include "update_kernels.hpp"

namespace dvl {

// ------------------------------------------------------------------ workspace

static inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t workspace_bytes(int64_t T, int M, int W, int64_t fcells) {
    size_t b = 0;
    b += al256((size_t)T * 8);             // local_prefix
    b += al256((size_t)T * 8);             // run_total
    b += al256((size_t)(T + 1) * 4);       // tile positions
    b += 2 * al256((size_t)T * 4);         // head/tail bin
    b += 2 * al256((size_t)2 * T * 4);     // rec first/last
    b += 2 * al256((size_t)W * 4);         // per-bin tile bounds
    b += al256((size_t)W * sizeof(EdgeRec));
    b += al256(8 * 8);                     // scalars
    b += al256((size_t)fcells * 4);        // stored importance
    return b;
}

void workspace_carve(void* base, int64_t T, int M, int W, int64_t fcells, UpdWorkspace* w) {
    char* p = (char*)base;
    auto take = [&](size_t bytes) { char* q = p; p += al256(bytes); return (void*)q; };
    w->local_prefix = (double*)take((size_t)T * 8);
    w->run_total = (double*)take((size_t)T * 8);
    w->x0 = (float*)take((size_t)(T + 1) * 4);
    w->head_bin = (int32_t*)take((size_t)T * 4);
    w->tail_bin = (int32_t*)take((size_t)T * 4);
    w->rec_first = (uint32_t*)take((size_t)2 * T * 4);
    w->rec_last = (uint32_t*)take((size_t)2 * T * 4);
    w->bin_t1 = (int32_t*)take((size_t)W * 4);
    w->bin_ta = (int32_t*)take((size_t)W * 4);
    w->edge = (EdgeRec*)take((size_t)W * sizeof(EdgeRec));
    w->scal = (double*)take(8 * 8);
    w->fstore = fcells ? (float*)take((size_t)fcells * 4) : nullptr;
}

// ------------------------------------------------------------------ K2

struct AccF64 {
    double v;
    __device__ static AccF64 zero() { return {0.0}; }
    __device__ void add(double x) { v += x; }
    __device__ static AccF64 combine(const AccF64& a, const AccF64& b) { return {a.v + b.v}; }
    __device__ double value() const { return v; }
    __device__ AccF64 shfl_up(int d) const { return {shfl_up_d(v, d)}; }
};

// compensated fp32: unevaluated sum hi + lo, error-free TwoSum on every add
struct AccKahan32 {
    float hi, lo;
    __device__ static AccKahan32 zero() { return {0.0f, 0.0f}; }
    __device__ static void two_sum(float a, float b, float& s, float& e) {
        s = a + b;
        const float bb = s - a;
        e = (a - (s - bb)) + (b - bb);
    }
    __device__ void add(double xd) {
        const float x = (float)xd;
        float s, e;
        two_sum(hi, x, s, e);
        lo += e;
        two_sum(s, lo, hi, lo);
    }
    __device__ static AccKahan32 combine(const AccKahan32& a, const AccKahan32& b) {
        float s, e;
        two_sum(a.hi, b.hi, s, e);
        AccKahan32 r;
        const float l = e + (a.lo + b.lo);
        two_sum(s, l, r.hi, r.lo);
        return r;
    }
    __device__ double value() const { return (double)hi + (double)lo; }
    __device__ AccKahan32 shfl_up(int d) const { return {shfl_up_f(hi, d), shfl_up_f(lo, d)}; }
};

struct AccF32 {
    float v;
    __device__ static AccF32 zero() { return {0.0f}; }
    __device__ void add(double x) { v += (float)x; }
    __device__ static AccF32 combine(const AccF32& a, const AccF32& b) { return {a.v + b.v}; }
    __device__ double value() const { return (double)v; }
    __device__ AccF32 shfl_up(int d) const { return {shfl_up_f(v, d)}; }
};

constexpr int kCarryThreads = 1024;
constexpr int kCarryItems = 8;                              // run totals per thread and round
constexpr int kCarryRound = kCarryThreads * kCarryItems;
constexpr int kCarryWaves = kCarryThreads / kWave;

// Bases of the runs a classifying workgroup needs (its 1024 tiles touch at
// most 1025 runs and the base after them).
constexpr int kClassifyTiles = kCarryThreads;
constexpr int kRunBases = kClassifyTiles + 2;
struct TileSpan {
    float x0, x1;                   // pixel positions of the tile's ends
};

// The exclusive scan of request q's R run totals, by the whole workgroup:
// base[r] = sum of the run totals before r for the runs r_lo .. r_hi + 1 (into
// LDS), and F_tot, the base after the last run.  A sequential prefix over each
// thread's 8 totals, a wave scan of the thread totals made monotone by a
// running maximum, and sequential wave and round bases; every base is clamped
// to the next thread's base, so the bases never decrease.
template <typename Acc>
__device__ __forceinline__ double carry_scan(const double* run_total, int R, int r_lo, int r_hi, double* base) {
    __shared__ double wave_base[kCarryWaves + 1];
    __shared__ Acc wave_acc[kCarryWaves];
    __shared__ Acc round_acc;
    __shared__ double round_end;
    const int tid = thread_x(), lane = lane_id(), w = tid / kWave;
    if (tid == 0) {
        round_acc = Acc::zero();
        round_end = 0.0;
    }
    __syncthreads();
    for (int r0 = 0; r0 < R; r0 += kCarryRound) {
        const int b0 = r0 + tid * kCarryItems;
        double v[kCarryItems];
#pragma unroll
        for (int k = 0; k < kCarryItems; ++k) v[k] = (b0 + k < R) ? gload<double>(run_total, b0 + k) : 0.0;
        Acc pre[kCarryItems];
        Acc run = Acc::zero();
#pragma unroll
        for (int k = 0; k < kCarryItems; ++k) {
            pre[k] = run;
            run.add(v[k]);
        }
        Acc inc = run;
        for (int d = 1; d < kWave; d <<= 1) {
            const Acc o = inc.shfl_up(d);
            if (lane >= d) inc = Acc::combine(o, inc);
        }
        if (lane == kWave - 1) wave_acc[w] = inc;
        __syncthreads();
        if (tid == 0) {
            Acc acc[kCarryWaves];
#pragma unroll
            for (int k = 0; k < kCarryWaves; ++k) acc[k] = wave_acc[k];
            Acc sum = round_acc;
            double prev = round_end;
#pragma unroll
            for (int k = 0; k < kCarryWaves; ++k) {
                prev = fmax(prev, sum.value());
                wave_base[k] = prev;
                sum = Acc::combine(sum, acc[k]);
            }
            prev = fmax(prev, sum.value());
            wave_base[kCarryWaves] = prev;
            round_end = prev;
            round_acc = sum;
        }
        __syncthreads();
        const double wb = wave_base[w], wn = wave_base[w + 1];
        const Acc exc = inc.shfl_up(1);
        double tb = lane == 0 ? wb : fmin(fmax(wb + exc.value(), wb), wn);
        for (int d = 1; d < kWave; d <<= 1) {
            const double o = shfl_up_d(tb, d);
            if (lane >= d) tb = fmax(tb, o);
        }
        const int src = lane + 1 < kWave ? lane + 1 : lane;
        const uint64_t u = __double_as_longlong(tb);
        const int nlo = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)u);
        const int nhi = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)(u >> 32));
        double nb = __longlong_as_double(((uint64_t)(uint32_t)nhi << 32) | (uint32_t)nlo);
        if (lane == kWave - 1) nb = wn;
        double c = tb;
#pragma unroll
        for (int k = 0; k < kCarryItems; ++k) {
            c = fmax(c, fmin(tb + pre[k].value(), nb));
            const int r = b0 + k;
            if (r < R && r >= r_lo && r <= r_hi + 1) base[r - r_lo] = c;
        }
        __syncthreads();
    }
    const double total = round_end;
    if (tid == 0 && r_hi + 1 >= R) base[R - r_lo] = total;
    __syncthreads();
    return total;
}

// Grid: x chunks of 1024 tiles, y requests.  Every workgroup scans its
// request's run totals itself (at most 8192 in the default layout: 64 KB from
// L2, the same code on the same inputs, so the same bits) and keeps the bases
// of its own runs in LDS: one kernel with no hand-off.  (One scanning
// workgroup per request that published its carry through a flag, polled by
// the others, took 8.5 us for 64 tiles, 11.4 for 2880 and 20 for 122363; this
// takes 6.3, 6.7 and 9.6.)
//
// K3a, a tile per thread.  A tile whose pixel interval lies inside one bin
// puts every cell in that bin: its head record is the whole tile and no cell
// is read (the projection is hierarchical over tiles).  The others are K3b's.
// Every tile also writes, for the bins its interval reaches, where K4 finds
// their tiles: with b0(t) = bin of X0(t) (the bin of the tile's first cell)
// and b1(t) = bin of X1(t) = b0(t + 1), the last tile touching bin b is the
// t with b0(t) <= b < b1(t) (bin_t1, the last tile: b0 <= b), and the first
// is the t with b1(t - 1) < b <= b1(t) (bin_ta, the first tile: b <= b1),
// or the next tile when tile t's last cell ends exactly at bin b's left edge
// (K4 checks it with the tile's tail bin).  These ranges partition the bins.
// A tile's first inner edge also gets the tile's record: K3b's worklist.
// FAR: with many bins per tile (far_tiles) the workgroup's waves write them
// together, a tile after another, a lane per bin.  (One cell plotted 4096 / 2^20
// wide, a lane each here and in the rescan: 0.52 / 124 ms; now 0.047 / 3.1, 0.26 M
// cells 2^20 wide 2.4 -> 0.7 ms.)
template <bool FAR>
__global__ __launch_bounds__(kCarryThreads) void k_carry_classify(BatchDev bd) {
    __shared__ double base[kRunBases];
    __shared__ TileSpan span[FAR ? kClassifyTiles : 1];
    const ReqDev& q = bd.reqs[block_y()];
    const VolDev& v = q.v;
    const int T = uni(v.n_tiles), tpr = uni(v.tiles_per_run), R = uni(v.n_runs);
    const int t0 = block_x() * kClassifyTiles;
    if (t0 >= T) return;
    const int64_t n = uni(v.n);
    const int t = t0 + thread_x();
    const int t_last = min(t0 + kClassifyTiles, T) - 1;
    const int r_lo = t0 / tpr, r_hi = min((t_last + 1) / tpr, R - 1);
    // in-run prefixes of this tile and the next, on their way during the scan
    const double lp = t < T ? gload<double>(q.ws.local_prefix, t) : 0.0;
    const double lp_next = t + 1 < T ? gload<double>(q.ws.local_prefix, t + 1) : 0.0;
    const int mode = uni(q.scan_mode);
    const double* run_total = uni(q.ws.run_total);
    double total;
    if (mode == DVL_SCAN_KAHAN_FP32)
        total = carry_scan<AccKahan32>(run_total, R, r_lo, r_hi, base);
    else if (mode == DVL_SCAN_NAIVE_FP32)
        total = carry_scan<AccF32>(run_total, R, r_lo, r_hi, base);
    else
        total = carry_scan<AccF64>(run_total, R, r_lo, r_hi, base);
    // a zero total means every f was zero: fall back to f = 1 (linear map; the
    // tile offsets then follow from the cell counts)
    const bool degenerate = !(total > 0.0);
    const double f_tot = degenerate ? (double)n : total;
    const int W = uni(q.W);
    const double scale = (double)W / f_tot;
    if (t0 == 0 && thread_x() == 0) {
        gstore<double>(q.ws.scal, 0, f_tot);
        gstore<double>(q.ws.scal, 1, degenerate ? 1.0 : 0.0);
        gstore<double>(q.ws.scal, 2, scale);
    }
    if (!FAR && t >= T) return;
    const int64_t tile_cells = (int64_t)uni(v.tile_steps) * kStepCells;
    // Sum of the importance of all tiles before tile u (u = T gives F_tot):
    // the run's base plus the tile's prefix inside its run, never above the
    // next run's base.  The same for both neighbours of a tile boundary, and
    // the offsets never decrease.
    auto offset = [&](int u, double prefix) -> double {
        if (degenerate) return u >= T ? (double)n : (double)(u * tile_cells);
        if (u >= T) return total;
        const int r = u / tpr - r_lo;
        const double lo = base[r], hi = base[r + 1];
        return fmin(fmax(lo + prefix, lo), hi);
    };
    const float X0 = (float)(offset(t, lp) * scale), X1 = (float)(offset(t + 1, lp_next) * scale);
    bool shared_bins = false;
    if constexpr (FAR) {
        shared_bins = far_tiles(T, W);
        if (shared_bins) {
            // by all waves, a tile after another (as many bins as tiles: no edge records)
            const int W1 = W - 1;
            int32_t* const t1 = uni(q.ws.bin_t1);
            int32_t* const ta = uni(q.ws.bin_ta);
            span[thread_x()] = TileSpan{X0, X1};
            __syncthreads();
            for (int i = thread_x() / kWave; i < t_last + 1 - t0; i += kCarryWaves) {
                const int u = t0 + i, c0 = bin_of(span[i].x0, W1), c1 = bin_of(span[i].x1, W1), end = u == T - 1 ? W : c1 + 1;
                for (int b = (u == 0 ? 0 : c0) + lane_id(); b < end; b += kWave) {
                    if (b >= c0 && (b < c1 || u == T - 1)) gstore<int32_t>(t1, b, u);
                    if (b > c0 || u == 0) gstore<int32_t>(ta, b, u);
                }
            }
        }
        if (t >= T) return;
    }
    gstore<float>(q.ws.x0, t, X0);
    const bool last_tile = t == T - 1;
    if (last_tile) gstore<float>(q.ws.x0, T, X1);
    const int W1 = W - 1;
    const int b0 = bin_of(X0, W1), b1 = bin_of(X1, W1);
    const bool edges = !uni(q.by_tile);
    int32_t* const t1 = uni(q.ws.bin_t1);
    int32_t* const ta = uni(q.ws.bin_ta);
    EdgeRec* const edge = uni(q.ws.edge);
    auto upto = [&](int b, int tile) {        // tile t ends in bin >= b
        gstore<int32_t>(ta, b, t);
        if (edges) gstore<u32x4>(edge, b, u32x4{(uint32_t)tile, __float_as_uint(X0), __float_as_uint(X1), 0u});
    };
    if (!shared_bins) {
        for (int b = b0; b < b1; ++b) {
            gstore<int32_t>(t1, b, t);
            upto(b + 1, b == b0 ? t : -1);
        }
        if (t == 0)
            for (int b = 0; b <= b0; ++b) upto(b, -1);
        if (last_tile)
            for (int b = b1; b <= W1; ++b) {
                gstore<int32_t>(t1, b, t);
                if (b > b1) upto(b, -1);
            }
    }
    if (b0 == b1) {
        const int64_t tbase = t * tile_cells;
        gstore<uint32_t>(q.ws.rec_first, t, (uint32_t)tbase);
        gstore<uint32_t>(q.ws.rec_last, t, (uint32_t)(min(tbase + tile_cells, n) - 1));
        gstore<int32_t>(q.ws.head_bin, t, b0);
        gstore<int32_t>(q.ws.tail_bin, t, b0);
    }
}

// ------------------------------------------------------------------ TF entry cache

// entries of 4 consecutive cells per lane, packed into one 32-bit store
template <typename S>
__global__ __launch_bounds__(256) void k_build_index(int64_t n_quads, const void* __restrict__ field, float s,
                                                     float b, float nmax, uint32_t* __restrict__ out) {
    const int64_t stride = (int64_t)grid_dim_x() * block_dim_x();
    for (int64_t i = (int64_t)block_x() * block_dim_x() + thread_x(); i < n_quads; i += stride) {
        Quad<S> q;
        q.load(field, i);
        uint32_t w = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) w |= (uint32_t)tf_entry(q.get(k), s, b, nmax) << (8 * k);
        out[i] = w;
    }
}

dvl_status launch_build_index(int64_t n_pad, int dtype, const void* field, float s, float b, int n_tf,
                              uint8_t* out, int n_cu, hipStream_t st) {
    const int64_t n_quads = n_pad / 4;
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n_quads + 255) / 256, (int64_t)n_cu * 16));
    const float nmax = (float)(n_tf - 1);
    if (dtype == DVL_F16)
        hipLaunchKernelGGL(k_build_index<F16>, dim3(grid), dim3(256), 0, st, n_quads, field, s, b, nmax, (uint32_t*)out);
    else if (dtype == DVL_BF16)
        hipLaunchKernelGGL(k_build_index<BF16>, dim3(grid), dim3(256), 0, st, n_quads, field, s, b, nmax, (uint32_t*)out);
    else
        hipLaunchKernelGGL(k_build_index<F32>, dim3(grid), dim3(256), 0, st, n_quads, field, s, b, nmax, (uint32_t*)out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// ------------------------------------------------------------------ launchers

dvl_status launch_carry_classify(const BatchDev& b, bool far, hipStream_t s) {
    const int blocks = (b.max_tiles + kClassifyTiles - 1) / kClassifyTiles;
    return far ? launch_rows<k_carry_classify<true>>(b, blocks, kCarryThreads, 0, s)
               : launch_rows<k_carry_classify<false>>(b, blocks, kCarryThreads, 0, s);
}

dvl_status launch_batch(const BatchLaunch& b, int dtype, int max_m, int n_cu, hipStream_t s, uint64_t layout,
                        hipEvent_t* ev) {
    if (layout != kDescriptorLayout) {
        set_error("descriptor layout mismatch between library objects (%llx vs %llx): rebuild the library",
                  (unsigned long long)layout, (unsigned long long)kDescriptorLayout);
        return DVL_E_INVALID;
    }
    if (dtype == DVL_F16) return launch_s<F16>(b, max_m, n_cu, s, layout, ev);
    if (dtype == DVL_BF16) return launch_s<BF16>(b, max_m, n_cu, s, layout, ev);
    return launch_s<F32>(b, max_m, n_cu, s, layout, ev);
}

}  // namespace dvl
