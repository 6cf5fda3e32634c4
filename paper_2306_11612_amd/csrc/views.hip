// Views of an update's bins beyond the lines themselves:
//
//   k_bin_histograms  per bin, the histogram of one field's values over its
//                     cells (the histogram heatmap of volume-line plots;
//                     paper section Prototypical User Interface)
//   k_rasterize       the lines drawn as polylines or bar charts into an
//                     image (the paper's RasterizeLines kernel, GPU section)
//   k_select_mask     brushing and linking: which cells (original order) have
//                     a Hilbert key inside one of the selected key ranges
//                     (paper section Brushing and Linking: regions of
//                     interest travel to the 3D view as Hilbert-code ranges)
#include "views.hpp"

#include <algorithm>

namespace dvl {

// ------------------------------------------------------------------ histograms

// One workgroup per bin (grid-stride over bins): the bin's sorted cells
// first..last are counted into an LDS histogram of H buckets; the bucket of a
// value is its entry under the quantiser of [lo, hi] for H entries (the TF entry
// rule), so the counts are exact integers independent of the order of the
// additions.  QUADS: streamed as aligned vectors of four, four in flight per
// thread; else a cell per thread.  Neighbouring cells mostly share a bucket, and
// the LDS adds equal addresses one after another: C copies of every counter lie
// in different banks and the lanes take them in turn (the rules are at
// histograms_typed).  11.8 M fp32 cells, 1920 bins, 64 buckets: 12.5 us, 3.8 TB/s
// (one load at a time and one copy: 50).
template <typename S, int C, bool QUADS>
__global__ __launch_bounds__(256) void k_bin_histograms(const typename S::raw* __restrict__ v, int32_t W,
                                                        const uint32_t* __restrict__ first,
                                                        const uint32_t* __restrict__ last, int32_t H,
                                                        float s, float b, uint32_t* __restrict__ counts) {
    extern __shared__ uint32_t hist[];   // [H][C]
    const float nmax = (float)(H - 1);
    const uint32_t copy = threadIdx.x & (C - 1);
    constexpr int kAhead = 4;
    for (int32_t bin = blockIdx.x; bin < W; bin += gridDim.x) {
        for (int32_t k = threadIdx.x; k < H * C; k += blockDim.x) hist[k] = 0u;
        __syncthreads();
        const uint32_t f = first[bin], l = last[bin];
        auto bucket = [&](float x) {
            return (uint32_t)(int)fminf(fmaxf(fmaf(x, s, b), 0.0f), nmax) * C + copy;
        };
        if (!QUADS && f <= l) {
            for (uint64_t h = (uint64_t)f + threadIdx.x; h <= (uint64_t)l; h += 256) atomicAdd(&hist[bucket(to_f32(S{}, v[h]))], 1u);
        } else if (f <= l) {
            const uint32_t q1 = l >> 2;
            for (uint64_t q0 = (f >> 2) + threadIdx.x; q0 <= q1; q0 += kAhead * 256) {
                Quad<S> d[kAhead];
#pragma unroll
                for (int g = 0; g < kAhead; ++g)
                    if (q0 + g * 256 <= q1) d[g].load(v, (int64_t)(q0 + g * 256));
#pragma unroll
                for (int g = 0; g < kAhead; ++g) {
                    if (q0 + g * 256 > q1) break;
                    const uint32_t c = (uint32_t)(q0 + g * 256) << 2;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (c + k < f || c + k > l) continue;
                        atomicAdd(&hist[bucket(d[g].get(k))], 1u);
                    }
                }
            }
        }
        __syncthreads();
        for (int32_t k = threadIdx.x; k < H; k += blockDim.x) {
            uint32_t sum = 0;
#pragma unroll
            for (int q = 0; q < C; ++q) sum += hist[k * C + q];
            counts[(int64_t)bin * H + k] = sum;
        }
        __syncthreads();
    }
}

// By the cells of a bin on average.  Eight copies of the counters pay where they
// are many more than it costs to clear and add the copies (16 H operations), and
// while their LDS lets eight workgroups run on a compute unit (H <= 512): 50 M
// fp32 cells, eight copies / one, 6.5 H cells a bin, H = 256 58 / 76 us, 3 H, H =
// 256 102 / 86, 3.3 H, H = 512 89 / 70; for few buckets from 64 cells on (100
// cells, H = 1 253 / 296, 47 cells 506 / 495).  Vectors of four pay from 256 cells
// on, whose quarter still fills a wave (vectors / single, 400 cells, H = 512 135 /
// 154, 200 cells, H = 256 203 / 197, 4 cells 44 / 37).
template <typename S>
static void histograms_typed(const void* field, int64_t n, int32_t W, const uint32_t* first, const uint32_t* last,
                             int32_t H, float s, float b, uint32_t* counts, int n_cu, hipStream_t st) {
    const dim3 grid((unsigned)std::max(1, std::min(W, n_cu * 16)));
    const auto* v = (const typename S::raw*)field;
    const size_t lds = (size_t)H * sizeof(uint32_t);
    if (H <= 512 && n >= W * std::max<int64_t>(64, 4 * H))
        hipLaunchKernelGGL((k_bin_histograms<S, 8, true>), grid, dim3(256), 8 * lds, st, v, W, first, last, H, s, b, counts);
    else if (n >= (int64_t)W * 256)
        hipLaunchKernelGGL((k_bin_histograms<S, 1, true>), grid, dim3(256), lds, st, v, W, first, last, H, s, b, counts);
    else
        hipLaunchKernelGGL((k_bin_histograms<S, 1, false>), grid, dim3(256), lds, st, v, W, first, last, H, s, b, counts);
}

dvl_status launch_bin_histograms(int dtype, const void* field, int64_t n, int32_t W, const uint32_t* first,
                                 const uint32_t* last, int32_t H, float s, float b, uint32_t* counts,
                                 int n_cu, hipStream_t st) {
    if (dtype == DVL_F16)
        histograms_typed<F16>(field, n, W, first, last, H, s, b, counts, n_cu, st);
    else if (dtype == DVL_BF16)
        histograms_typed<BF16>(field, n, W, first, last, H, s, b, counts, n_cu, st);
    else
        histograms_typed<F32>(field, n, W, first, last, H, s, b, counts, n_cu, st);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// ------------------------------------------------------------------ raster

// the row of a height y in [0, 1] on H rows (row 0 at the bottom)
__device__ __forceinline__ int raster_row(float y, int H) {
    const float t = y * (float)H;
    if (!(t >= 0.0f)) return 0;
    return min((int)floorf(t), H - 1);
}

// One thread per pixel (row-major image, rows of W pixels, coalesced along
// a row).  Polyline: column b spans the rows between its height's row and
// the next column's; bars: rows 0 .. its height's row.  `y` holds the
// heights of `lines` lines, one after another (W each); image l is at
// img + l * H * W.
__global__ __launch_bounds__(256) void k_rasterize(const float* __restrict__ y, int32_t W, int32_t H,
                                                   int32_t lines, int32_t mode, uint8_t* __restrict__ img) {
    const int64_t total = (int64_t)lines * H * W;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const int64_t l = i / ((int64_t)H * W);
        const int64_t p = i - l * H * W;
        const int r = (int)(p / W), b = (int)(p - (int64_t)r * W);
        const float* yl = y + l * W;
        const int r0 = raster_row(yl[b], H);
        int lo, hi;
        if (mode == kRasterBars) {
            lo = 0;
            hi = r0;
        } else {
            const int r1 = b + 1 < W ? raster_row(yl[b + 1], H) : r0;
            lo = min(r0, r1);
            hi = max(r0, r1);
        }
        img[i] = (r >= lo && r <= hi) ? 1 : 0;
    }
}

dvl_status launch_rasterize(const float* y, int32_t W, int32_t H, int32_t lines, int32_t mode, uint8_t* img,
                            hipStream_t st) {
    const int64_t total = (int64_t)lines * H * W;
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 65536));
    hipLaunchKernelGGL(k_rasterize, dim3(grid), dim3(256), 0, st, y, W, H, lines, mode, img);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// ------------------------------------------------------------------ brushing

// 1 at the original index of every cell whose key lies in one of the n_ranges
// closed ranges [lo[i], hi[i]], else 0.  The keys are sorted, so a chunk of cells
// is compared by its first and last key first, two ranges per lane: a chunk
// outside every range, or inside one, needs no other key, and the cells of the
// others are compared only with the ranges that reach into their chunk.
// ALL: every byte is written, in one launch.  Else the mask is cleared and the
// ones are written, so that only selected cells need their index.  Whole calls,
// every key against every range / this: 0.26 M cells 1 range 13.1 / 10.5 us, 128
// ranges 25.3 / 20.1; 3 M cells 16.3 / 13.5 and 97.6 / 21.5; a fifth of 20 M cells
// 80.9 / 25, of 100 M 520 / 84; all of 100 M cells 520 / 390.
// (the ranges travel as a kernel argument: no device buffer is needed)
struct KeyRanges {
    int32_t n;
    uint64_t lohi[2 * kMaxSelectRanges];
};

__global__ __launch_bounds__(256) void k_clear(int64_t n, uint8_t* __restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // the caller's pointer may have any alignment: bytes up to a 16-byte line, lines, bytes
    const int64_t head = min(n, (int64_t)((16 - (reinterpret_cast<uintptr_t>(out) & 15)) & 15));
    const int64_t lines = (n - head) >> 4;
    u32x4* mid = reinterpret_cast<u32x4*>(out + head);
    for (int64_t i = tid; i < lines; i += stride) mid[i] = u32x4{0u, 0u, 0u, 0u};
    for (int64_t i = tid; i < head; i += stride) out[i] = 0;
    for (int64_t i = head + (lines << 4) + tid; i < n; i += stride) out[i] = 0;
}

template <bool ALL, int AHEAD>
__global__ __launch_bounds__(256) void k_select_mask(int64_t n, const uint64_t* __restrict__ keys_sorted,
                                                     const uint32_t* __restrict__ perm, KeyRanges rg,
                                                     uint8_t* __restrict__ mask) {
    __shared__ uint64_t lohi[2 * kMaxSelectRanges];
    static_assert(2 * kMaxSelectRanges <= 256 && kMaxSelectRanges <= 2 * kWave, "a thread per bound, two ranges per lane");
    if ((int)threadIdx.x < 2 * rg.n) lohi[threadIdx.x] = rg.lohi[threadIdx.x];
    __syncthreads();
    constexpr int kChunk = 256 * AHEAD;
    const int lane = lane_id();
    for (int64_t c0 = (int64_t)blockIdx.x * kChunk; c0 < n; c0 += (int64_t)gridDim.x * kChunk) {
        const int64_t c1 = min(c0 + kChunk, n), h0 = c0 + threadIdx.x;
        uint32_t o[AHEAD];
        if (ALL) {
#pragma unroll
            for (int g = 0; g < AHEAD; ++g) o[g] = h0 + 256 * g < c1 ? perm[h0 + 256 * g] : 0xFFFFFFFFu;
        }
        // the ranges that reach into the chunk: two per lane
        const uint64_t k0 = keys_sorted[c0], k1 = keys_sorted[c1 - 1];
        uint64_t some[2];
        bool all = false;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = lane + q * kWave;
            const uint64_t lo = i < rg.n ? lohi[2 * i] : 1ull, hi = i < rg.n ? lohi[2 * i + 1] : 0ull;
            some[q] = __ballot(i < rg.n && lo <= k1 && k0 <= hi);
            all |= __ballot(i < rg.n && lo <= k0 && k1 <= hi) != 0ull;
        }
        if (!ALL && !(some[0] | some[1])) continue;
        bool in[AHEAD];
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) in[g] = all;
        if (!all && (some[0] | some[1])) {
            uint64_t k[AHEAD];
#pragma unroll
            for (int g = 0; g < AHEAD; ++g) k[g] = h0 + 256 * g < c1 ? keys_sorted[h0 + 256 * g] : 0ull;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                for (uint64_t m = some[q]; m; m &= m - 1) {
                    const int i = q * kWave + __builtin_ctzll(m);
                    const uint64_t lo = lohi[2 * i], hi = lohi[2 * i + 1];
#pragma unroll
                    for (int g = 0; g < AHEAD; ++g) in[g] |= k[g] >= lo && k[g] <= hi;
                }
        }
        if (!ALL) {
#pragma unroll
            for (int g = 0; g < AHEAD; ++g) o[g] = in[g] && h0 + 256 * g < c1 ? perm[h0 + 256 * g] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int g = 0; g < AHEAD; ++g)
            if (o[g] < (uint64_t)n) mask[o[g]] = in[g];
    }
}

dvl_status launch_select_mask(int64_t n, const uint64_t* keys_sorted, const uint32_t* perm, int32_t n_ranges,
                              const uint64_t* ranges, uint8_t* mask, hipStream_t st) {
    if (n_ranges < 0 || n_ranges > kMaxSelectRanges) return DVL_E_INVALID;
    KeyRanges rg;
    rg.n = n_ranges;
    for (int i = 0; i < 2 * kMaxSelectRanges; ++i) rg.lohi[i] = i < 2 * n_ranges ? ranges[i] : 0;
    // Every byte written while that costs less than a second launch (3 M cells 13.5
    // us against 19.4, 6 M 21.3 against 19.4); a cell per thread while larger chunks
    // leave compute units idle (1000 cells in 128 ranges 30 -> 20 us).
    auto grid = [&](int64_t ahead) { return dim3((unsigned)std::min<int64_t>((n + 256 * ahead - 1) / (256 * ahead), 1 << 20)); };
    if (n <= 65536) {
        hipLaunchKernelGGL((k_select_mask<true, 1>), grid(1), dim3(256), 0, st, n, keys_sorted, perm, rg, mask);
    } else if (n <= 4000000) {
        hipLaunchKernelGGL((k_select_mask<true, 8>), grid(8), dim3(256), 0, st, n, keys_sorted, perm, rg, mask);
    } else {
        hipLaunchKernelGGL(k_clear, dim3((unsigned)std::min<int64_t>((n / 16 + 255) / 256, 2048)), dim3(256), 0, st, n, mask);
        hipLaunchKernelGGL((k_select_mask<false, 8>), grid(8), dim3(256), 0, st, n, keys_sorted, perm, rg, mask);
    }
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// The cell range of bins b0 .. b1 and its keys, into memory the host can read
// once the stream is synchronised: out[0] = first | last << 32, [1], [2] = keys
// (0 when the range is no range of the volume).
__global__ void k_pick(const uint32_t* first_cell, const uint32_t* last_cell, int b0, int b1, int64_t n,
                       const uint64_t* keys_sorted, uint64_t* out) {
    const uint32_t f = first_cell[b0], l = last_cell[b1];
    const bool ok = f <= l && (int64_t)l < n;
    out[0] = (uint64_t)f | ((uint64_t)l << 32);
    out[1] = ok ? keys_sorted[f] : 0ull;
    out[2] = ok ? keys_sorted[l] : 0ull;
}

dvl_status launch_pick(const uint32_t* first_cell, const uint32_t* last_cell, int b0, int b1, int64_t n,
                       const uint64_t* keys_sorted, uint64_t* out, hipStream_t st) {
    hipLaunchKernelGGL(k_pick, dim3(1), dim3(1), 0, st, first_cell, last_cell, b0, b1, n, keys_sorted, out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// ------------------------------------------------------------------ bins to the host

// The arrays of an update's bins written one after another into pinned host
// memory by one kernel (blockIdx.y: the array).  Eight device-to-host copies
// of a few KB to 31 KB each cost about 15 us apiece (a serving burst of eight
// requests, 960 to 3840 bins of 4 fields: 1.8 ms a burst); one launch whose
// stores cross PCIe takes 5 us (0.96 ms a burst).
__global__ __launch_bounds__(256) void k_pack(PackList l, uint32_t* __restrict__ out) {
    const int a = blockIdx.y;
    const uint32_t* __restrict__ src = l.src[a];
    uint32_t* __restrict__ dst = out + l.at[a];
    const uint32_t n = l.words[a], stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

dvl_status launch_pack(const PackList& l, uint32_t* out, hipStream_t st) {
    uint32_t most = 1;
    for (int a = 0; a < l.n; ++a) most = std::max(most, l.words[a]);
    hipLaunchKernelGGL(k_pack, dim3(std::min<uint32_t>((most + 255) / 256, 64), l.n), dim3(256), 0, st, l, out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// ------------------------------------------------------------------ zoom

// Keys of a range of sorted cells, and the identity permutation (a zoomed
// volume's original order is the range).  Four cells per thread in flight; the
// source starts at any cell, so loads are single keys.  2.4 M cells: 13 us (copy
// and fill apart: 19.5).
__global__ __launch_bounds__(256) void k_range_order(int64_t n, const uint64_t* __restrict__ src,
                                                     uint64_t* __restrict__ keys, uint32_t* __restrict__ perm) {
    constexpr int kAhead = 4;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += kAhead * stride) {
        uint64_t k[kAhead];
#pragma unroll
        for (int g = 0; g < kAhead; ++g)
            if (i + g * stride < n) k[g] = src[i + g * stride];
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            if (i + g * stride >= n) continue;
            keys[i + g * stride] = k[g];
            perm[i + g * stride] = (uint32_t)(i + g * stride);
        }
    }
}

dvl_status launch_range_order(int64_t n, const uint64_t* src, uint64_t* keys, uint32_t* perm, hipStream_t st) {
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 1023) / 1024, 4096));
    hipLaunchKernelGGL(k_range_order, dim3(grid), dim3(256), 0, st, n, src, keys, perm);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

}  // namespace dvl
