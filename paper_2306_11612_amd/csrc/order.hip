// One-time ordering: Hilbert keys at finest-level resolution, LSD radix
// sort of (key, original index), gather of levels and fields into sorted
// order, and per-field data ranges.
//
// Paper: Background (AMR cells snapped to the logical grid: lower corner +
// level, width 2^L), Dynamic Volume Lines (cells represented by quantised
// centroids, ordered along a Hilbert curve), GPU section (the order is
// established once; only the spacing changes afterwards).
#include "order.hpp"
#include "update.hpp"

#include <algorithm>

namespace dvl {

// ===================================================================
// extent: max(corner + 2^level) over all cells and axes, plus range checks.
// Each workgroup writes its own maximum and flags; k_extent_fold takes them
// together.  (Every wave's atomicMax on one word cost about 12 ns each
// whatever the cell count, 32768 waves x 2 atomics: 771 us for 50 M cells;
// 142 + 6 us like this.)
// ===================================================================
constexpr int kReduceThreads = 256;
constexpr int kReduceBlocks = 2048;   // at most; two words of partial result each

struct ExtentPart {
    unsigned long long upper;    // max(corner + 2^level)
    uint32_t bad, level;         // a check failed; max level
};

__device__ __forceinline__ void extent_add(int32_t cx, int32_t cy, int32_t cz, uint32_t L, int64_t& mx,
                                           uint32_t& bad, uint32_t& lmax) {
    bad |= (cx < 0) | (cy < 0) | (cz < 0) | (L > 20u);
    lmax = max(lmax, L);
    const int64_t w = (int64_t)1 << (L & 31u);
    mx = max(mx, max(max((int64_t)cx, (int64_t)cy), (int64_t)cz) + w);
}

// the workgroup's partial result (in thread 0); kWaves: waves of the workgroup
template <int kWaves>
__device__ __forceinline__ ExtentPart extent_block(int64_t mx, uint32_t bad, uint32_t lmax) {
    __shared__ ExtentPart part[kWaves];
    // mx < 2^33: the high word is 0 or 1, reduced first
    const uint32_t hi = wave_highest_u((uint32_t)((uint64_t)mx >> 32));
    const uint32_t lo = wave_highest_u((uint32_t)((uint64_t)mx >> 32) == hi ? (uint32_t)mx : 0u);
    bad = __ballot(bad != 0u) != 0ull;
    lmax = wave_highest_u(lmax);
    if (lane_id() == 0) part[threadIdx.x / kWave] = ExtentPart{((unsigned long long)hi << 32) | lo, bad, lmax};
    __syncthreads();
    ExtentPart r = part[0];
    if (threadIdx.x == 0) {
        for (int k = 1; k < kWaves; ++k) {
            r.upper = max(r.upper, part[k].upper);
            r.bad |= part[k].bad;
            r.level = max(r.level, part[k].level);
        }
    }
    return r;
}

// Four consecutive cells per thread and iteration with vector loads when the
// caller's arrays allow it (V4: x, y, z 16-byte and level 4-byte aligned,
// checked by the launcher); the last n % 4 cells, or all, one by one.
template <bool V4>
__global__ __launch_bounds__(kReduceThreads) void k_extent(int64_t n, const int32_t* __restrict__ x,
                                                           const int32_t* __restrict__ y,
                                                           const int32_t* __restrict__ z,
                                                           const uint8_t* __restrict__ level,
                                                           ExtentPart* __restrict__ part) {
    int64_t mx = 0;
    uint32_t bad = 0, lmax = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nq = V4 ? n >> 2 : 0;
    if constexpr (V4) {
        for (int64_t q = tid; q < nq; q += stride) {
            const int4 cx = reinterpret_cast<const int4*>(x)[q];
            const int4 cy = reinterpret_cast<const int4*>(y)[q];
            const int4 cz = reinterpret_cast<const int4*>(z)[q];
            const uint32_t lw = reinterpret_cast<const uint32_t*>(level)[q];
            extent_add(cx.x, cy.x, cz.x, lw & 0xFFu, mx, bad, lmax);
            extent_add(cx.y, cy.y, cz.y, (lw >> 8) & 0xFFu, mx, bad, lmax);
            extent_add(cx.z, cy.z, cz.z, (lw >> 16) & 0xFFu, mx, bad, lmax);
            extent_add(cx.w, cy.w, cz.w, lw >> 24, mx, bad, lmax);
        }
    }
    for (int64_t i = 4 * nq + tid; i < n; i += stride) extent_add(x[i], y[i], z[i], level[i], mx, bad, lmax);
    const ExtentPart r = extent_block<kReduceThreads / kWave>(mx, bad, lmax);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// out: [0] max upper corner, [1] bad, [2] max level, [3] 0 (the duplicate flag of k_dup)
__global__ __launch_bounds__(1024) void k_extent_fold(int n_part, const ExtentPart* __restrict__ part,
                                                      unsigned long long* __restrict__ out) {
    int64_t mx = 0;
    uint32_t bad = 0, lmax = 0;
    for (int i = threadIdx.x; i < n_part; i += blockDim.x) {
        const ExtentPart p = part[i];
        mx = max(mx, (int64_t)p.upper);
        bad |= p.bad;
        lmax = max(lmax, p.level);
    }
    const ExtentPart r = extent_block<1024 / kWave>(mx, bad, lmax);
    if (threadIdx.x == 0) {
        out[0] = r.upper;
        out[1] = r.bad;
        out[2] = r.level;
        out[3] = 0ull;
    }
}

// ===================================================================
// Hilbert index (Skilling 2004, "Programming the Hilbert curve"): the
// axes are turned into the transposed index by undoing the recursive
// construction's excess work plane by plane from the top, then Gray-coded;
// the bits are interleaved with axis x most significant in every 3-bit
// digit.  The final Gray correction is computed in closed form: its bit j is
// the parity of the bits of the last axis above j.
// ===================================================================
__device__ __forceinline__ uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint64_t hilbert3(uint32_t a, uint32_t b, uint32_t c, int bits) {
    for (int j = bits - 1; j >= 1; --j) {
        const uint32_t Q = 1u << j, P = Q - 1u;
        // axis 0 against itself: invert when set, exchanging with itself is a no-op
        a ^= (a & Q) ? P : 0u;
        if (b & Q) {
            a ^= P;
        } else {
            const uint32_t t = (a ^ b) & P;
            a ^= t;
            b ^= t;
        }
        if (c & Q) {
            a ^= P;
        } else {
            const uint32_t t = (a ^ c) & P;
            a ^= t;
            c ^= t;
        }
    }
    b ^= a;
    c ^= b;
    uint32_t t = c >> 1;          // bit j of t = xor of bits > j of c
    t ^= t >> 1;
    t ^= t >> 2;
    t ^= t >> 4;
    t ^= t >> 8;
    t ^= t >> 16;
    const uint32_t mask = (bits >= 32) ? 0xFFFFFFFFu : ((1u << bits) - 1u);
    t &= mask;
    a ^= t;
    b ^= t;
    c ^= t;
    return (spread3(a) << 2) | (spread3(b) << 1) | spread3(c);
}

__global__ __launch_bounds__(256) void k_keys(int64_t n, const int32_t* __restrict__ x,
                                              const int32_t* __restrict__ y,
                                              const int32_t* __restrict__ z,
                                              const uint8_t* __restrict__ level, int bits,
                                              uint64_t* __restrict__ keys, uint32_t* __restrict__ idx) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t half = (1u << level[i]) >> 1;
        keys[i] = hilbert3((uint32_t)x[i] + half, (uint32_t)y[i] + half, (uint32_t)z[i] + half, bits);
        idx[i] = (uint32_t)i;
    }
}

// The same over four consecutive cells per thread and iteration (x, y, z
// 16-byte aligned and level 4-byte aligned, checked by the launcher): vector
// loads of the coordinates and levels, vector stores of the keys and indices;
// the last n % 4 cells one by one.
__global__ __launch_bounds__(256) void k_keys4(int64_t n, const int32_t* __restrict__ x,
                                               const int32_t* __restrict__ y,
                                               const int32_t* __restrict__ z,
                                               const uint8_t* __restrict__ level, int bits,
                                               uint64_t* __restrict__ keys, uint32_t* __restrict__ idx) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nq = n >> 2;
    for (int64_t q = tid; q < nq; q += stride) {
        const int4 cx = reinterpret_cast<const int4*>(x)[q];
        const int4 cy = reinterpret_cast<const int4*>(y)[q];
        const int4 cz = reinterpret_cast<const int4*>(z)[q];
        const uint32_t lw = reinterpret_cast<const uint32_t*>(level)[q];
        const int32_t xs[4] = {cx.x, cx.y, cx.z, cx.w}, ys[4] = {cy.x, cy.y, cy.z, cy.w},
                      zs[4] = {cz.x, cz.y, cz.z, cz.w};
        uint64_t k4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t half = (1u << ((lw >> (8 * k)) & 0xFFu)) >> 1;
            k4[k] = hilbert3((uint32_t)xs[k] + half, (uint32_t)ys[k] + half, (uint32_t)zs[k] + half, bits);
        }
        u64x2* kd = reinterpret_cast<u64x2*>(keys + 4 * q);
        kd[0] = u64x2{k4[0], k4[1]};
        kd[1] = u64x2{k4[2], k4[3]};
        const uint32_t i0 = (uint32_t)(4 * q);
        reinterpret_cast<u32x4*>(idx)[q] = u32x4{i0, i0 + 1, i0 + 2, i0 + 3};
    }
    for (int64_t i = 4 * nq + tid; i < n; i += stride) {
        const uint32_t half = (1u << level[i]) >> 1;
        keys[i] = hilbert3((uint32_t)x[i] + half, (uint32_t)y[i] + half, (uint32_t)z[i] + half, bits);
        idx[i] = (uint32_t)i;
    }
}

// ===================================================================
// LSD radix sort, 8-bit digits.  Per pass:
//   k_digit_hist   per-tile digit counts, stored digit-major [256][T_pad]
//                  (T_pad: tiles rounded up to a group of 16); one workgroup
//                  counts 16 consecutive tiles and writes each digit's 16
//                  counts as one contiguous 64-byte run
//   scan_u32       exclusive scan of that array (global bucket offsets)
//   k_scatter      stable in-tile ranking (wave match of equal digits),
//                  staging of the tile in digit order in LDS, then writes of
//                  contiguous runs to the global offsets
// ===================================================================
constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;                       // per thread
constexpr int kSortTile = kSortThreads * kSortItems; // 4096 keys
constexpr int kWavesPerSortTile = kSortThreads / kWave;
constexpr int kRadix = 256;
constexpr int kXcds = 8;   // accelerator complex dies of an MI355X, each with its own L2

constexpr int kHistGroup = 16;   // tiles per k_digit_hist workgroup (64 B of counts per digit)

__global__ __launch_bounds__(kSortThreads) void k_digit_hist(int64_t n, const uint64_t* __restrict__ keys,
                                                             int shift, int64_t t_pad,
                                                             uint32_t* __restrict__ counts) {
    __shared__ uint32_t hist[kWavesPerSortTile][kRadix];
    __shared__ uint32_t out[kRadix][kHistGroup];
    const int w = threadIdx.x / kWave;
    const int64_t tile0 = (int64_t)blockIdx.x * kHistGroup;
    for (int g = 0; g < kHistGroup; ++g) {
        for (int i = threadIdx.x; i < kWavesPerSortTile * kRadix; i += kSortThreads)
            (&hist[0][0])[i] = 0;
        __syncthreads();
        const int64_t base = (tile0 + g) * kSortTile;
#pragma unroll 4
        for (int r = 0; r < kSortItems; ++r) {
            const int64_t i = base + (int64_t)r * kSortThreads + threadIdx.x;
            if (i < n) {
                const uint32_t d = (uint32_t)(keys[i] >> shift) & 0xFFu;
                atomicAdd(&hist[w][d], 1u);
            }
        }
        __syncthreads();
        for (int d = threadIdx.x; d < kRadix; d += kSortThreads) {
            uint32_t c = 0;
#pragma unroll
            for (int q = 0; q < kWavesPerSortTile; ++q) c += hist[q][d];
            out[d][g] = c;
        }
        __syncthreads();
    }
    // digit d's counts of the group's 16 tiles: one 64-byte run
    for (int d = threadIdx.x; d < kRadix; d += kSortThreads) {
        uint4* dst = reinterpret_cast<uint4*>(counts + (int64_t)d * t_pad + tile0);
#pragma unroll
        for (int q = 0; q < kHistGroup / 4; ++q)
            dst[q] = make_uint4(out[d][4 * q], out[d][4 * q + 1], out[d][4 * q + 2], out[d][4 * q + 3]);
    }
}

// exclusive scan of uint32 (values and totals fit 32 bits: n_cells < 2^32)
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanBlock = kScanThreads * kScanItems;

__device__ __forceinline__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t* sh /* [kScanThreads/64] */,
                                                        uint32_t* total) {
    // wave inclusive scan (shuffles), then wave totals through LDS
    uint32_t x = v;
    for (int d = 1; d < kWave; d <<= 1) {
        uint32_t t = (uint32_t)shfl_up_i((int)x, d);
        if (lane_id() >= d) x += t;
    }
    const int w = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) sh[w] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int q = 0; q < (int)(blockDim.x / kWave); ++q) {
        if (q < w) off += sh[q];
        tot += sh[q];
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(int64_t n, const uint32_t* __restrict__ in,
                                                              uint32_t* __restrict__ partial) {
    __shared__ uint32_t sh[kScanThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanBlock;
    uint32_t s = 0;
    for (int r = 0; r < kScanItems; ++r) {
        const int64_t i = base + (int64_t)r * kScanThreads + threadIdx.x;
        if (i < n) s += in[i];
    }
    uint32_t tot;
    block_excl_scan_u32(s, sh, &tot);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_partials(int64_t n_part, uint32_t* __restrict__ partial) {
    __shared__ uint32_t sh[1024 / kWave];
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < n_part; b0 += blockDim.x) {
        const int64_t i = b0 + threadIdx.x;
        const uint32_t v = i < n_part ? partial[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan_u32(v, sh, &tot);
        if (i < n_part) partial[i] = carry + ex;
        carry += tot;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_down(int64_t n, const uint32_t* __restrict__ in,
                                                            const uint32_t* __restrict__ partial,
                                                            uint32_t* __restrict__ out) {
    __shared__ uint32_t sh[kScanThreads / kWave];
    // blocked arrangement: thread t owns items [t*kScanItems, (t+1)*kScanItems)
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < kScanItems; ++r) {
        const int64_t i = base + r;
        v[r] = i < n ? in[i] : 0u;
        s += v[r];
    }
    uint32_t tot;
    uint32_t run = partial[blockIdx.x] + block_excl_scan_u32(s, sh, &tot);
#pragma unroll
    for (int r = 0; r < kScanItems; ++r) {
        const int64_t i = base + r;
        if (i < n) out[i] = run;
        run += v[r];
    }
}

static dvl_status scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* partial,
                           hipStream_t s) {
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanThreads), 0, s, n, in, partial);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, s, nb, partial);
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kScanThreads), 0, s, n, in, partial, out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

int64_t scan_partial_count(int64_t n) { return (n + kScanBlock - 1) / kScanBlock; }

__global__ __launch_bounds__(kSortThreads) void k_scatter(int64_t n, const uint64_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin, int shift,
                                                          int64_t t_pad, const uint32_t* __restrict__ offs,
                                                          uint64_t* __restrict__ kout,
                                                          uint32_t* __restrict__ vout) {
    __shared__ uint32_t whist[kWavesPerSortTile][kRadix];   // per-wave digit counts, then bases
    __shared__ uint32_t tbase[kRadix];                      // tile-local start of each digit
    __shared__ uint32_t gbase[kRadix];                      // global start of each digit for this tile
    __shared__ uint32_t wsum[kSortThreads / kWave];
    // the tile in digit order: keys first, then (in the same space) values,
    // so that four workgroups fit a compute unit's LDS
    __shared__ uint64_t stage[kSortTile];
    uint32_t* sval = reinterpret_cast<uint32_t*>(stage);

    const int w = threadIdx.x / kWave;
    const int lane = lane_id();
    // Workgroups go to the 8 XCDs in turn; consecutive tiles on one XCD share
    // the L2 lines of their digit offsets (16 tiles per 64-byte run), so XCD x
    // takes the x-th contiguous eighth of the tiles.
    const int64_t nb = gridDim.x, bid = blockIdx.x;
    const int64_t xcd = bid % kXcds, per = nb / kXcds, rem = nb % kXcds;
    const int64_t tile = xcd * per + min(xcd, rem) + bid / kXcds;
    const int64_t tbeg = tile * kSortTile;
    const int n_here = (int)min((int64_t)kSortTile, n - tbeg);

    for (int i = threadIdx.x; i < kWavesPerSortTile * kRadix; i += kSortThreads) (&whist[0][0])[i] = 0;
    __syncthreads();

    // each wave owns a contiguous quarter of the tile; round r covers 64 keys
    uint64_t key[kSortItems];
    uint32_t val[kSortItems];
    uint32_t rank[kSortItems];
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int li = w * (kWave * kSortItems) + r * kWave + lane;   // tile-local index
        const bool ok = li < n_here;
        key[r] = ok ? kin[tbeg + li] : 0ull;
        val[r] = ok ? vin[tbeg + li] : 0u;
        const uint32_t d = ok ? ((uint32_t)(key[r] >> shift) & 0xFFu) : 0u;
        // lanes holding the same digit
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t b = __ballot((d >> bit) & 1u);
            peers &= ((d >> bit) & 1u) ? b : ~b;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lt);
        const uint32_t old = ok ? whist[w][d] : 0u;
        rank[r] = old + before;
        // the lowest peer bumps the counter by the group size
        if (ok && before == 0) whist[w][d] = old + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // per digit: wave bases inside the tile and the tile's digit start
    if (threadIdx.x < kRadix) {
        const int d = threadIdx.x;
        uint32_t run = 0;
#pragma unroll
        for (int q = 0; q < kWavesPerSortTile; ++q) {
            const uint32_t c = whist[q][d];
            whist[q][d] = run;
            run += c;
        }
        tbase[d] = run;   // tile count of digit d for now
        gbase[d] = offs[(int64_t)d * t_pad + tile];
    }
    __syncthreads();
    // exclusive scan of the 256 tile counts (threads 0..255 hold one each)
    {
        const uint32_t c = threadIdx.x < kRadix ? tbase[threadIdx.x] : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan_u32(c, wsum, &tot);
        __syncthreads();
        if (threadIdx.x < kRadix) tbase[threadIdx.x] = ex;
    }
    __syncthreads();

    // positions in digit order, kept for the value pass
    uint32_t pos[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int li = w * (kWave * kSortItems) + r * kWave + lane;
        pos[r] = 0xFFFFFFFFu;
        if (li < n_here) {
            const uint32_t d = (uint32_t)(key[r] >> shift) & 0xFFu;
            const uint32_t p = tbase[d] + whist[w][d] + rank[r];
            if (p < (uint32_t)kSortTile) {
                pos[r] = p;
                stage[p] = key[r];
            }
        }
    }
    __syncthreads();
    // keys out (contiguous runs per digit); remember each slot's destination
    uint32_t dest[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = r * kSortThreads + threadIdx.x;
        dest[r] = 0xFFFFFFFFu;
        if (i < n_here) {
            const uint64_t k = stage[i];
            const uint32_t d = (uint32_t)(k >> shift) & 0xFFu;
            const int64_t g = (int64_t)gbase[d] + (i - (int64_t)tbase[d]);
            if (g >= 0 && g < n) {
                kout[g] = k;
                dest[r] = (uint32_t)g;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
        if (pos[r] != 0xFFFFFFFFu) sval[pos[r]] = val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = r * kSortThreads + threadIdx.x;
        if (i < n_here && dest[r] != 0xFFFFFFFFu) vout[dest[r]] = sval[i];
    }
}

// flag adjacent equal keys
__global__ __launch_bounds__(256) void k_dup(int64_t n, const uint64_t* __restrict__ k,
                                             unsigned long long* __restrict__ flag) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    uint32_t d = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x + 1; i < n; i += stride)
        d |= (k[i] == k[i - 1]);
    if (__ballot(d) != 0ull && lane_id() == 0) atomicOr(flag, 1ull);
}

dvl_status radix_sort(int64_t n, int key_bits, uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp,
                      uint32_t* vals_tmp, uint32_t* counts, uint32_t* partial, hipStream_t s,
                      uint64_t** keys_out, uint32_t** vals_out) {
    const int64_t n_tiles = (n + kSortTile - 1) / kSortTile;
    const int64_t t_pad = sort_tile_count(n);
    const int passes = std::max(1, (key_bits + 7) / 8);
    uint64_t* ka = keys; uint64_t* kb = keys_tmp;
    uint32_t* va = vals; uint32_t* vb = vals_tmp;
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
        hipLaunchKernelGGL(k_digit_hist, dim3((unsigned)(t_pad / kHistGroup)), dim3(kSortThreads), 0, s, n, ka,
                           shift, t_pad, counts);
        DVL_HIP(hipGetLastError());
        dvl_status st = scan_u32(counts, counts, (int64_t)kRadix * t_pad, partial, s);
        if (st != DVL_OK) return st;
        hipLaunchKernelGGL(k_scatter, dim3((unsigned)n_tiles), dim3(kSortThreads), 0, s, n, ka, va, shift,
                           t_pad, counts, kb, vb);
        DVL_HIP(hipGetLastError());
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    *keys_out = ka;
    *vals_out = va;
    return DVL_OK;
}

int64_t sort_tile_count(int64_t n) {
    const int64_t t = (n + kSortTile - 1) / kSortTile;
    return (t + kHistGroup - 1) / kHistGroup * kHistGroup;
}

// ===================================================================
// data ranges: order-preserving unsigned keys of floats, a NaN above them all
// ===================================================================
constexpr uint32_t kRangeNan = 0xFFFFFFFFu;   // above the key of +inf

__device__ __forceinline__ void range_add(float f, uint32_t& lo, uint32_t& hi) {
    uint32_t u = __float_as_uint(f);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    lo = min(lo, u);
    hi = max(hi, f != f ? kRangeNan : u);
}

// a workgroup's range (in thread 0)
__device__ __forceinline__ uint2 range_block(uint32_t lo, uint32_t hi, uint2* part) {
    lo = wave_lowest_u(lo);
    hi = wave_highest_u(hi);
    if (lane_id() == 0) part[threadIdx.x / kWave] = make_uint2(lo, hi);
    __syncthreads();
    uint2 r = part[0];
    if (threadIdx.x == 0)
        for (int k = 1; k < (int)(blockDim.x / kWave); ++k) {
            r.x = min(r.x, part[k].x);
            r.y = max(r.y, part[k].y);
        }
    return r;
}

// Range of n values in any order: one partial range per workgroup (the
// same-address atomics of every wave took 745 us whatever n, see k_extent;
// 11.8 M fp32 values: 13 + 6 us).
// V4: the values are aligned for vector loads of four, four of them in flight.
template <typename S, bool V4>
__global__ __launch_bounds__(kReduceThreads) void k_range(int64_t n, const typename S::raw* __restrict__ v,
                                                          uint2* __restrict__ part) {
    __shared__ uint2 sh[kReduceThreads / kWave];
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nq = V4 ? n >> 2 : 0;
    if constexpr (V4) {
        int64_t q = tid;
        for (; q + 3 * stride < nq; q += 4 * stride) {
            Quad<S> d[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) d[g].load(v, q + g * stride);
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int k = 0; k < 4; ++k) range_add(d[g].get(k), lo, hi);
        }
        for (; q < nq; q += stride) {
            Quad<S> d;
            d.load(v, q);
#pragma unroll
            for (int k = 0; k < 4; ++k) range_add(d.get(k), lo, hi);
        }
    }
    for (int64_t i = 4 * nq + tid; i < n; i += stride) range_add(to_f32(S{}, v[i]), lo, hi);
    const uint2 r = range_block(lo, hi, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// Workgroup m folds the n_part partial ranges part[m * n_part ..] of field m:
// out[4 m] = min key, [4 m + 1] = max key, [4 m + 2] = NaN seen.
__global__ __launch_bounds__(1024) void k_range_fold(int64_t n_part, const uint2* __restrict__ part,
                                                     unsigned int* __restrict__ out) {
    __shared__ uint2 sh[1024 / kWave];
    const uint2* p = part + (int64_t)blockIdx.x * n_part;
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (int64_t i = threadIdx.x; i < n_part; i += blockDim.x) {
        const uint2 r = p[i];
        lo = min(lo, r.x);
        hi = max(hi, r.y);
    }
    const uint2 r = range_block(lo, hi, sh);
    if (threadIdx.x == 0) {
        out[4 * blockIdx.x] = r.x;
        out[4 * blockIdx.x + 1] = r.y;
        out[4 * blockIdx.x + 2] = r.y == kRangeNan;
    }
}

// ===================================================================
// Sorted arrays of a volume, one pass: gather by the permutation (or a copy
// of a contiguous range, perm NULL), zero padding, data range, per-tile and
// per-step statistics, level codes.
//
// One workgroup per (tile, array): arrays 0 .. M - 1 are the fields, array M
// (when present) the levels.  Its four waves take a quarter of the tile's
// steps each, G steps' loads in flight (4 G scattered loads per lane).
// Bound by the scattered reads.  The cells of a tile are neighbours on the
// Hilbert curve, a compact block whose rows share the cache lines of the
// original order, so a tile is read by one workgroup, and the tiles are dealt
// to the 8 XCDs in contiguous eighths: lines shared by neighbouring tiles are
// fetched into one L2, and a tile's permutation is read from HBM once for all
// its arrays.  Statistics and ranges come from the registers that hold the
// gathered values, instead of a second pass over the sorted arrays.
// 50 M cells, 4 fp32 fields: 536 us (before, in separate passes: 4 gathers of
// 769, 4 statistics passes of 73, levels 69, codes 38 us); 11.8 M cells, one
// field of a data change: 33 us (gather 31 + statistics 30).
// Tile sums: per lane, fp32 sums of 4 values accumulated in fp64 over the
// wave's steps, then the wave, then the four waves in order; step sums: per
// lane the fp64 sum of its 4 values, then the wave.
// ===================================================================
template <typename T>
struct alignas(4 * sizeof(T)) Four {
    T v[4];
};

// the four original indices of the sorted cells c .. c + 3 (n for cells past the end)
__device__ __forceinline__ Four<uint32_t> source_quad(const uint32_t* perm, int64_t c, int64_t n) {
    Four<uint32_t> r;
    if (perm && c + 3 < n) return *reinterpret_cast<const Four<uint32_t>*>(perm + c);
#pragma unroll
    for (int k = 0; k < 4; ++k) r.v[k] = c + k < n ? (perm ? perm[c + k] : (uint32_t)(c + k)) : (uint32_t)n;
    return r;
}

template <typename S, int G>
__device__ __forceinline__ void place_field(int64_t n, int64_t t, int tile_steps, const uint32_t* __restrict__ perm,
                                            const typename S::raw* __restrict__ src, typename S::raw* __restrict__ dst,
                                            int64_t stat, const PlaceStats& st) {
    using raw = typename S::raw;
    constexpr int kWaves = kReduceThreads / kWave;
    __shared__ double wsum[kWaves];
    __shared__ float wmin[kWaves], wmax[kWaves];
    __shared__ uint2 wrange[kWaves];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const int per = tile_steps / kWaves;
    const int64_t step0 = t * tile_steps + (int64_t)w * per;
    double acc = 0.0;
    float lo = INFINITY, hi = -INFINITY;
    uint32_t rlo = 0xFFFFFFFFu, rhi = 0u;
    for (int s = 0; s < per; s += G) {
        Four<uint32_t> p[G];
        Four<raw> r[G];
#pragma unroll
        for (int g = 0; g < G; ++g) p[g] = source_quad(perm, (step0 + s + g) * kStepCells + 4 * lane, n);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int k = 0; k < 4; ++k) r[g].v[k] = p[g].v[k] < (uint64_t)n ? src[p[g].v[k]] : raw(0);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t c = (step0 + s + g) * kStepCells + 4 * lane;
            *reinterpret_cast<Four<raw>*>(dst + c) = r[g];
            float s4 = 0.0f, slo = INFINITY, shi = -INFINITY;
            double d4 = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (c + k < n) {
                    const float v = to_f32(S{}, r[g].v[k]);
                    s4 += v;
                    d4 += (double)v;
                    slo = fminf(slo, v);
                    shi = fmaxf(shi, v);
                    range_add(v, rlo, rhi);
                }
            }
            acc += (double)s4;
            lo = fminf(lo, slo);
            hi = fmaxf(hi, shi);
            d4 = wave_total_d(d4);
            slo = wave_lowest_f(slo);
            shi = wave_highest_f(shi);
            if (lane == 0) {
                const int64_t o = stat * tile_steps * st.n_tiles + step0 + s + g;
                st.step_sum[o] = d4;
                st.step_min[o] = slo;
                st.step_max[o] = shi;
            }
        }
    }
    acc = wave_total_d(acc);
    lo = wave_lowest_f(lo);
    hi = wave_highest_f(hi);
    if (lane == 0) {
        wsum[w] = acc;
        wmin[w] = lo;
        wmax[w] = hi;
    }
    const uint2 range = range_block(rlo, rhi, wrange);   // a barrier: the other waves' sums are there
    if (threadIdx.x == 0) {
        for (int k = 1; k < kWaves; ++k) {
            acc += wsum[k];
            lo = fminf(lo, wmin[k]);
            hi = fmaxf(hi, wmax[k]);
        }
        const int64_t o = stat * st.n_tiles + t;
        st.tile_sum[o] = acc;
        st.tile_min[o] = lo;
        st.tile_max[o] = hi;
        if (st.range) st.range[o] = range;
    }
}

// Levels of one tile, with the 32-bit code of each 256-cell step: byte k
// describes the cells [64 k, 64 k + 64) of the step (lanes 16 k .. 16 k + 15):
// their common level, or 0xFF when they differ.
template <int G>
__device__ __forceinline__ void place_levels(int64_t n, int64_t t, int tile_steps, const uint32_t* __restrict__ perm,
                                             const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
                                             uint32_t* __restrict__ codes) {
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const int per = tile_steps / (kReduceThreads / kWave);
    const int64_t step0 = t * tile_steps + (int64_t)w * per;
    for (int s = 0; s < per; s += G) {
        Four<uint32_t> p[G];
        Four<uint8_t> r[G];
#pragma unroll
        for (int g = 0; g < G; ++g) p[g] = source_quad(perm, (step0 + s + g) * kStepCells + 4 * lane, n);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int k = 0; k < 4; ++k) r[g].v[k] = p[g].v[k] < (uint64_t)n ? src[p[g].v[k]] : (uint8_t)0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            *reinterpret_cast<Four<uint8_t>*>(dst + (step0 + s + g) * kStepCells + 4 * lane) = r[g];
            const uint32_t word = __builtin_bit_cast(uint32_t, r[g]);
            const uint32_t b0 = word & 0xFFu;
            uint32_t code = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t first = readlane(b0, 16 * k);
                const uint64_t same = __ballot(word == first * 0x01010101u) >> (16 * k);
                code |= ((same & 0xFFFFull) == 0xFFFFull ? first : 0xFFu) << (8 * k);
            }
            if (lane == 0) codes[step0 + s + g] = code;
        }
    }
}

template <typename S, int G>
__global__ __launch_bounds__(kReduceThreads) void k_place(int64_t n, int tile_steps, const uint32_t* __restrict__ perm,
                                                          PlaceArrays a, PlaceStats st) {
    const int n_arrays = a.n_fields + (a.level_src ? 1 : 0);
    const int64_t units = st.n_tiles * n_arrays, bid = blockIdx.x;
    // one round unless there are more units than a launch may have workgroups
    for (int64_t u0 = 0; u0 + bid < units; u0 += gridDim.x) {
        const int64_t nb = min((int64_t)gridDim.x, units - u0);
        const int64_t xcd = bid % kXcds, per = nb / kXcds, rem = nb % kXcds;
        const int64_t u = u0 + xcd * per + min(xcd, rem) + bid / kXcds;
        const int64_t t = u / n_arrays;
        const int m = (int)(u - t * n_arrays);
        if (m < a.n_fields)
            place_field<S, G>(n, t, tile_steps, perm, reinterpret_cast<const typename S::raw*>(a.src[m]),
                              reinterpret_cast<typename S::raw*>(a.dst[m]), a.first_field + m, st);
        else
            place_levels<G>(n, t, tile_steps, perm, a.level_src, a.level_dst, a.codes);
        __syncthreads();
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_scatter_back(int64_t n, const uint32_t* __restrict__ perm,
                                                      const T* __restrict__ sorted, T* __restrict__ orig) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t p = perm[i];
        if (p < (uint64_t)n) orig[p] = sorted[i];
    }
}

static unsigned grid_for(int64_t n, int per_block = 256, int max_blocks = 8192) {
    int64_t g = (n + per_block - 1) / per_block;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, max_blocks));
}

// the caller's coordinate and level arrays allow the 4-cell loads
static bool vec4_inputs(const int32_t* x, const int32_t* y, const int32_t* z, const uint8_t* level) {
    return ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(z)) & 15u) == 0 &&
           (reinterpret_cast<uintptr_t>(level) & 3u) == 0;
}

size_t extent_scratch_bytes() { return (size_t)kReduceBlocks * sizeof(ExtentPart); }

dvl_status launch_extent(int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                         const uint8_t* level, unsigned long long* out, void* scratch, hipStream_t s) {
    ExtentPart* part = reinterpret_cast<ExtentPart*>(scratch);
    const unsigned grid = grid_for((n + 3) / 4, kReduceThreads, kReduceBlocks);
    if (vec4_inputs(x, y, z, level))
        hipLaunchKernelGGL(k_extent<true>, dim3(grid), dim3(kReduceThreads), 0, s, n, x, y, z, level, part);
    else
        hipLaunchKernelGGL(k_extent<false>, dim3(grid), dim3(kReduceThreads), 0, s, n, x, y, z, level, part);
    hipLaunchKernelGGL(k_extent_fold, dim3(1), dim3(1024), 0, s, (int)grid, part, out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

dvl_status launch_keys(int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                       const uint8_t* level, int bits, uint64_t* keys, uint32_t* idx, hipStream_t s) {
    if (vec4_inputs(x, y, z, level))
        hipLaunchKernelGGL(k_keys4, dim3(grid_for((n + 3) / 4)), dim3(256), 0, s, n, x, y, z, level, bits, keys, idx);
    else
        hipLaunchKernelGGL(k_keys, dim3(grid_for(n)), dim3(256), 0, s, n, x, y, z, level, bits, keys, idx);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

dvl_status launch_dup(int64_t n, const uint64_t* keys, unsigned long long* flag, hipStream_t s) {
    hipLaunchKernelGGL(k_dup, dim3(grid_for(n)), dim3(256), 0, s, n, keys, flag);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

dvl_status launch_scatter_back(int64_t n, const uint32_t* perm, const void* sorted, void* orig,
                               int elem_bytes, hipStream_t s) {
    if (elem_bytes == 8)
        hipLaunchKernelGGL(k_scatter_back<uint64_t>, dim3(grid_for(n)), dim3(256), 0, s, n, perm,
                           (const uint64_t*)sorted, (uint64_t*)orig);
    else
        return DVL_E_INVALID;
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

size_t range_scratch_bytes() { return (size_t)kReduceBlocks * sizeof(uint2); }

template <typename S>
static void range_of(int64_t n, const void* v, uint2* part, unsigned grid, hipStream_t s) {
    const auto* p = reinterpret_cast<const typename S::raw*>(v);
    if ((reinterpret_cast<uintptr_t>(v) & (Quad<S>::kBytes - 1)) == 0)
        hipLaunchKernelGGL((k_range<S, true>), dim3(grid), dim3(kReduceThreads), 0, s, n, p, part);
    else
        hipLaunchKernelGGL((k_range<S, false>), dim3(grid), dim3(kReduceThreads), 0, s, n, p, part);
}

dvl_status launch_range(int64_t n, int dtype, const void* v, unsigned int* out, void* scratch, hipStream_t s) {
    uint2* part = reinterpret_cast<uint2*>(scratch);
    const unsigned grid = grid_for((n + 3) / 4, kReduceThreads, kReduceBlocks);
    if (dtype == DVL_F32)
        range_of<F32>(n, v, part, grid, s);
    else if (dtype == DVL_F16)
        range_of<F16>(n, v, part, grid, s);
    else
        range_of<BF16>(n, v, part, grid, s);
    hipLaunchKernelGGL(k_range_fold, dim3(1), dim3(1024), 0, s, (int64_t)grid, part, out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

template <typename S>
static void place_typed(int64_t n, int tile_steps, const uint32_t* perm, const PlaceArrays& a, const PlaceStats& st,
                        unsigned grid, hipStream_t s) {
    // tiles of 8 steps: two steps per wave; 16 and 32: four at a time
    if (tile_steps < 16)
        hipLaunchKernelGGL((k_place<S, 2>), dim3(grid), dim3(kReduceThreads), 0, s, n, tile_steps, perm, a, st);
    else
        hipLaunchKernelGGL((k_place<S, 4>), dim3(grid), dim3(kReduceThreads), 0, s, n, tile_steps, perm, a, st);
}

dvl_status launch_place(int64_t n, int dtype, int tile_steps, const uint32_t* perm, const PlaceArrays& a,
                        const PlaceStats& st, unsigned int* ranges, hipStream_t s) {
    const int64_t units = st.n_tiles * (a.n_fields + (a.level_src ? 1 : 0));
    const unsigned grid = (unsigned)std::min<int64_t>(units, (int64_t)1 << 23);   // below 2^32 work-items
    if (dtype == DVL_F32)
        place_typed<F32>(n, tile_steps, perm, a, st, grid, s);
    else if (dtype == DVL_F16)
        place_typed<F16>(n, tile_steps, perm, a, st, grid, s);
    else
        place_typed<BF16>(n, tile_steps, perm, a, st, grid, s);
    DVL_HIP(hipGetLastError());
    if (ranges) {
        hipLaunchKernelGGL(k_range_fold, dim3(a.n_fields), dim3(1024), 0, s, st.n_tiles, st.range, ranges);
        DVL_HIP(hipGetLastError());
    }
    return DVL_OK;
}

}  // namespace dvl
