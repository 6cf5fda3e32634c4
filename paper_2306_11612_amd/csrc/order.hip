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
// 98 + 4 us like this.)
// ===================================================================
constexpr int kReduceThreads = 256;
constexpr int kReduceBlocks = kRangeParts;   // at most

// Above this many cells the passes read their arrays as non-temporal streams and
// write the sorted fields so: the 8-byte words of the sort alone exceed the 256
// MB Infinity Cache, nothing is left of them for the next pass, and they stream
// faster past the caches (50 M cells: extent 136 -> 98 us, a count 103 -> 78, a
// scatter 187 -> 182, the sorted arrays 519 -> 512; the keys' pass, which writes
// after the scattered writes of whatever ran before, gained nothing).  Volumes
// that fit read what the pass before left there (1.1 M cells, the keys' pass
// 12.2 us against 14.4).
constexpr int64_t kStreamCells = (int64_t)1 << 25;
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM, typename T>
__device__ __forceinline__ T read(const T* p) {
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}

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
template <bool V4, bool STREAM>
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
            const i32x4 cx = read<STREAM>(reinterpret_cast<const i32x4*>(x) + q);
            const i32x4 cy = read<STREAM>(reinterpret_cast<const i32x4*>(y) + q);
            const i32x4 cz = read<STREAM>(reinterpret_cast<const i32x4*>(z) + q);
            const uint32_t lw = read<STREAM>(reinterpret_cast<const uint32_t*>(level) + q);
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

// out (pinned host memory): [0] max upper corner, [1] bad, [2] max level; dup:
// the duplicate flag of k_dup, cleared
__global__ __launch_bounds__(1024) void k_extent_fold(int n_part, const ExtentPart* __restrict__ part,
                                                      unsigned long long* __restrict__ out,
                                                      unsigned long long* __restrict__ dup) {
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
        *dup = 0ull;
    }
}

// ===================================================================
// Hilbert index.  The curve is Skilling's ("Programming the Hilbert curve",
// 2004): per plane of bits from the top, axis i's bit set inverts the lower
// bits of axis 0, clear exchanges the lower bits of axes 0 and i; then the
// Gray code, and axis x most significant in every 3-bit digit.  What the
// planes above did to the bits of a plane is an exchange and inversion of the
// axes, and the Gray code's correction is one parity bit: 48 states are
// reached, and a plane's digit and next state follow from the state and the
// plane's three bits.  The state table is derived here from those rules, two
// planes per step (64 input patterns); an odd number of planes starts in the
// state that an empty plane turns into the initial one.
//
// About 10 vector instructions and one LDS lookup per two planes instead of
// some 36: the plane-by-plane form took 272 us for the keys of 50 M cells (11
// planes) alone, bound by its arithmetic; with the first pass's counts it
// took 376 us, this 242 (keys read and written at 4.4 TB/s).
// ===================================================================
constexpr int kHilbertStates = 48;
struct HilbertTable {
    uint16_t next[kHilbertStates * 64];   // state << 6 | (x pair << 4 | y pair << 2 | z pair) -> next state << 6 | 6 key bits
    uint16_t start_odd;                   // state before an empty plane that leads to state 0
};

struct HilbertState {
    int perm[3], flip[3], t;   // axis i's lower bits: original axis perm[i], inverted if flip[i]; Gray parity
    constexpr bool operator==(const HilbertState& o) const {
        for (int i = 0; i < 3; ++i)
            if (perm[i] != o.perm[i] || flip[i] != o.flip[i]) return false;
        return t == o.t;
    }
};

// one plane: bits o of the original axes -> the 3-bit digit; the state moves on
constexpr int hilbert_plane(HilbertState& s, const int (&o)[3]) {
    int a[3] = {};
    for (int i = 0; i < 3; ++i) a[i] = o[s.perm[i]] ^ s.flip[i];
    for (int i = 0; i < 3; ++i) {
        if (a[i]) {
            s.flip[0] ^= 1;
        } else {
            const int p = s.perm[0], f = s.flip[0];
            s.perm[0] = s.perm[i];
            s.flip[0] = s.flip[i];
            s.perm[i] = p;
            s.flip[i] = f;
        }
    }
    const int b = a[0] ^ a[1], c = b ^ a[2];
    const int d = ((a[0] ^ s.t) << 2) | ((b ^ s.t) << 1) | (c ^ s.t);
    s.t ^= c;
    return d;
}

constexpr HilbertTable make_hilbert_table() {
    HilbertTable T{};
    HilbertState st[kHilbertStates] = {};
    st[0] = HilbertState{{0, 1, 2}, {0, 0, 0}, 0};
    int n = 1;
    auto index = [&](const HilbertState& s) {
        for (int k = 0; k < n; ++k)
            if (st[k] == s) return k;
        st[n] = s;
        return n++;
    };
    // single planes first, so that every state is reached and numbered
    for (int k = 0; k < n; ++k)
        for (int v = 0; v < 8; ++v) {
            HilbertState s = st[k];
            const int o[3] = {v >> 2, (v >> 1) & 1, v & 1};
            const int d = hilbert_plane(s, o);
            if (index(s) == 0 && v == 0 && d == 0) T.start_odd = (uint16_t)k;
        }
    for (int k = 0; k < n; ++k)
        for (int v = 0; v < 64; ++v) {
            HilbertState s = st[k];
            const int x = v >> 4, y = (v >> 2) & 3, z = v & 3;
            const int o1[3] = {x >> 1, y >> 1, z >> 1}, o0[3] = {x & 1, y & 1, z & 1};
            const int d1 = hilbert_plane(s, o1), d0 = hilbert_plane(s, o0);
            T.next[k * 64 + v] = (uint16_t)(index(s) << 6 | d1 << 3 | d0);
        }
    return T;
}
static __constant__ const HilbertTable kHilbert = make_hilbert_table();

// keys of N cells at once (N independent lookup chains); `table`: the state
// table in LDS
template <int N>
__device__ __forceinline__ void hilbert_keys(const uint16_t* table, uint32_t start_odd, int bits, const uint32_t (&x)[N],
                                             const uint32_t (&y)[N], const uint32_t (&z)[N], uint64_t (&key)[N]) {
    uint32_t e[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        key[k] = 0ull;
        e[k] = (bits & 1) ? start_odd << 6 : 0u;
    }
    for (int j = ((bits + 1) & ~1) - 2; j >= 0; j -= 2) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const uint32_t v = (((x[k] >> j) & 3u) << 4) | (((y[k] >> j) & 3u) << 2) | ((z[k] >> j) & 3u);
            e[k] = table[(e[k] & ~63u) | v];
            key[k] = (key[k] << 6) | (e[k] & 63u);
        }
    }
}

// ===================================================================
// Stable LSD radix sort of (key, original index) in digits of D bits.
//
// Words.  When the key's bits and the bits of an index fit 64 together, a
// word holds both (key << idx_bits | index): 8 bytes per cell and pass instead
// of 12, and one LDS exchange per tile; the last pass splits it.  Longer keys
// of large volumes (36 bits and 501 M cells need 65) keep key and index apart.
//
// Per pass:
//   k_count    a workgroup counts the digits of a chunk of consecutive tiles:
//              for every tile the counts of the chunk's earlier tiles (a row
//              of kRadix words), and the chunk's totals.  The first pass's
//              counts are taken while the keys are made (k_words).
//   k_columns  exclusive scan of the chunk totals down every digit's column,
//              and the digit totals
//   k_scatter  stable in-tile ranking (wave match of equal digits), the tile
//              exchanged into digit order through LDS, then runs of equal
//              digits written to digit base + column scan + chunk row
// Rows are tile-major, so counting writes and scattering reads whole rows.
//
// 50 M cells, 33-bit keys, MI355X: 4 passes of 78 (count) + 8 (columns) + 182 us
// (scatter: 16 bytes per cell at 4.4 TB/s) after 242 us for the keys, the first
// of them without its count: 1.24 ms.  With 12-byte pairs, 8-bit
// digits, counts in digit-major order and a scan over all of them it was 5
// passes of 167 + 33 + 405 us after 285: 3.31 ms.
// ===================================================================
constexpr int kSortThreads = 256;
// Keys per thread: 16, tiles of 4096; 4, tiles of 1024, while the larger ones
// would give a compute unit one workgroup, whose 16 rounds of ranking follow
// one another (a scatter of 1.1 M cells 15 -> 10.6 us; building 0.2 M cells 154 ->
// 127 us, 1.0 M 172 -> 156, 2.0 M and more the same or slower).
constexpr int kSortItems = 16, kSortItemsSmall = 4;
constexpr int64_t kSmallCells = (int64_t)3 << 19;
constexpr int sort_tile(int items) { return kSortThreads * items; }
constexpr int kSortWaves = kSortThreads / kWave;

// Tiles per counting workgroup: up to 16, fewer while that leaves compute
// units idle (1.1 M cells in groups of 16 were 17 workgroups, 79 us a pass).
static int sort_chunk(int64_t n_tiles) { return (int)std::max<int64_t>(1, std::min<int64_t>(16, n_tiles / 1024)); }

template <int D>
__device__ __forceinline__ uint32_t digit_of(uint64_t w, int shift) {
    return (uint32_t)(w >> shift) & ((1u << D) - 1u);
}

// LDS of a counting workgroup: digit counts of the current tile, per wave and
// in kCountCopies copies beside each other (in other banks) that the lanes
// take in turn: cells of coarse levels share their low key digits, and equal
// digits of one wave are added one after another.
constexpr int kCountCopies = 4;
template <int D>
struct CountLds {
    uint32_t hist[kSortWaves][1 << D][kCountCopies];
    __device__ __forceinline__ void add(uint32_t d) {
        atomicAdd(&hist[threadIdx.x / kWave][d][threadIdx.x & (kCountCopies - 1)], 1u);
    }
};

// counts of the tile (cleared before the first one) -> its row and the running
// totals of the chunk, kept in registers (thread t: digits t, t + 256, ...)
template <int D>
__device__ __forceinline__ void count_row(CountLds<D>& l, uint32_t (&run)[(1 << D) / kSortThreads], uint32_t* row) {
    constexpr int R = 1 << D;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R / kSortThreads; ++k) {
        const int d = k * kSortThreads + threadIdx.x;
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) {
            u32x4* h = reinterpret_cast<u32x4*>(l.hist[q][d]);
            const u32x4 v = *h;
            c += (v.x + v.y) + (v.z + v.w);
            *h = u32x4{0u, 0u, 0u, 0u};
        }
        row[d] = run[k];
        run[k] += c;
    }
    __syncthreads();
}

template <int D>
__device__ __forceinline__ void count_clear(CountLds<D>& l, uint32_t (&run)[(1 << D) / kSortThreads]) {
    static_assert(kCountCopies == 4, "read and cleared as one 16-byte word");
    for (int i = threadIdx.x; i < kSortWaves << D; i += kSortThreads)
        reinterpret_cast<u32x4*>(&l.hist[0][0][0])[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < (1 << D) / kSortThreads; ++k) run[k] = 0u;
    __syncthreads();
}

template <int D>
__device__ __forceinline__ void count_totals(const uint32_t (&run)[(1 << D) / kSortThreads], uint32_t* totals) {
#pragma unroll
    for (int k = 0; k < (1 << D) / kSortThreads; ++k) totals[k * kSortThreads + threadIdx.x] = run[k];
}

// Keys (and, packed, the index below them) of a chunk of tiles, with the
// digit counts of the first pass.  Four consecutive cells per thread with
// vector loads and stores when the caller's arrays allow it (V4: x, y, z
// 16-byte and level 4-byte aligned, checked by the launcher).
template <int D, int ITEMS, bool PACKED, bool V4>
__global__ __launch_bounds__(kSortThreads) void k_words(int64_t n, const int32_t* __restrict__ x,
                                                        const int32_t* __restrict__ y, const int32_t* __restrict__ z,
                                                        const uint8_t* __restrict__ level, int bits, int idx_bits,
                                                        int chunk, int64_t n_tiles, uint64_t* __restrict__ words,
                                                        uint32_t* __restrict__ idx, uint32_t* __restrict__ rows,
                                                        uint32_t* __restrict__ totals) {
    constexpr int kTile = sort_tile(ITEMS);
    __shared__ alignas(16) CountLds<D> l;
    __shared__ alignas(16) uint16_t table[kHilbertStates * 64];
    static_assert(sizeof(table) % 4 == 0, "copied in 32-bit words");
    for (int i = threadIdx.x; i < (int)sizeof(table) / 4; i += kSortThreads)
        reinterpret_cast<uint32_t*>(table)[i] = reinterpret_cast<const uint32_t*>(kHilbert.next)[i];
    const uint32_t start_odd = kHilbert.start_odd;
    uint32_t run[(1 << D) / kSortThreads];
    count_clear(l, run);
    const int64_t t0 = (int64_t)blockIdx.x * chunk, t1 = min(t0 + chunk, n_tiles);
    auto word = [&](int64_t i, uint64_t k) -> uint64_t {
        l.add(digit_of<D>(k, 0));
        return PACKED ? (k << idx_bits) | (uint64_t)i : k;
    };
    auto half = [](uint32_t lev) { return (1u << lev) >> 1; };
    for (int64_t t = t0; t < t1; ++t) {
#pragma unroll
        for (int r = 0; r < ITEMS / 4; ++r) {
            const int64_t i = t * kTile + 4 * ((int64_t)r * kSortThreads + threadIdx.x);
            if (V4 && i + 3 < n) {
                const i32x4 cx = *reinterpret_cast<const i32x4*>(x + i);
                const i32x4 cy = *reinterpret_cast<const i32x4*>(y + i);
                const i32x4 cz = *reinterpret_cast<const i32x4*>(z + i);
                const uint32_t lw = *reinterpret_cast<const uint32_t*>(level + i);
                const uint32_t h[4] = {half(lw & 0xFFu), half((lw >> 8) & 0xFFu), half((lw >> 16) & 0xFFu), half(lw >> 24)};
                const uint32_t xs[4] = {cx.x + h[0], cx.y + h[1], cx.z + h[2], cx.w + h[3]};
                const uint32_t ys[4] = {cy.x + h[0], cy.y + h[1], cy.z + h[2], cy.w + h[3]};
                const uint32_t zs[4] = {cz.x + h[0], cz.y + h[1], cz.z + h[2], cz.w + h[3]};
                uint64_t k[4];
                hilbert_keys<4>(table, start_odd, bits, xs, ys, zs, k);
                u64x2* kd = reinterpret_cast<u64x2*>(words + i);
                kd[0] = u64x2{word(i, k[0]), word(i + 1, k[1])};
                kd[1] = u64x2{word(i + 2, k[2]), word(i + 3, k[3])};
                if (!PACKED) {
                    const uint32_t i0 = (uint32_t)i;
                    *reinterpret_cast<u32x4*>(idx + i) = u32x4{i0, i0 + 1, i0 + 2, i0 + 3};
                }
            } else {
                for (int64_t c = i; c < min(i + 4, n); ++c) {
                    const uint32_t h = half(level[c]);
                    const uint32_t xs[1] = {x[c] + h}, ys[1] = {y[c] + h}, zs[1] = {z[c] + h};
                    uint64_t k[1];
                    hilbert_keys<1>(table, start_odd, bits, xs, ys, zs, k);
                    words[c] = word(c, k[0]);
                    if (!PACKED) idx[c] = (uint32_t)c;
                }
            }
        }
        count_row(l, run, rows + (t << D));
    }
    count_totals<D>(run, totals + ((int64_t)blockIdx.x << D));
}

template <int D, int ITEMS, bool STREAM>
__global__ __launch_bounds__(kSortThreads) void k_count(int64_t n, const uint64_t* __restrict__ words, int shift,
                                                        int chunk, int64_t n_tiles, uint32_t* __restrict__ rows,
                                                        uint32_t* __restrict__ totals) {
    constexpr int kTile = sort_tile(ITEMS);
    __shared__ alignas(16) CountLds<D> l;
    uint32_t run[(1 << D) / kSortThreads];
    count_clear(l, run);
    const int64_t t0 = (int64_t)blockIdx.x * chunk, t1 = min(t0 + chunk, n_tiles);
    for (int64_t t = t0; t < t1; ++t) {
        const int64_t base = t * kTile;
        if (base + kTile <= n) {
            u64x2 v[ITEMS / 2];
#pragma unroll
            for (int r = 0; r < ITEMS / 2; ++r)
                v[r] = read<STREAM>(reinterpret_cast<const u64x2*>(words + base) + r * kSortThreads + threadIdx.x);
#pragma unroll
            for (int r = 0; r < ITEMS / 2; ++r) {
                l.add(digit_of<D>(v[r].x, shift));
                l.add(digit_of<D>(v[r].y, shift));
            }
        } else {
            for (int64_t i = base + threadIdx.x; i < n; i += kSortThreads)
                l.add(digit_of<D>(words[i], shift));
        }
        count_row(l, run, rows + (t << D));
    }
    count_totals<D>(run, totals + ((int64_t)blockIdx.x << D));
}

// exclusive scan within a workgroup (values and totals fit 32 bits: n_cells < 2^32)
__device__ __forceinline__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t* sh /* [threads / 64] */, uint32_t* total) {
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

// Column scan of the chunk totals [n_chunks][1 << D], in place, and the digit
// totals.  A workgroup takes 16 digits (64-byte pieces of the rows); its 64
// groups of 16 lanes take a 64th of the rows each: sums first, then the
// exclusive prefixes.  Bound by the latency of its loads, so many groups with
// 8 loads in flight each: 1110 rows of 512 digits 7.6 us (14.8 with 64 digits
// per workgroup and 16 groups).
constexpr int kColumnDigits = 16, kColumnGroups = 64;
template <int D>
__global__ __launch_bounds__(kColumnDigits * kColumnGroups) void k_columns(int64_t n_chunks,
                                                                           uint32_t* __restrict__ totals,
                                                                           uint32_t* __restrict__ digits) {
    __shared__ uint32_t part[kColumnGroups][kColumnDigits];
    const int g = threadIdx.x / kColumnDigits, j = threadIdx.x % kColumnDigits;
    const int d = blockIdx.x * kColumnDigits + j;
    const int64_t per = (n_chunks + kColumnGroups - 1) / kColumnGroups;
    const int64_t r0 = min(g * per, n_chunks), r1 = min(r0 + per, n_chunks);
    uint32_t sum = 0;
#pragma unroll 8
    for (int64_t r = r0; r < r1; ++r) sum += totals[(r << D) + d];
    part[g][j] = sum;
    __syncthreads();
    uint32_t run = 0, all = 0;
#pragma unroll 16
    for (int q = 0; q < kColumnGroups; ++q) {
        if (q < g) run += part[q][j];
        all += part[q][j];
    }
    if (g == 0) digits[d] = all;
    int64_t r = r0;
    for (; r + 8 <= r1; r += 8) {
        uint32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = totals[((r + k) << D) + d];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            totals[((r + k) << D) + d] = run;
            run += v[k];
        }
    }
    for (; r < r1; ++r) {
        const uint32_t v = totals[(r << D) + d];
        totals[(r << D) + d] = run;
        run += v;
    }
}

// PACKED: words hold key and index (LAST: split them into kout and vout);
// otherwise the indices travel as vin -> vout.
template <int D, int ITEMS, bool PACKED, bool LAST, bool STREAM>
__global__ __launch_bounds__(kSortThreads) void k_scatter(int64_t n, const uint64_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin, int shift, int idx_bits,
                                                          int chunk, const uint32_t* __restrict__ rows,
                                                          const uint32_t* __restrict__ columns,
                                                          const uint32_t* __restrict__ digits,
                                                          uint64_t* __restrict__ kout, uint32_t* __restrict__ vout) {
    constexpr int kTile = sort_tile(ITEMS);
    constexpr int R = 1 << D;
    constexpr int per_thread = R / kSortThreads;
    __shared__ alignas(16) uint16_t whist[kSortWaves][R];   // per-wave digit counts, then starts in the tile (<= 4096)
    __shared__ uint32_t gbase[R];               // global position of the digit's first cell here minus its start in the tile
    __shared__ uint32_t wsum[2][kSortWaves];
    // the tile in digit order: keys first, then (in the same space) values
    __shared__ uint64_t stage[kTile];
    uint32_t* sval = reinterpret_cast<uint32_t*>(stage);

    const int w = threadIdx.x / kWave;
    const int lane = lane_id();
    // Workgroups go to the 8 XCDs in turn; consecutive tiles write neighbouring
    // runs (parts of the same cache lines), so XCD x takes the x-th contiguous
    // eighth of the tiles.
    const int64_t nb = gridDim.x, bid = blockIdx.x;
    const int64_t xcd = bid % kXcds, per = nb / kXcds, rem = nb % kXcds;
    const int64_t tile = xcd * per + min(xcd, rem) + bid / kXcds;
    const int64_t tbeg = tile * kTile;
    const int n_here = (int)min((int64_t)kTile, n - tbeg);

    // each wave owns a contiguous quarter of the tile; round r covers 64 keys
    uint64_t key[ITEMS];
    uint32_t val[PACKED ? 1 : ITEMS];
    uint32_t rank[ITEMS];
    const int li0 = w * (kWave * ITEMS) + lane;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int li = li0 + r * kWave;
        key[r] = li < n_here ? read<STREAM>(kin + tbeg + li) : 0ull;
        if constexpr (!PACKED) val[r] = li < n_here ? read<STREAM>(vin + tbeg + li) : 0u;
    }
    // this tile's digit positions, consecutive digits per thread
    uint32_t row[per_thread], col[per_thread], tot[per_thread];
#pragma unroll
    for (int k = 0; k < per_thread; ++k) {
        const int d = threadIdx.x * per_thread + k;
        row[k] = rows[(tile << D) + d];
        col[k] = columns[((tile / chunk) << D) + d];
        tot[k] = digits[d];
    }
    {
        uint32_t* z = reinterpret_cast<uint32_t*>(&whist[0][0]);
        for (int i = threadIdx.x; i < kSortWaves * R / 2; i += kSortThreads) z[i] = 0;
    }
    __syncthreads();

    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool ok = li0 + r * kWave < n_here;
        const uint32_t d = digit_of<D>(key[r], shift);
        // lanes holding the same digit
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < D; ++bit) {
            const uint64_t b = __ballot((d >> bit) & 1u);
            peers &= ((d >> bit) & 1u) ? b : ~b;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lt);
        const uint32_t old = ok ? whist[w][d] : 0u;
        rank[r] = old + before;
        // the lowest peer bumps the counter by the group size
        if (ok && before == 0) whist[w][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // per digit: the waves' starts inside the tile, the tile's digit start and
    // the global digit base (both exclusive scans over the digits)
    {
        uint32_t cnt[per_thread], csum = 0, tsum = 0;
#pragma unroll
        for (int k = 0; k < per_thread; ++k) {
            const int d = threadIdx.x * per_thread + k;
            cnt[k] = 0;
#pragma unroll
            for (int q = 0; q < kSortWaves; ++q) cnt[k] += whist[q][d];
            csum += cnt[k];
            tsum += tot[k];
        }
        uint32_t all;
        uint32_t here = block_excl_scan_u32(csum, wsum[0], &all);
        uint32_t base = block_excl_scan_u32(tsum, wsum[1], &all);
#pragma unroll
        for (int k = 0; k < per_thread; ++k) {
            const int d = threadIdx.x * per_thread + k;
            gbase[d] = base + col[k] + row[k] - here;
            uint32_t run = here;
#pragma unroll
            for (int q = 0; q < kSortWaves; ++q) {
                const uint32_t c = whist[q][d];
                whist[q][d] = (uint16_t)run;
                run += c;
            }
            here += cnt[k];
            base += tot[k];
        }
    }
    __syncthreads();

    // positions in digit order (kept for the value pass)
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (li0 + r * kWave < n_here) {
            rank[r] += whist[w][digit_of<D>(key[r], shift)];
            stage[rank[r] & (kTile - 1)] = key[r];
        }
    }
    __syncthreads();
    // out in contiguous runs per digit; remember each slot's destination
    uint32_t dest[PACKED ? 1 : ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = r * kSortThreads + threadIdx.x;
        if (i < n_here) {
            const uint64_t k = stage[i];
            const uint32_t g = gbase[digit_of<D>(k, shift)] + (uint32_t)i;
            if constexpr (!PACKED) dest[r] = g;
            if ((int64_t)g < n) {
                if constexpr (PACKED && LAST) {
                    kout[g] = k >> idx_bits;
                    vout[g] = (uint32_t)(k & ((1ull << idx_bits) - 1ull));
                } else {
                    kout[g] = k;
                }
            }
        }
    }
    if constexpr (!PACKED) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (li0 + r * kWave < n_here) sval[rank[r] & (kTile - 1)] = val[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const int i = r * kSortThreads + threadIdx.x;
            if (i < n_here && (int64_t)dest[r] < n) vout[dest[r]] = sval[i];
        }
    }
}

// Flag adjacent equal keys: two keys a thread, the one before them from the
// lane before, four such pairs in flight.  50 M keys: 74 us (one key and its
// neighbour at a time: 86; the neighbour of four keys by a load of its own: 95).
template <bool STREAM>
__global__ __launch_bounds__(256) void k_dup(int64_t n, const uint64_t* __restrict__ k,
                                             unsigned long long* __restrict__ flag) {
    constexpr int kAhead = 4;
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * 256;
    const int64_t p0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool first_lane = lane_id() == 0;
    uint32_t d = 0;
    // every lane of a wave stays while one of them has keys
    for (int64_t p = p0; p - lane_id() < np; p += kAhead * stride) {
        u64x2 v[kAhead];
        uint64_t before[kAhead];
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            const int64_t i = p + g * stride;
            v[g] = u64x2{0ull, 0ull};
            before[g] = 0ull;
            if (i < np) v[g] = read<STREAM>(reinterpret_cast<const u64x2*>(k) + i);
            if (first_lane && i > 0 && i < np) before[g] = k[2 * i - 1];
        }
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            const int64_t i = p + g * stride;
            const uint32_t lo = __float_as_uint(wave_shr1(__uint_as_float((uint32_t)v[g].y), __uint_as_float((uint32_t)before[g])));
            const uint32_t hi = __float_as_uint(wave_shr1(__uint_as_float((uint32_t)(v[g].y >> 32)), __uint_as_float((uint32_t)(before[g] >> 32))));
            const uint64_t left = ((uint64_t)hi << 32) | lo;
            if (i < np) d |= (i > 0 && v[g].x == left) | (v[g].y == v[g].x);
        }
    }
    if (p0 == 0 && (n & 1) && n > 1) d |= k[n - 1] == k[n - 2];
    if (__ballot(d) != 0ull && lane_id() == 0) atomicOr(flag, 1ull);
}

// ===================================================================
// data ranges: order-preserving unsigned keys of floats, a NaN above them all
// ===================================================================
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

// Workgroup m folds the n_part partial ranges part[m * n_part ..] of field m
// into out[m] (pinned host memory); flag (optional): copied behind them.
__global__ __launch_bounds__(1024) void k_range_fold(int64_t n_part, const uint2* __restrict__ part,
                                                     uint2* __restrict__ out,
                                                     const unsigned long long* __restrict__ flag) {
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
        out[blockIdx.x] = r;
        if (blockIdx.x == 0 && flag) out[gridDim.x] = make_uint2((uint32_t)(*flag != 0ull), 0u);
    }
}

// ===================================================================
// Sorted arrays of a volume, one pass: gather by the permutation (or a copy
// of a contiguous range, perm NULL), zero padding, data range, per-tile and
// per-segment statistics, level codes.
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
// wave's steps, then the wave, then the four waves in order; segment sums: per
// lane the fp64 sum of its 4 values, then the row of 16 lanes.
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

template <bool STREAM, typename T>
__device__ __forceinline__ void put(T* dst, const Four<T>& v) {
    using W = typename std::conditional<sizeof(T) == 4, u32x4, u32x2>::type;
    if constexpr (STREAM)
        __builtin_nontemporal_store(__builtin_bit_cast(W, v), reinterpret_cast<W*>(dst));
    else
        *reinterpret_cast<Four<T>*>(dst) = v;
}

template <typename S, int G, bool STREAM>
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
            put<STREAM>(dst + c, r[g]);
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
            // a row of 16 lanes holds one segment
            d4 = row_total_d(d4);
            slo = row_lowest_f(slo);
            shi = row_highest_f(shi);
            if ((lane & 15) == 15) st.seg[((step0 + s + g) * kSegsPerStep + (lane >> 4)) * st.M + stat] = FieldStat{d4, slo, shi};
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
        st.tile[t * st.M + stat] = FieldStat{acc, lo, hi};
        if (st.range) st.range[stat * st.n_tiles + t] = range;
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

template <typename S, int G, bool STREAM>
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
            place_field<S, G, STREAM>(n, t, tile_steps, perm, reinterpret_cast<const typename S::raw*>(a.src[m]),
                              reinterpret_cast<typename S::raw*>(a.dst[m]), a.first_field + m, st);
        else
            place_levels<G>(n, t, tile_steps, perm, a.level_src, a.level_dst, a.codes);
        __syncthreads();
    }
}

// orig[perm[i]] = sorted[i]; the permutation itself to perm_out (or NULL) in the
// same pass
template <bool STREAM>
__global__ __launch_bounds__(256) void k_keys_back(int64_t n, const uint32_t* __restrict__ perm,
                                                   const uint64_t* __restrict__ sorted, uint64_t* __restrict__ orig,
                                                   uint32_t* __restrict__ perm_out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t p = read<STREAM>(perm + i);
        if (p < (uint64_t)n) orig[p] = read<STREAM>(sorted + i);
        if (perm_out) {
            if constexpr (STREAM)
                __builtin_nontemporal_store(p, perm_out + i);
            else
                perm_out[i] = p;
        }
    }
}

// Digits of 9 bits when that saves a pass over 8 (33-bit keys: 4 passes
// instead of 5; 50 M cells 2.92 against 3.10 ms in all), else 8: at 9 bits the
// runs of a 4096-cell tile are 8 words, 183 against 163 us a pass.  10 and 11
// bits were no faster (runs of 4 and 2 words: 195 and 274 us a pass).
static int sort_digit_bits(int key_bits) { return (key_bits + 8) / 9 < (key_bits + 7) / 8 ? 9 : 8; }

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

dvl_status launch_extent(int64_t n, const int32_t* x, const int32_t* y, const int32_t* z, const uint8_t* level,
                         unsigned long long* out, unsigned long long* dup, void* scratch, hipStream_t s) {
    ExtentPart* part = reinterpret_cast<ExtentPart*>(scratch);
    const unsigned grid = grid_for((n + 3) / 4, kReduceThreads, kReduceBlocks);
    if (vec4_inputs(x, y, z, level) && n > kStreamCells)
        hipLaunchKernelGGL((k_extent<true, true>), dim3(grid), dim3(kReduceThreads), 0, s, n, x, y, z, level, part);
    else if (vec4_inputs(x, y, z, level))
        hipLaunchKernelGGL((k_extent<true, false>), dim3(grid), dim3(kReduceThreads), 0, s, n, x, y, z, level, part);
    else
        hipLaunchKernelGGL((k_extent<false, false>), dim3(grid), dim3(kReduceThreads), 0, s, n, x, y, z, level, part);
    hipLaunchKernelGGL(k_extent_fold, dim3(1), dim3(1024), 0, s, (int)grid, part, out, dup);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

SortPlan sort_plan(int64_t n, int key_bits) {
    SortPlan p{};
    const int tile = sort_tile(n <= kSmallCells ? kSortItemsSmall : kSortItems);
    p.n_tiles = (n + tile - 1) / tile;
    p.chunk = sort_chunk(p.n_tiles);
    p.n_chunks = (p.n_tiles + p.chunk - 1) / p.chunk;
    p.idx_bits = 1;
    while (p.idx_bits < 32 && ((int64_t)1 << p.idx_bits) < n) ++p.idx_bits;
    p.packed = key_bits + p.idx_bits <= 64;
    p.digit_bits = sort_digit_bits(key_bits);
    p.passes = (key_bits + p.digit_bits - 1) / p.digit_bits;
    const size_t R = (size_t)1 << p.digit_bits;
    p.rows_words = (size_t)p.n_tiles * R;
    p.scratch_bytes = (p.rows_words + (size_t)p.n_chunks * R + R) * 4;
    return p;
}

template <int D, int ITEMS, bool PACKED, bool STREAM>
static dvl_status sort_typed(const SortPlan& p, int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                             const uint8_t* level, int bits, uint64_t* ka, uint64_t* kb, uint32_t* va, uint32_t* vb,
                             uint32_t* scratch, hipStream_t s, bool* in_second) {
    uint32_t* rows = scratch;
    uint32_t* totals = rows + p.rows_words;
    uint32_t* digits = totals + ((size_t)p.n_chunks << D);
    const dim3 chunks((unsigned)p.n_chunks), tiles((unsigned)p.n_tiles), thr(kSortThreads);
    const int low = PACKED ? p.idx_bits : 0;
    if (vec4_inputs(x, y, z, level))
        hipLaunchKernelGGL((k_words<D, ITEMS, PACKED, true>), chunks, thr, 0, s, n, x, y, z, level, bits, p.idx_bits, p.chunk,
                           p.n_tiles, ka, va, rows, totals);
    else
        hipLaunchKernelGGL((k_words<D, ITEMS, PACKED, false>), chunks, thr, 0, s, n, x, y, z, level, bits, p.idx_bits, p.chunk,
                           p.n_tiles, ka, va, rows, totals);
    DVL_HIP(hipGetLastError());
    *in_second = false;
    for (int i = 0; i < p.passes; ++i) {
        const int shift = low + D * i;
        if (i > 0) {
            hipLaunchKernelGGL((k_count<D, ITEMS, STREAM>), chunks, thr, 0, s, n, ka, shift, p.chunk, p.n_tiles, rows, totals);
            DVL_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(k_columns<D>, dim3((1 << D) / kColumnDigits), dim3(kColumnDigits * kColumnGroups), 0, s, p.n_chunks, totals,
                           digits);
        if (i + 1 == p.passes)
            hipLaunchKernelGGL((k_scatter<D, ITEMS, PACKED, true, STREAM>), tiles, thr, 0, s, n, ka, va, shift, p.idx_bits, p.chunk,
                               rows, totals, digits, kb, PACKED ? va : vb);   // packed: vin is not read
        else
            hipLaunchKernelGGL((k_scatter<D, ITEMS, PACKED, false, STREAM>), tiles, thr, 0, s, n, ka, va, shift, p.idx_bits, p.chunk,
                               rows, totals, digits, kb, vb);
        DVL_HIP(hipGetLastError());
        std::swap(ka, kb);
        if constexpr (!PACKED) std::swap(va, vb);   // packed: va is the permutation, vb may be NULL
        *in_second = !*in_second;
    }
    return DVL_OK;
}

dvl_status launch_order(const SortPlan& p, int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                        const uint8_t* level, int bits, uint64_t* ka, uint64_t* kb, uint32_t* va, uint32_t* vb,
                        uint32_t* scratch, hipStream_t s, bool* in_second) {
    const bool small = n <= kSmallCells, stream = n > kStreamCells;
#define DVL_SORT(D, ITEMS, STREAM)                                                                                     \
    if (p.digit_bits == D && small == (ITEMS == kSortItemsSmall) && stream == STREAM)                                  \
        return p.packed ? sort_typed<D, ITEMS, true, STREAM>(p, n, x, y, z, level, bits, ka, kb, va, vb, scratch, s,    \
                                                             in_second)                                                 \
                        : sort_typed<D, ITEMS, false, STREAM>(p, n, x, y, z, level, bits, ka, kb, va, vb, scratch, s,   \
                                                              in_second);
    DVL_SORT(8, kSortItemsSmall, false)
    DVL_SORT(9, kSortItemsSmall, false)
    DVL_SORT(8, kSortItems, false)
    DVL_SORT(9, kSortItems, false)
    DVL_SORT(8, kSortItems, true)
    DVL_SORT(9, kSortItems, true)
#undef DVL_SORT
    set_error("sort digits of %d bits", p.digit_bits);
    return DVL_E_INVALID;
}

dvl_status launch_dup(int64_t n, const uint64_t* keys, unsigned long long* flag, hipStream_t s) {
    const dim3 grid(grid_for((n + 7) / 8, 256, 2048));
    if (n > kStreamCells)
        hipLaunchKernelGGL(k_dup<true>, grid, dim3(256), 0, s, n, keys, flag);
    else
        hipLaunchKernelGGL(k_dup<false>, grid, dim3(256), 0, s, n, keys, flag);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

dvl_status launch_keys_back(int64_t n, const uint32_t* perm, const uint64_t* sorted, uint64_t* orig, uint32_t* perm_out,
                            hipStream_t s) {
    if (n > kStreamCells)
        hipLaunchKernelGGL(k_keys_back<true>, dim3(grid_for(n)), dim3(256), 0, s, n, perm, sorted, orig, perm_out);
    else
        hipLaunchKernelGGL(k_keys_back<false>, dim3(grid_for(n)), dim3(256), 0, s, n, perm, sorted, orig, perm_out);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

template <typename S>
static void range_of(int64_t n, const void* v, uint2* part, unsigned grid, hipStream_t s) {
    const auto* p = reinterpret_cast<const typename S::raw*>(v);
    if ((reinterpret_cast<uintptr_t>(v) & (Quad<S>::kBytes - 1)) == 0)
        hipLaunchKernelGGL((k_range<S, true>), dim3(grid), dim3(kReduceThreads), 0, s, n, p, part);
    else
        hipLaunchKernelGGL((k_range<S, false>), dim3(grid), dim3(kReduceThreads), 0, s, n, p, part);
}

dvl_status launch_range(int64_t n, int dtype, const void* v, uint2* part, int* n_part, hipStream_t s) {
    const unsigned grid = grid_for((n + 3) / 4, kReduceThreads, kReduceBlocks);
    if (dtype == DVL_F32)
        range_of<F32>(n, v, part, grid, s);
    else if (dtype == DVL_F16)
        range_of<F16>(n, v, part, grid, s);
    else
        range_of<BF16>(n, v, part, grid, s);
    DVL_HIP(hipGetLastError());
    *n_part = (int)grid;
    return DVL_OK;
}

template <typename S>
static void place_typed(int64_t n, int tile_steps, const uint32_t* perm, const PlaceArrays& a, const PlaceStats& st,
                        unsigned grid, hipStream_t s) {
    // tiles of 8 steps: two steps per wave; 16 and 32: four at a time
    if (tile_steps < 16)
        hipLaunchKernelGGL((k_place<S, 2, false>), dim3(grid), dim3(kReduceThreads), 0, s, n, tile_steps, perm, a, st);
    else if (n > kStreamCells)
        hipLaunchKernelGGL((k_place<S, 4, true>), dim3(grid), dim3(kReduceThreads), 0, s, n, tile_steps, perm, a, st);
    else
        hipLaunchKernelGGL((k_place<S, 4, false>), dim3(grid), dim3(kReduceThreads), 0, s, n, tile_steps, perm, a, st);
}

dvl_status launch_place(int64_t n, int dtype, int tile_steps, const uint32_t* perm, const PlaceArrays& a,
                        const PlaceStats& st, uint2* ranges, const unsigned long long* flag, hipStream_t s) {
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
        hipLaunchKernelGGL(k_range_fold, dim3(a.n_fields), dim3(1024), 0, s, st.n_tiles, st.range, ranges, flag);
        DVL_HIP(hipGetLastError());
    }
    return DVL_OK;
}

}  // namespace dvl
