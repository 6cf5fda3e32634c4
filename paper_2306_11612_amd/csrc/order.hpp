// Launchers of the one-time ordering kernels (order.hip).
#pragma once

#include "common.hpp"

namespace dvl {

// out (memory the host can read once the stream is synchronised):
// [0] max(corner + 2^level), [1] a cell fails the checks, [2] max level;
// dup: device word, zeroed; scratch: extent_scratch_bytes() of device memory
size_t extent_scratch_bytes();
dvl_status launch_extent(int64_t n, const int32_t* x, const int32_t* y, const int32_t* z, const uint8_t* level,
                         unsigned long long* out, unsigned long long* dup, void* scratch, hipStream_t s);
// The ordering of n cells with keys of key_bits bits: sort layout and scratch.
struct SortPlan {
    int64_t n_tiles, n_chunks;
    int chunk;               // tiles per counting workgroup
    int idx_bits;            // bits of a cell index
    bool packed;             // key and index in one 64-bit word
    int digit_bits, passes;
    size_t rows_words;
    size_t scratch_bytes;    // device scratch of launch_order
};
SortPlan sort_plan(int64_t n, int key_bits);
// Hilbert keys of the cells (bits per axis) and a stable sort of (key, index):
// the sorted keys end in kb when *in_second, else in ka, the permutation
// likewise in vb or va; with p.packed vb is not used (may be NULL) and the
// permutation is in va.  ka, kb: 8 bytes per cell; va, vb: 4.
dvl_status launch_order(const SortPlan& p, int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                        const uint8_t* level, int bits, uint64_t* ka, uint64_t* kb, uint32_t* va, uint32_t* vb,
                        uint32_t* scratch, hipStream_t s, bool* in_second);
dvl_status launch_dup(int64_t n, const uint64_t* keys, unsigned long long* flag, hipStream_t s);
// orig[perm[i]] = sorted[i]; perm_out (or NULL): a copy of perm
dvl_status launch_keys_back(int64_t n, const uint32_t* perm, const uint64_t* sorted, uint64_t* orig, uint32_t* perm_out,
                            hipStream_t s);
// Partial ranges of n values: part[i] = (min, max) as order-preserving uint
// keys for i < *n_part <= kRangeParts, max = kRangeNan where there is a NaN.
// part: memory the host can read once the stream is synchronised.
constexpr int kRangeParts = 1024;
constexpr uint32_t kRangeNan = 0xFFFFFFFFu;   // above the key of +inf
dvl_status launch_range(int64_t n, int dtype, const void* v, uint2* part, int* n_part, hipStream_t s);

// The sorted arrays of a volume: fields src -> dst (statistics rows
// first_field ..) and, when level_src is not NULL, the levels and their codes.
// dst arrays hold whole tiles; cells past n are zeroed.
struct PlaceArrays {
    const void* src[kMaxFields];
    void* dst[kMaxFields];
    int n_fields;
    int first_field;
    const uint8_t* level_src;
    uint8_t* level_dst;
    uint32_t* codes;         // one 32-bit level code per 256-cell step
};
struct PlaceStats {
    int64_t n_tiles;
    int M;                   // fields of the volume
    FieldStat* tile;         // [n_tiles][M]
    FieldStat* seg;          // [n_tiles * tile_steps * kSegsPerStep][M]
    uint2* range;            // [n_fields][n_tiles] range keys per tile, or NULL
};
// sorted cell i from original cell perm[i], or from src[i] when perm is NULL;
// ranges (optional, needs st.range and first_field 0): per field as
// launch_range, then, with `flag`, whether that device word is set; memory the
// host can read once the stream is synchronised
dvl_status launch_place(int64_t n, int dtype, int tile_steps, const uint32_t* perm, const PlaceArrays& a,
                        const PlaceStats& st, uint2* ranges, const unsigned long long* flag, hipStream_t s);

}  // namespace dvl
