// Per-update kernels (update.hip): device descriptors and launchers.
//
// An update batch is a list of requests; a request is one resident volume, its
// TF tables, parameters and outputs.  A single dvl_update is a batch of one.
#pragma once

#include <vector>

#include "common.hpp"

namespace dvl {

constexpr int kUpdThreads = 256;                 // 4 waves per workgroup
constexpr int kUpdWaves = kUpdThreads / kWave;
constexpr int kCellsPerLane = 4;                 // one 4-vector per field per step
constexpr int kStepCells = kWave * kCellsPerLane;    // 256 cells per wave step
constexpr int kDefaultTileSteps = 16;            // 4096-cell tiles unless tuned
constexpr int kPhases = 5;                       // exact vmax, tile sums, carry + classification, rescan, bin statistics
constexpr int kPathValues = 1;                   // requests that read the field values
constexpr int kPathEntries = 2;                  // requests that read cached TF entries
constexpr int kPathBinStoredF = 4;               // requests whose projection reads stored f,
constexpr int kPathBinEntries = 8;               // cached entries,
constexpr int kPathBinValues = 16;               // or values
constexpr int kPathAlone = 32;                   // value readers that belong to no Share
constexpr int kIdxTable = 256;                   // LDS floats per table on the cached-entry path

// A bin edge's tile and its pixel interval, when the edge is the tile's first
// inner edge; else tile < 0 (another edge has the tile, or no tile holds it).
struct alignas(16) EdgeRec {
    int32_t tile;
    float X0, X1;
    int32_t pad_;
};

// Workspace of one request on a volume of T tiles and M fields.
struct UpdWorkspace {
    double* local_prefix; // [T]  sum of the importance of earlier tiles of the same run
    double* run_total;    // [R]  sum over each run of consecutive tiles
    float* x0;            // [T + 1]  pixel position of the tile's first cell; x0[T]: end of the last
    int32_t* head_bin;    // [T]  bin of the tile's first cell
    int32_t* tail_bin;    // [T]  bin of the tile's last cell
    uint32_t* rec_first;  // [2][T]  cell range of the tile's head bin, then of its tail bin
    uint32_t* rec_last;   // [2][T]
    int32_t* bin_t1;      // [W]  last tile whose first cell's bin is <= b (the last tile touching bin b)
    int32_t* bin_ta;      // [W]  first tile whose pixel interval ends in bin >= b (bin b's first
                          //      tile, or the one before it when that tile's last cell ends exactly at b)
    EdgeRec* edge;        // [W]  the tile that holds bin edge b (left edge of bin b)
    double* scal;         // [0] F_tot, [1] degenerate (0/1), [2] pixels per importance
    float* fstore;        // [n_pad] importance of every cell, or NULL (see wants_fstore)
};

// n_bins: the request's W; fcells: cells of the stored importance (0: none)
size_t workspace_bytes(int64_t n_tiles, int M, int n_bins, int64_t fcells = 0);
void workspace_carve(void* base, int64_t n_tiles, int M, int n_bins, int64_t fcells, UpdWorkspace* w);

// Whether a request stores f in the importance pass for the projection to
// reuse: worth its 4 B per cell once about a quarter or more of the tiles
// hold a bin edge (the projection then rescans most of the volume).
inline bool wants_fstore(int64_t n_tiles, int n_bins) { return (int64_t)n_bins * 4 >= n_tiles; }

// The volume of a request.
struct VolDev {
    int64_t n;
    int n_tiles;              // below 2^21 (n < 2^32, tiles of at least 2048 cells)
    int tiles_per_run;        // importance-pass run r owns tiles [r k, (r + 1) k)
    int n_runs;
    int M;
    int tile_steps;           // 256-cell steps per tile
    int split;                // a workgroup's waves share one tile (see k_tile_sums)
    const uint8_t* level;
    const uint32_t* lcode;    // per-step level codes (launch_place)
    const FieldStat* tile_stat;   // [T][M]
    const FieldStat* seg_stat;    // [T * tile_steps * kSegsPerStep][M]
    const void* fields[kMaxFields];
    const uint8_t* idx[kMaxFields];   // cached TF entries per field (entries path)
};

constexpr int kNoFold = 0x100;
constexpr int kValuesShared = 2;
// One request: everything its kernels read, in one place (a kernel's first
// loads are its chain of cold misses: one descriptor, no pointer to another).
struct ReqDev {
    VolDev v;
    const float* tf;          // this request's tables (device)
    float* vmax_dev;          // max(V) used: host value, or computed (exact mode)
    UpdWorkspace ws;
    int W;
    int entries;              // the importance pass reads cached entries (1), values (0), values in a Share (2)
    int bin_path;             // the projection reads values (0), cached entries (1) or stored f (2)
    int by_tile;              // k_bin: a workgroup per tile (1) or per bin edge (0)
    int tf_total;             // floats in this request's block
    float exponent;
    float fmin;
    int exp_is_one;
    int clamp_mode;
    int level_shift;          // 1: 2^L, 3: 8^L; | kNoFold: V / max V may round as a subnormal that shows in f
    int scan_mode;
    int vmax_exact;
    uint32_t* first_cell;
    uint32_t* last_cell;
    float* mean;
    float* vmin;
    float* vmax;
    float* y;
    double* f_total;
    float* vmax_used;
    float s[kMaxFields];      // quantiser scale per field
    float b[kMaxFields];      // quantiser offset per field
    float nmax[kMaxFields];   // n_tf - 1 per field
    int tf_off[kMaxFields];   // start of field m's table inside this request's block
};

// The importance pass's units of work are numbered request after request
// (unit0: each request's first).  Requests on one volume run at the same pace
// side by side, so that their cells come from the caches after the first.  (A
// kernel that evaluated up to 8 requests per read of a cell held 183 KB of code
// against 64 KB of instruction cache: 341 us for 4 requests on each of two 20
// M-cell volumes, cached entries; one request at a time takes 119 us.)
struct BatchDev {
    const int64_t* unit0;     // [n_reqs]
    const ReqDev* reqs;
    int n_reqs;
    int64_t k1_units;
    int64_t chain;            // consecutive units a workgroup of the importance pass or K0 takes
    int64_t n_steps;          // 256-cell steps of all requests
    int stream;               // read the cells as streams that bypass the caches (see batch_dev)
    int any_exact;
    int paths;                // kPath*: which variants of the importance pass and the projection to launch
    int max_req_tf;           // largest request table block (floats)
    int max_fields;           // most fields of a volume
    int max_tile_steps;       // largest tile (256-cell steps) of the batch's volumes
    int max_tiles;            // most tiles of a volume
    int max_w;                // most bins of a request
    int max_bin_units;        // most k_bin workgroups of a request
    int share;                // requests of a share launched by itself, 0: the rest of the batch
};

// Requests [req0, req0 + n_req) on one volume that read its values in one launch
// of the importance pass, side by side, so that each cell is fetched from HBM
// once for all of them; units: importance-pass units of each.
struct Share {
    int req0, n_req;
    int64_t units;
    bool operator==(const Share& o) const { return req0 == o.req0 && n_req == o.n_req && units == o.units; }
};

// What launch_batch is given: the batch as the kernels see it, its shares, and
// whether a plot is so wide that single cells or tiles reach many bins.
struct BatchLaunch {
    BatchDev dev;
    std::vector<Share> shares;
    bool far;
};

// Whether a plot is so wide that writing the bins of one tile, or of one cell,
// is worth the whole wave or workgroup: 32 bins per tile, one per 16 cells.  (Only
// then the kernels that can do it run: the tests cost the others 0.4 us each.)
constexpr int kFarTile = 32, kFarCells = 16;
__host__ __device__ inline bool far_tiles(int64_t n_tiles, int n_bins) { return n_bins >= kFarTile * n_tiles; }
__host__ __device__ inline bool far_bins(int64_t n, int64_t n_tiles, int n_bins) {
    return far_tiles(n_tiles, n_bins) || (int64_t)n_bins * kFarCells >= n;
}

// The descriptor layout a translation unit was compiled with.  The host
// code that writes the descriptors and every unit whose kernels read them
// must agree; launch_batch refuses a mismatch (objects built from different
// versions of this header) before any kernel runs.
constexpr uint64_t kDescriptorLayout =
    ((uint64_t)sizeof(ReqDev) << 40) | ((uint64_t)sizeof(VolDev) << 20) | (uint64_t)sizeof(BatchDev);

// Launch the five phases for the batch described by `b` (descriptors already
// resident on the device).  `max_m`: the field count when every volume has
// the same (1 to 8), else kMaxFields.  `layout`: the caller's
// kDescriptorLayout.  ev (optional): kPhases + 1 events.
dvl_status launch_batch(const BatchLaunch& b, int dtype, int max_m, int n_cu, hipStream_t s, uint64_t layout,
                        hipEvent_t* ev = nullptr);

// TF entry of every cell of one sorted field under quantiser (s, b) with
// n_tf <= 256 entries, one byte per cell, over all n_pad (padded) cells.
dvl_status launch_build_index(int64_t n_pad, int dtype, const void* field, float s, float b, int n_tf,
                              uint8_t* out, int n_cu, hipStream_t st);

}  // namespace dvl
