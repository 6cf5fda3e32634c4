// C ABI of the DVL library: validation, buffer ownership, host-side TF
// preparation (Eqs. 5-6 run on the host, as in the paper's GPU section),
// batch planning and kernel launches.  Declarations and contracts:
// include/dvl.h.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "order.hpp"
#include "update.hpp"
#include "views.hpp"

namespace dvl {

static thread_local std::string g_err;

void set_error(const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
}

dvl_status hip_fail(hipError_t e, const char* what) {
    set_error("HIP error %d (%s) in %s", (int)e, hipGetErrorString(e), what);
    return DVL_E_HIP;
}

static dvl_status fail(dvl_status code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

static int elem_bytes_of(int dtype) { return dtype == DVL_F32 ? 4 : 2; }

// Device memory of the library: through the caller's dvl_allocator when one
// was given, else hipMalloc / hipFree.  Every buffer is released through the
// allocator that made it.
struct Alloc {
    dvl_allocator a{};
    bool custom = false;
    void* get(size_t bytes, hipStream_t s) const {
        if (bytes == 0) bytes = 1;
        if (custom) return a.alloc(a.ctx, bytes, (void*)s);
        void* p = nullptr;
        if (hipMalloc(&p, bytes) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        return p;
    }
    void put(void* p, hipStream_t s) const {
        if (!p) return;
        if (custom)
            a.release(a.ctx, p, (void*)s);
        else
            (void)hipFree(p);
    }
};

static dvl_status make_alloc(const dvl_allocator* a, Alloc& out) {
    out = Alloc();
    if (!a) return DVL_OK;
    if (!a->alloc || !a->release) return fail(DVL_E_INVALID, "allocator needs both alloc and release");
    out.a = *a;
    out.custom = true;
    return DVL_OK;
}

// device buffer owned by RAII until released
struct DevBuf {
    const Alloc* A;
    void* p = nullptr;
    bool idle = false;      // the stream of every kernel that used it was synchronised
    explicit DevBuf(const Alloc& a) : A(&a) {}
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    // a buffer still owned here is a temporary or the leftover of a failing
    // call: kernels enqueued on it may still run, so wait before handing it back
    ~DevBuf() {
        if (p) {
            if (!idle) (void)hipDeviceSynchronize();
            A->put(p, nullptr);
        }
    }
    dvl_status alloc(size_t bytes, const char* what) {
        p = A->get(bytes, nullptr);
        if (!p) return fail(DVL_E_NOMEM, "device allocation of %zu bytes for %s failed", bytes, what);
        return DVL_OK;
    }
    void* release() { void* q = p; p = nullptr; return q; }
};

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// Pinned host memory for a call that waits for results: a kernel writes them
// there directly, and the host reads them after it has synchronised the stream
// (a copy of a few bytes into pageable memory costs 10 to 15 us more).  Buffers
// come from a process-wide list of at most kKept free ones (allocating one takes
// longer than most calls that need it); a buffer is used by one call at a time,
// whatever its thread, stream and volume, and goes back when the call ends,
// after the device is idle unless the call says it has synchronised.
template <size_t kBytes, int kKept>
struct HostBuffer {
    inline static std::mutex mu;
    inline static void* kept[kKept];
    inline static int n_kept = 0;
    void* p = nullptr;
    bool idle = false;
    HostBuffer() = default;
    HostBuffer(const HostBuffer&) = delete;
    HostBuffer& operator=(const HostBuffer&) = delete;
    dvl_status take() {
        {
            std::lock_guard<std::mutex> lk(mu);
            if (n_kept > 0) {
                p = kept[--n_kept];
                return DVL_OK;
            }
        }
        if (hipHostMalloc(&p, kBytes, hipHostMallocPortable) != hipSuccess) {
            p = nullptr;
            (void)hipGetLastError();
            return fail(DVL_E_NOMEM, "pinned host allocation of %zu bytes failed", kBytes);
        }
        return DVL_OK;
    }
    ~HostBuffer() {
        if (!p) return;
        if (!idle) (void)hipDeviceSynchronize();
        {
            std::lock_guard<std::mutex> lk(mu);
            if (n_kept < kKept) {
                kept[n_kept++] = p;
                return;
            }
        }
        (void)hipHostFree(p);
    }
};
// a few results; the bins that dvl_read_bins returns, up to this size through one
// kernel (1920 bins of 16 fields: 0.5 MB), larger ones array by array, where the
// copies' own rate counts
constexpr size_t kHostPageBytes = 16384, kReadStageBytes = (size_t)1 << 20;
using HostPage = HostBuffer<kHostPageBytes, 8>;
using ReadStage = HostBuffer<kReadStageBytes, 4>;
static_assert((size_t)kRangeParts * sizeof(uint2) <= kHostPageBytes, "the partial ranges fit a page");

// order-preserving uint key (as produced by the range kernel) back to float
static float unkey(unsigned int u) {
    const unsigned int b = (u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u;
    float f;
    memcpy(&f, &b, 4);
    return f;
}

constexpr int kRing = 4;                 // descriptor uploads that may be in flight

// The quantisers of every field: the TF entry of a cell depends on its value
// and on these only, not on the alpha tables.
struct CacheKey {
    int M = 0;
    int n_tf[kMaxFields] = {};
    float s[kMaxFields] = {}, b[kMaxFields] = {};
    float lo[kMaxFields] = {}, hi[kMaxFields] = {};   // the windows (informational, not compared)
    bool operator==(const CacheKey& o) const {
        return M == o.M && memcmp(n_tf, o.n_tf, sizeof n_tf) == 0 && memcmp(s, o.s, sizeof s) == 0 &&
               memcmp(b, o.b, sizeof b) == 0;
    }
};

// Uploads through kernel arguments (the allocation-free entry point): k_poke
// writes up to kPokeWords words carried in its arguments, in the stream's own
// queue (no memcpy or memset node).
constexpr int kPokeWords = 768;
struct PokeArgs {
    uint32_t* dst;
    uint32_t n;
    uint32_t w[kPokeWords];
};

__global__ __launch_bounds__(256) void k_poke(PokeArgs a) {
    for (uint32_t i = threadIdx.x; i < a.n; i += blockDim.x) a.dst[i] = a.w[i];
}

static dvl_status poke(char* dst, const char* src, size_t bytes, hipStream_t s) {
    const size_t nw = bytes / 4;
    PokeArgs a;
    for (size_t i = 0; i < nw; i += kPokeWords) {
        a.dst = reinterpret_cast<uint32_t*>(dst) + i;
        a.n = (uint32_t)std::min<size_t>(kPokeWords, nw - i);
        memcpy(a.w, src + 4 * i, (size_t)a.n * 4);
        hipLaunchKernelGGL(k_poke, dim3(1), dim3(256), 0, s, a);
        DVL_HIP(hipGetLastError());
    }
    return DVL_OK;
}

struct Executor;

}  // namespace dvl

using namespace dvl;

struct dvl_volume {
    int64_t n = 0;
    int64_t n_pad = 0;       // cells rounded up to whole tiles
    int64_t n_tiles = 0;
    int32_t tile_steps = kDefaultTileSteps;
    int64_t tiles_per_run = 1;
    int64_t n_runs = 1;
    int32_t M = 0;
    int32_t dtype = DVL_F32;
    int32_t bits = 0;
    int32_t max_level = 0;
    int device = 0;
    int n_cu = 256;
    uint8_t* level_s = nullptr;
    uint32_t* lcode_s = nullptr;      // per-step level codes [n_pad / 256]
    void* fields_s[kMaxFields] = {};
    uint64_t* keys_s = nullptr;
    uint32_t* perm = nullptr;
    float dmin[kMaxFields] = {};
    float dmax[kMaxFields] = {};
    // statistics of the sorted fields per tile and per 64-cell segment
    FieldStat* tile_stat = nullptr;   // [T][M]
    FieldStat* seg_stat = nullptr;    // [T * tile_steps * kSegsPerStep][M]
    // TF entry cache: one byte per sorted cell and field for one CacheKey
    // (policy DVL_ENTRY_CACHE_*); `cand` is the key of the last update that
    // could have used a cache, so a key seen twice in a row gets one
    uint8_t* idx_s[kMaxFields] = {};
    int32_t idx_policy = DVL_ENTRY_CACHE_AUTO;
    bool idx_valid = false;
    CacheKey idx_key;
    bool cand_set = false;
    CacheKey cand_key;
    // (the cache of every field is one allocation, idx_s[0])
    // Ordering of cache rebuilds against the launches that read the cache,
    // by events instead of device synchronisation: a rebuild on stream s
    // first waits for the last reading launch on every stream; a launch that
    // reads the cache first waits for the rebuild (`cache_ready`).
    hipEvent_t cache_ready = nullptr;
    bool cache_ready_recorded = false;
    hipStream_t cache_ready_stream = nullptr;   // where the last rebuild ran
    std::vector<hipStream_t> cache_readers;     // streams whose launches read the cache
    // the volume's own transfer functions (used by dvl_update)
    bool tf_set[kMaxFields] = {};
    std::vector<float> alpha[kMaxFields];
    float lo[kMaxFields] = {}, hi[kMaxFields] = {};
    Executor* ex = nullptr;  // private executor of dvl_update
    dvl::Alloc alloc;        // every device buffer of the volume comes from here
    char* slab = nullptr;    // the arrays above in one hipMalloc, when the caller gave no allocator
    size_t slab_size = 0, slab_used = 0;
    dvl_status sticky = DVL_OK;
    size_t bytes = 0;
};

namespace dvl {

// ================================================================== host TF prep

// FP32 quantiser of the window [lo, hi] for n_tf entries
static void quantiser(int n_tf, float lo, float hi, float* s, float* b) {
    const float sf = (float)((double)n_tf / ((double)hi - (double)lo));
    *s = sf;
    *b = (float)(-(double)lo * (double)sf);
}

static int host_entry(float x, float s, float b, int n_tf) {
    float t = fmaf(x, s, b);
    if (!(t >= 0.0f)) return 0;
    if (t > (float)(n_tf - 1)) return n_tf - 1;
    return (int)t;
}

// One update request as the host sees it: tables, windows, parameters, outputs.
struct ReqHost {
    dvl_volume* v = nullptr;
    int n_tf[kMaxFields] = {};       // entries of field m's table
    int off[kMaxFields] = {};        // start of field m's table in `alpha`
    int total = 0;                   // floats in `alpha`
    std::vector<float> alpha;        // tables, field after field
    float lo[kMaxFields] = {}, hi[kMaxFields] = {};
    float qs[kMaxFields] = {}, qb[kMaxFields] = {};
    dvl_params p{};
    dvl_bins out{};
    size_t tf_pos = 0;               // floats from the start of the batch's tables
};

// Eqs. 5-6 and the bound variant (section "Computing the Maximum Local
// Ensemble Variation"): max(V_h) from the TFs and the fields' data ranges
static float host_vmax(const ReqHost& r) {
    const dvl_volume* v = r.v;
    const int M = v->M;
    auto A = [&](int m, int a) { return r.alpha[(size_t)r.off[m] + std::min(a, r.n_tf[m] - 1)]; };
    int im[kMaxFields], jm[kMaxFields];
    for (int m = 0; m < M; ++m) {
        im[m] = host_entry(v->dmin[m], r.qs[m], r.qb[m], r.n_tf[m]);
        jm[m] = host_entry(v->dmax[m], r.qs[m], r.qb[m], r.n_tf[m]);
    }
    auto bound = [&]() {
        float hi = -INFINITY, lo = INFINITY;
        for (int m = 0; m < M; ++m)
            for (int a = im[m]; a <= jm[m]; ++a) {
                hi = std::max(hi, A(m, a));
                lo = std::min(lo, A(m, a));
            }
        return hi - lo;
    };
    if (r.p.vmax_mode == DVL_VMAX_TF_BOUND) return bound();
    int i = im[0], j = jm[0];
    for (int m = 1; m < M; ++m) { i = std::min(i, im[m]); j = std::max(j, jm[m]); }
    float best = 0.0f;
    for (int a = i; a <= j; ++a) {
        float hi = -INFINITY, lo = INFINITY;
        for (int m = 0; m < M; ++m) {
            hi = std::max(hi, A(m, a));
            lo = std::min(lo, A(m, a));
        }
        best = std::max(best, hi - lo);
    }
    if (best <= 0.0f) best = bound();   // the literal approximation can vanish (e.g. equal TFs)
    return best;
}

static dvl_status check_params(const dvl_params* p) {
    if (!p) return fail(DVL_E_INVALID, "params is NULL");
    if (p->n_bins < 1 || p->n_bins > (1 << 20)) return fail(DVL_E_INVALID, "n_bins=%d outside [1, 2^20]", p->n_bins);
    if (!(p->exponent >= 0.0f && p->exponent <= 16.0f)) return fail(DVL_E_INVALID, "exponent %g outside [0, 16]", p->exponent);
    if (!(p->min_importance >= 0.0f) || !isfinite(p->min_importance))
        return fail(DVL_E_INVALID, "min_importance %g must be finite and >= 0", p->min_importance);
    if (p->vmax_mode < 0 || p->vmax_mode > 2) return fail(DVL_E_INVALID, "vmax_mode %d", p->vmax_mode);
    if (p->clamp_mode < 0 || p->clamp_mode > 1) return fail(DVL_E_INVALID, "clamp_mode %d", p->clamp_mode);
    if (p->level_scale != 1 && p->level_scale != 3) return fail(DVL_E_INVALID, "level_scale %d (1 or 3)", p->level_scale);
    if (p->scan_mode < 0 || p->scan_mode > 2) return fail(DVL_E_INVALID, "scan_mode %d", p->scan_mode);
    return DVL_OK;
}

static dvl_status check_bins(const dvl_bins* b) {
    if (!b) return fail(DVL_E_INVALID, "bins is NULL");
    if (!b->first_cell || !b->last_cell || !b->mean || !b->vmin || !b->vmax || !b->y || !b->f_total ||
        !b->vmax_used)
        return fail(DVL_E_INVALID, "a bins pointer is NULL");
    return DVL_OK;
}

static dvl_status check_volume(const dvl_volume* v) {
    if (!v) return fail(DVL_E_INVALID, "volume is NULL");
    if (v->sticky != DVL_OK) return fail(v->sticky, "volume is in a failed state after an earlier device error");
    return DVL_OK;
}

// Resolve field m's window (NULL bounds: the data range), its quantiser, and
// check both are usable in fp32.
static dvl_status set_window(ReqHost& r, int m, const float* lo, const float* hi) {
    const dvl_volume* v = r.v;
    float l = lo ? lo[m] : v->dmin[m], h = hi ? hi[m] : v->dmax[m];
    if (!lo && !hi && !(h > l)) h = nextafterf(l, INFINITY);   // constant field
    if (!isfinite(l) || !isfinite(h) || !(l < h))
        return fail(DVL_E_INVALID, "window [%g, %g] of field %d is not finite with lo < hi", l, h, m);
    r.lo[m] = l;
    r.hi[m] = h;
    quantiser(r.n_tf[m], l, h, &r.qs[m], &r.qb[m]);
    if (!isfinite(r.qs[m]) || !isfinite(r.qb[m]))
        return fail(DVL_E_INVALID, "window [%g, %g] of field %d is too narrow for fp32", l, h, m);
    return DVL_OK;
}

static dvl_status check_tables(const ReqHost& r) {
    if (r.total > kMaxTfTotal) return fail(DVL_E_INVALID, "sum of TF sizes %d exceeds %d", r.total, kMaxTfTotal);
    for (float a : r.alpha)
        if (!isfinite(a)) return fail(DVL_E_INVALID, "an alpha entry is not finite");
    return DVL_OK;
}

// A request from caller inputs: alpha [M][n_tf], windows lo/hi [M] or NULL.
static dvl_status make_request(dvl_volume* v, const float* alpha, int n_tf, const float* lo, const float* hi,
                               const dvl_params* p, const dvl_bins* out, ReqHost& r) {
    if (dvl_status st = check_volume(v)) return st;
    if (dvl_status st = check_params(p)) return st;
    if (dvl_status st = check_bins(out)) return st;
    if (!alpha) return fail(DVL_E_INVALID, "alpha is NULL");
    if (n_tf < 2 || n_tf > kMaxTfEntries) return fail(DVL_E_INVALID, "n_tf=%d outside [2, %d]", n_tf, kMaxTfEntries);
    r = ReqHost();
    r.v = v;
    for (int m = 0; m < v->M; ++m) {
        r.n_tf[m] = n_tf;
        r.off[m] = m * n_tf;
    }
    r.total = v->M * n_tf;
    if (r.total > kMaxTfTotal) return fail(DVL_E_INVALID, "n_fields * n_tf = %d exceeds %d", r.total, kMaxTfTotal);
    r.alpha.assign(alpha, alpha + r.total);
    if (dvl_status st = check_tables(r)) return st;
    for (int m = 0; m < v->M; ++m)
        if (dvl_status st = set_window(r, m, lo, hi)) return st;
    r.p = *p;
    r.out = *out;
    return DVL_OK;
}

// A request from the volume's own TF state (dvl_set_tf).
static dvl_status volume_request(dvl_volume* v, const dvl_params* p, const dvl_bins* out, ReqHost& r) {
    if (dvl_status st = check_volume(v)) return st;
    for (int m = 0; m < v->M; ++m)
        if (!v->tf_set[m]) return fail(DVL_E_STATE, "field %d has no transfer function", m);
    if (dvl_status st = check_params(p)) return st;
    if (dvl_status st = check_bins(out)) return st;
    r = ReqHost();
    r.v = v;
    for (int m = 0; m < v->M; ++m) {
        r.n_tf[m] = (int)v->alpha[m].size();
        r.off[m] = r.total;
        r.total += r.n_tf[m];
        r.alpha.insert(r.alpha.end(), v->alpha[m].begin(), v->alpha[m].end());
        r.lo[m] = v->lo[m];
        r.hi[m] = v->hi[m];
        quantiser(r.n_tf[m], r.lo[m], r.hi[m], &r.qs[m], &r.qb[m]);
    }
    r.p = *p;
    r.out = *out;
    return DVL_OK;
}

// the largest importance a cell can reach, times a tile, must stay finite in fp32
static dvl_status check_range(const ReqHost& r, float vmax) {
    float amax = -INFINITY, amin = INFINITY;
    for (float a : r.alpha) { amax = std::max(amax, a); amin = std::min(amin, a); }
    const double vr = (double)amax - (double)amin;
    const bool exact = r.p.vmax_mode == DVL_VMAX_EXACT;
    const double rmax = exact ? 1.0 : (vmax > 0.0f ? vr / (double)vmax : 0.0);
    const double g = std::max((double)r.p.min_importance, rmax) * ldexp(1.0, r.p.level_scale * r.v->max_level);
    const double fmax_cell = std::max((double)r.p.min_importance, pow(g, (double)r.p.exponent));
    if (!(fmax_cell * (double)r.v->tile_steps * kStepCells < 1e37))
        return fail(DVL_E_RANGE, "importance can reach %g: exponent and levels overflow fp32", fmax_cell);
    return DVL_OK;
}

// Whether the importance pass may scale 1 / max V by the level scale instead of
// V / max V (kNoFold: it may not).  The products differ only where V / max V is
// subnormal and rounds: below 2^-126, which the largest level scale (2^60)
// takes to 2^-66.  A minimum importance from there on hides it, and so do alphas
// none of which is tiny: they are multiples of 2^-24 times the smallest of them
// but 0, and so is V, and max V is at most their span.
static bool folds(const ReqHost& r) {
    if (r.p.min_importance >= 0x1p-66f) return true;
    float amax = -INFINITY, amin = INFINITY, least = INFINITY;
    for (float a : r.alpha) {
        amax = std::max(amax, a);
        amin = std::min(amin, a);
        if (a != 0.0f) least = std::min(least, fabsf(a));
    }
    return (double)least >= ((double)amax - (double)amin) * 0x1p-100;
}

// ================================================================== batch plans

// The requests on one volume, consecutive in the batch.
struct VolReqs {
    int req0, n_req;
};

struct Plan {
    std::vector<ReqHost> reqs;       // grouped by volume
    std::vector<int> where;          // caller's request index -> index in `reqs`
    std::vector<VolReqs> groups;     // one per volume
    std::vector<Share> shares;       // value readers that share reads (plan_paths)
    std::vector<int64_t> unit0;      // each request's first importance-pass unit
    std::vector<ReqDev> rdev;
    std::vector<float*> fstore;      // where each request may store f, or NULL
    int dtype = DVL_F32;
    int max_m = 1;
    int max_fields = 1;
    int max_req_tf = 0;
    int max_tile_steps = 8;
    int max_tiles = 1;
    int max_w = 1;
    int max_bin_units = 1;
    int any_exact = 0;
    bool far = false;
    int64_t k1_units = 0;
    int64_t n_steps = 0;
    size_t tf_floats = 0;
    // descriptor block, uploaded before every launch:
    //   [unit0 x reqs][ReqDev x reqs][max V x reqs][tables]
    size_t off_reqs = 0, off_vmax = 0, off_tf = 0, block_bytes = 0;
};

// Volumes of at most this many one-tile runs have each tile shared by a
// workgroup's four waves in the importance pass: a wave per tile would leave
// half the chip's wave slots or more idle.  Whole updates, W = 1920, fp32, a wave
// per tile / four: P = 2 (4 fields, entries) 1264 tiles 90 / 71 us, 2040 93 / 89,
// 2880 108 / 104; entries of 4 fields 1000 tiles 50 / 48, 1400 53 / 54, 2040 57 / 62,
// 2880 61 / 65; values of 8 fields 1000 67 / 72, 1400 77 / 84, 2040 100 / 109, 2100
// 120 / 111, 2880 134 / 141.  The line is where it pays with an exponent; without
// one a wave per tile is up to 14 % ahead from some 1200 tiles on.
constexpr int kSplitTiles = 2048;

static VolDev vol_dev(const dvl_volume* v) {
    VolDev d{};
    d.n = v->n;
    d.n_tiles = (int)v->n_tiles;
    d.tiles_per_run = (int)v->tiles_per_run;
    d.n_runs = (int)v->n_runs;
    d.M = v->M;
    d.tile_steps = v->tile_steps;
    // a wave's quarter of a tile must start on a group of four level codes
    d.split = v->tiles_per_run == 1 && v->n_tiles <= kSplitTiles && v->tile_steps >= 16;
    d.level = v->level_s;
    d.lcode = v->lcode_s;
    for (int m = 0; m < v->M; ++m) d.fields[m] = v->fields_s[m];
    d.tile_stat = v->tile_stat;
    d.seg_stat = v->seg_stat;
    return d;
}

// Units of the importance pass of one request: a run per wave, or a tile.
static int64_t request_units(const VolDev& v) {
    return v.split ? v.n_runs : (v.n_runs + kUpdWaves - 1) / kUpdWaves;
}

// Group the requests by volume and lay out the work units of every phase and
// the descriptor block.
static dvl_status plan_batch(std::vector<ReqHost>&& reqs, Plan& P) {
    P = Plan();
    if (reqs.empty()) return fail(DVL_E_INVALID, "empty batch");
    P.dtype = reqs[0].v->dtype;
    for (auto& r : reqs)
        if (r.v->dtype != P.dtype) return fail(DVL_E_INVALID, "a batch mixes field storage types");
    std::vector<bool> taken(reqs.size(), false);
    P.where.assign(reqs.size(), 0);
    for (size_t i = 0; i < reqs.size(); ++i) {
        if (taken[i]) continue;
        VolReqs g{};
        g.req0 = (int)P.reqs.size();
        dvl_volume* v = reqs[i].v;
        for (size_t k = i; k < reqs.size(); ++k)
            if (!taken[k] && reqs[k].v == v) {
                P.where[k] = (int)P.reqs.size();
                P.reqs.push_back(std::move(reqs[k]));
                taken[k] = true;
            }
        g.n_req = (int)P.reqs.size() - g.req0;
        P.groups.push_back(g);
    }
    // The kernels are specialised on the field count: batches whose volumes
    // all have the same 1 to 8 fields run that variant; others the general one,
    // which reads M per volume.
    P.max_m = P.reqs[0].v->M;
    P.rdev.resize(P.reqs.size());
    P.fstore.assign(P.reqs.size(), nullptr);
    for (size_t q = 0; q < P.reqs.size(); ++q) {
        ReqHost& r = P.reqs[q];
        ReqDev& d = P.rdev[q];
        d = ReqDev{};
        d.v = vol_dev(r.v);
        r.tf_pos = P.tf_floats;
        P.tf_floats += r.total;
        for (int m = 0; m < r.v->M; ++m) {
            d.nmax[m] = (float)(r.n_tf[m] - 1);
            d.tf_off[m] = r.off[m];
        }
        d.tf_total = r.total;
        d.W = r.p.n_bins;
        d.exponent = r.p.exponent;
        d.fmin = r.p.min_importance;
        d.exp_is_one = r.p.exponent == 1.0f;
        d.clamp_mode = r.p.clamp_mode;
        d.level_shift = r.p.level_scale;
        d.scan_mode = r.p.scan_mode;
        // the other scan arithmetics' sums depend on their order: a wave per run
        d.v.split = d.v.split && d.scan_mode == DVL_SCAN_FP64;
        P.unit0.push_back(P.k1_units);
        P.n_steps += (int64_t)d.v.n_tiles * d.v.tile_steps;
        P.k1_units += request_units(d.v);
        d.vmax_exact = r.p.vmax_mode == DVL_VMAX_EXACT;
        // a workgroup of k_bin per tile when there are no more tiles than
        // bins, else per bin edge
        d.by_tile = d.v.n_tiles <= d.W;
        d.first_cell = r.out.first_cell;
        d.last_cell = r.out.last_cell;
        d.mean = r.out.mean;
        d.vmin = r.out.vmin;
        d.vmax = r.out.vmax;
        d.y = r.out.y;
        d.f_total = r.out.f_total;
        d.vmax_used = r.out.vmax_used;
        if (r.v->M != P.max_m) P.max_m = kMaxFields;
        P.max_fields = std::max(P.max_fields, r.v->M);
        P.max_req_tf = std::max(P.max_req_tf, r.total);
        P.max_tile_steps = std::max(P.max_tile_steps, d.v.tile_steps);
        P.max_tiles = std::max(P.max_tiles, d.v.n_tiles);
        P.max_w = std::max(P.max_w, d.W);
        P.max_bin_units = std::max(P.max_bin_units, d.by_tile ? d.v.n_tiles : d.W - 1);
        P.any_exact |= d.vmax_exact;
        P.far |= far_bins(d.v.n, d.v.n_tiles, d.W);
    }
    if (P.max_m > 8) P.max_m = kMaxFields;
    P.off_reqs = (P.unit0.size() * sizeof(int64_t) + 63) & ~(size_t)63;
    P.off_vmax = P.off_reqs + P.rdev.size() * sizeof(ReqDev);
    P.off_tf = (P.off_vmax + P.rdev.size() * sizeof(float) + 63) & ~(size_t)63;
    P.block_bytes = al256(P.off_tf + P.tf_floats * sizeof(float));
    return DVL_OK;
}

// Write the descriptor block into host image `h` for device address `d`:
// current tables and quantisers, max(V) of the TF modes (0 for the exact
// mode, which the first kernel raises with atomics), pointers into the block.
static dvl_status fill_block(Plan& P, char* h, char* d) {
    float* vmax_h = (float*)(h + P.off_vmax);
    float* tf_h = (float*)(h + P.off_tf);
    for (size_t q = 0; q < P.reqs.size(); ++q) {
        ReqHost& r = P.reqs[q];
        const float vm = r.p.vmax_mode == DVL_VMAX_EXACT ? 0.0f : host_vmax(r);
        if (dvl_status st = check_range(r, vm)) return st;
        vmax_h[q] = vm;
        P.rdev[q].level_shift = r.p.level_scale | (folds(r) ? 0 : kNoFold);
        memcpy(tf_h + r.tf_pos, r.alpha.data(), r.alpha.size() * sizeof(float));
        for (int m = 0; m < r.v->M; ++m) {
            P.rdev[q].s[m] = r.qs[m];
            P.rdev[q].b[m] = r.qb[m];
        }
        P.rdev[q].tf = (const float*)(d + P.off_tf) + r.tf_pos;
        P.rdev[q].vmax_dev = (float*)(d + P.off_vmax) + q;
    }
    memcpy(h, P.unit0.data(), P.unit0.size() * sizeof(int64_t));
    memcpy(h + P.off_reqs, P.rdev.data(), P.rdev.size() * sizeof(ReqDev));
    return DVL_OK;
}

// The entry-cache key of a request, if its tables fit in a byte index.
static bool key_of(const ReqHost& r, CacheKey& k) {
    k = CacheKey();
    k.M = r.v->M;
    for (int m = 0; m < r.v->M; ++m) {
        if (r.n_tf[m] > 256) return false;
        k.n_tf[m] = r.n_tf[m];
        k.s[m] = r.qs[m];
        k.b[m] = r.qb[m];
        k.lo[m] = r.lo[m];
        k.hi[m] = r.hi[m];
    }
    return true;
}

struct CacheBuild {
    dvl_volume* v;
    CacheKey key;
};

// requests [k0, k1) of group g read their volume's entry cache
static void use_cache(Plan& P, const VolReqs& g, int k0, int k1) {
    const dvl_volume* v = P.reqs[g.req0].v;
    for (int k = k0; k < k1; ++k) {
        ReqDev& d = P.rdev[g.req0 + k];
        d.entries = 1;
        for (int m = 0; m < v->M; ++m) d.v.idx[m] = v->idx_s[m];
    }
}

// whether some request of group g reads cached entries (true) or values (false)
static bool some_read(const Plan& P, const VolReqs& g, bool cached) {
    for (int k = 0; k < g.n_req; ++k)
        if ((P.rdev[g.req0 + k].entries == 1) == cached) return true;
    return false;
}

// Choose, per request, between reading the field values and reading the
// volume's TF entry cache; schedule the cache (re)builds this launch needs.
// The requests on one volume decide in turns of up to kCacheTurn (fewer with
// tables that exceed kCacheTurnFloats together): a turn reads the cache if its
// requests share one key and the cache holds it (or is built for it now).  One
// volume's cache serves one key per launch.  A whole batch deciding at once
// would let one client with windows of its own send all others to the values.
constexpr int kCacheTurn = 8, kCacheTurnFloats = 32768;
static dvl_status decide_cache(Plan& P, std::vector<CacheBuild>& builds) {
    builds.clear();
    for (const VolReqs& g : P.groups) {
        for (int k = 0; k < g.n_req; ++k) P.rdev[g.req0 + k].entries = 0;
        dvl_volume* v = P.reqs[g.req0].v;
        if (v->idx_policy == DVL_ENTRY_CACHE_NEVER) continue;
        bool serving = false;
        CacheKey served;
        for (int k0 = 0, k1; k0 < g.n_req; k0 = k1) {
            CacheKey key;
            bool agree = key_of(P.reqs[g.req0 + k0], key);
            int floats = P.reqs[g.req0 + k0].total;
            for (k1 = k0 + 1; k1 < g.n_req && k1 - k0 < kCacheTurn; ++k1) {
                floats += P.reqs[g.req0 + k1].total;
                if (floats > kCacheTurnFloats) break;
                CacheKey k2;
                agree = agree && key_of(P.reqs[g.req0 + k1], k2) && k2 == key;
            }
            if (!agree) continue;
            bool use = false;
            if (serving) {
                use = served == key;
            } else if (v->idx_valid && v->idx_key == key) {
                use = true;
            } else if (v->idx_policy == DVL_ENTRY_CACHE_ALWAYS || (v->cand_set && v->cand_key == key)) {
                if (!v->idx_s[0]) {
                    DevBuf b(v->alloc);
                    if (dvl_status st = b.alloc((size_t)v->n_pad * v->M, "TF entry cache")) return st;
                    uint8_t* base = (uint8_t*)b.release();
                    for (int m = 0; m < v->M; ++m) v->idx_s[m] = base + (size_t)m * v->n_pad;
                    v->bytes += (size_t)v->n_pad * v->M;
                }
                builds.push_back({v, key});
                use = true;
            } else {
                v->cand_key = key;
                v->cand_set = true;
            }
            if (!use) continue;
            serving = true;
            served = key;
            use_cache(P, g, k0, k1);
        }
    }
    return DVL_OK;
}

// Rebuild the scheduled caches on stream s.  Launches on other streams may
// still read a cache and later launches on any stream must see the new one;
// both are ordered by events (see dvl_volume::cache_readers), so the host
// never waits here.
// One reader event per (device, stream), shared by every volume: re-recorded
// after each launch on that stream that reads an entry cache.  A rebuild
// waits for the latest record on each other reader stream, which follows
// every earlier launch there (stream order): one record per launch instead
// of one per volume, each of which is a queue packet.  The events live until
// the process ends.
struct ReaderEvent {
    int dev;
    hipStream_t s;
    hipEvent_t ev;
};
static std::mutex g_reader_mu;
static std::vector<ReaderEvent> g_readers;

static dvl_status reader_event(hipStream_t s, bool create, hipEvent_t* out) {
    *out = nullptr;
    int dev = -1;
    DVL_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_reader_mu);
    for (const ReaderEvent& r : g_readers)
        if (r.dev == dev && r.s == s) {
            *out = r.ev;
            return DVL_OK;
        }
    if (!create) return DVL_OK;
    hipEvent_t ev = nullptr;
    DVL_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    g_readers.push_back({dev, s, ev});
    *out = ev;
    return DVL_OK;
}

static dvl_status run_cache_builds(const std::vector<CacheBuild>& builds, hipStream_t s) {
    for (const CacheBuild& cb : builds) {
        dvl_volume* v = cb.v;
        for (hipStream_t r : v->cache_readers) {
            if (r == s) continue;
            hipEvent_t ev = nullptr;
            if (dvl_status st = reader_event(r, false, &ev)) return st;
            if (ev) DVL_HIP(hipStreamWaitEvent(s, ev, 0));
        }
        v->idx_valid = false;
        for (int m = 0; m < v->M; ++m)
            if (dvl_status st = launch_build_index(v->n_pad, v->dtype, v->fields_s[m], cb.key.s[m], cb.key.b[m],
                                                   cb.key.n_tf[m], v->idx_s[m], v->n_cu, s))
                return st;
        DVL_HIP(hipEventRecord(v->cache_ready, s));
        v->cache_ready_recorded = true;
        v->cache_ready_stream = s;
        v->idx_key = cb.key;
        v->idx_valid = true;
        v->cand_set = false;
    }
    return DVL_OK;
}

// Before a launch on stream s that reads the caches of the volumes in `P`: wait
// for their latest rebuild when it ran on another stream (on s itself the
// stream order already follows it).
static dvl_status cache_wait(const Plan& P, hipStream_t s) {
    for (const VolReqs& g : P.groups) {
        if (!some_read(P, g, true)) continue;
        dvl_volume* v = P.reqs[g.req0].v;
        if (v->cache_ready_recorded && v->cache_ready_stream != s)
            DVL_HIP(hipStreamWaitEvent(s, v->cache_ready, 0));
    }
    return DVL_OK;
}

// After such a launch: s is a reader stream of those volumes (returns
// whether any request read a cache).  The caller records s's reader event.
static bool cache_add_readers(const Plan& P, hipStream_t s) {
    bool any = false;
    for (const VolReqs& g : P.groups) {
        if (!some_read(P, g, true)) continue;
        dvl_volume* v = P.reqs[g.req0].v;
        if (std::find(v->cache_readers.begin(), v->cache_readers.end(), s) == v->cache_readers.end())
            v->cache_readers.push_back(s);
        any = true;
    }
    return any;
}

// ... and records its reader event once when one did
static dvl_status cache_mark_readers(const Plan& P, hipStream_t s) {
    if (!cache_add_readers(P, s)) return DVL_OK;
    hipEvent_t ev = nullptr;
    if (dvl_status st = reader_event(s, true, &ev)) return st;
    DVL_HIP(hipEventRecord(ev, s));
    return DVL_OK;
}

// The requests that read the values of one volume, in shares of up to 8 (caches
// decided).  With one field the lookups bound the pass, and on few cells the
// launch of its own costs what the reads save: from 64 MB of values on every
// share was faster (two requests on 64 MB 75 -> 67 us, eight 147 -> 105; 8 MB
// of them +-1 %; one field, 200 MB, five requests 107 -> 115).
constexpr int kMaxShare = 8;
constexpr double kShareBytes = 64e6;
static void plan_shares(Plan& P) {
    P.shares.clear();
    for (const VolReqs& g : P.groups) {
        ReqDev* r = &P.rdev[g.req0];
        if (r->v.M < 2 || (double)r->v.n * r->v.M * elem_bytes_of(P.dtype) < kShareBytes) continue;
        for (int k = 0, e; k < g.n_req; k = e) {
            for (e = k + 1; e < g.n_req && e - k < kMaxShare && r[e].entries == r[k].entries && r[e].v.split == r[k].v.split;) ++e;
            if (e - k < 2 || r[k].entries == 1) continue;
            for (int i = k; i < e; ++i) r[i].entries = kValuesShared;
            P.shares.push_back({g.req0 + k, e - k, request_units(r[k].v)});
        }
    }
}

// What each request's projection reads (caches decided), and the kernel
// variants that have work.  A request whose bins number a quarter of its tiles
// or more rescans most of the volume; it stores f in the importance pass (4
// bytes per cell written and read again) unless reading the cached entries
// again (M bytes) costs no more and f is cheap to compute again (no pow).  Whole
// updates from entries, stored / again, 1, 4 and 8 fields: 60 M cells, W = 3670, 88 /
// 59, 154 / 103, 209 / 164 us; 20 M, W = 9764 (every tile), 73 / 58, 89 / 87, 120 / 123; 8
// M, W = 3906, 49 / 44, 62 / 61, 81 / 85.
static int plan_paths(Plan& P) {
    int paths = 0;
    plan_shares(P);
    for (size_t q = 0; q < P.rdev.size(); ++q) {
        ReqDev& d = P.rdev[q];
        const bool cached = d.entries == 1, again = cached && d.v.M <= 8 && d.exp_is_one;
        d.ws.fstore = again ? nullptr : P.fstore[q];
        d.bin_path = d.ws.fstore ? 2 : (cached ? 1 : 0);
        paths |= cached ? kPathEntries : kPathValues;
        if (d.entries == 0) paths |= kPathAlone;
        paths |= d.bin_path == 2 ? kPathBinStoredF : (d.bin_path == 1 ? kPathBinEntries : kPathBinValues);
    }
    return paths;
}

// Whether the importance pass reads the cells as non-temporal streams: when the
// volumes' cells exceed the 256 MB of the Infinity Cache, so that nothing is
// left of them for the next update (501 M cells from entries 407 -> 350 us, 150 M
// 16-bit values 240 -> 216, 50 M fp32 values 136 -> 124; updates of 320 MB 118 ->
// 113, but of 160 MB 80 -> 87).  Requests on one volume share the cells through
// that cache while they run: twice as many then (four requests on 680 MB 608 ->
// 580 us, on 460 MB 466 -> 562).
static bool streams(const Plan& P) {
    double bytes = 0.0;
    bool shared = false;
    for (const VolReqs& g : P.groups) {
        const ReqDev& d = P.rdev[g.req0];
        bytes += (double)d.v.n * d.v.M * ((some_read(P, g, true) ? 1 : 0) + (some_read(P, g, false) ? elem_bytes_of(P.dtype) : 0));
        shared |= g.n_req > 1;
    }
    return bytes > (shared ? 512.0 : 256.0) * 1048576.0;
}

// `paths`: the variants to launch (plan_paths)
static BatchLaunch batch_dev(const Plan& P, char* d, int paths) {
    BatchLaunch l;
    l.shares = P.shares;
    BatchDev& b = l.dev;
    b = BatchDev{};
    b.unit0 = (const int64_t*)d;
    b.reqs = (const ReqDev*)(d + P.off_reqs);
    b.n_reqs = (int)P.rdev.size();
    b.k1_units = P.k1_units;
    b.n_steps = P.n_steps;
    b.stream = streams(P);
    b.any_exact = P.any_exact;
    l.far = P.far;
    b.chain = 1;
    b.paths = paths;
    b.max_req_tf = P.max_req_tf;
    b.max_fields = P.max_fields;
    b.max_tile_steps = P.max_tile_steps;
    b.max_tiles = P.max_tiles;
    b.max_w = P.max_w;
    b.max_bin_units = P.max_bin_units;
    return l;
}

static int64_t fstore_cells(const dvl_volume* v, int n_bins) {
    return wants_fstore(v->n_tiles, n_bins) ? v->n_pad : 0;
}
static size_t request_ws_bytes(const dvl_volume* v, int n_bins) {
    return workspace_bytes(v->n_tiles, v->M, n_bins, fstore_cells(v, n_bins));
}
// request q's workspace at `base`; fcells: see workspace_bytes
static void carve_request(Plan& P, size_t q, void* base, int64_t fcells) {
    const ReqHost& r = P.reqs[q];
    workspace_carve(base, r.v->n_tiles, r.v->M, r.p.n_bins, fcells, &P.rdev[q].ws);
    P.fstore[q] = P.rdev[q].ws.fstore;
}

// ================================================================== executor

struct Executor {
    int n_cu = 256;
    Alloc alloc;                    // workspaces and descriptor blocks
    // The descriptor block: one device buffer, rewritten before each launch.
    // Launches on one stream run in order, so a launch rewrites the block
    // only after the previous launch's kernels have read it.  Blocks of up
    // to kPokeMaxBytes (a few requests) are written by k_poke from a host
    // image carried in kernel arguments: no staging buffer whose reuse the
    // host would have to wait for, and no event.  Larger ones (a batch of
    // many requests: tens of KB of tables) are copied from a ring of pinned
    // staging buffers, each released by an event after its copy.
    static constexpr size_t kPokeMaxBytes = (size_t)4 * kPokeWords * 4;
    // A buffer of the executor; lent: part of the volume's own allocation.
    struct Buffer {
        void* p = nullptr;
        size_t cap = 0;
        bool lent = false;
    };
    Buffer blk;
    std::vector<char> img;
    struct Staging {
        char* host = nullptr;
        size_t cap = 0;
        hipEvent_t ev = nullptr;
        bool used = false;
    };
    Staging ring[kRing];
    int next = 0;
    std::vector<Buffer> ws;         // workspace pool: one per request position
    // The end of the latest launch is marked by the reader event of its
    // stream (reader_event), recorded after every launch: it serves the
    // entry-cache ordering and this executor alike, one queue packet.
    hipStream_t last_stream = nullptr;
    bool launched = false;
    int timing = 0;                 // 0 off, 1 every phase, 2 the importance pass only
    std::vector<std::vector<hipEvent_t>> ev_pool, ev_pending;
    std::vector<int> ev_mode;       // the timing mode of each pending event set
    std::vector<hipEvent_t> ev_sel; // the events handed to the launcher (unused phases NULL)
    double phase_ms[kPhases] = {};
    int32_t timed = 0;
    size_t bytes = 0;

    ~Executor() {
        (void)hipDeviceSynchronize();
        give_back(blk);
        for (auto& r : ring) {
            if (r.host) (void)hipHostFree(r.host);
            if (r.ev) (void)hipEventDestroy(r.ev);
        }
        for (auto& w : ws) give_back(w);
        for (auto* pool : {&ev_pool, &ev_pending})
            for (auto& set : *pool)
                for (auto e : set) (void)hipEventDestroy(e);
    }

    dvl_status init() {
        int dev = 0;
        DVL_HIP(hipGetDevice(&dev));
        DVL_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
        return DVL_OK;
    }

    // the end of the latest launch (the reader event of its stream, recorded
    // after it or after later work on that stream)
    dvl_status last_event(hipEvent_t* ev) {
        *ev = nullptr;
        if (!launched) return DVL_OK;
        return reader_event(last_stream, false, ev);
    }

    // the executor's earlier launches are the only users of its buffers:
    // waiting for the latest one frees them for reuse
    dvl_status wait_idle() {
        hipEvent_t ev = nullptr;
        if (dvl_status st = last_event(&ev)) return st;
        if (ev) DVL_HIP(hipEventSynchronize(ev));
        return DVL_OK;
    }

    void give_back(Buffer& b) {
        if (!b.lent && b.p) {
            alloc.put(b.p, nullptr);
            bytes -= b.cap;
        }
        b = Buffer();
    }

    // a larger buffer in place of `b`, whose users are waited for; if the
    // allocation fails the old one stays, so smaller requests keep working
    dvl_status grow(Buffer& b, size_t cap, const char* what) {
        DevBuf d(alloc);
        if (dvl_status st = d.alloc(cap, what)) return st;
        if (b.p)
            if (dvl_status st = wait_idle()) return st;
        give_back(b);
        b.p = d.release();
        b.cap = cap;
        bytes += cap;
        return DVL_OK;
    }

    // workspace i of at least `need` bytes
    dvl_status ensure_ws(size_t i, size_t need) {
        if (ws.size() <= i) ws.resize(i + 1);
        return ws[i].cap >= need ? DVL_OK : grow(ws[i], need, "request workspace");
    }

    // a descriptor block of at least `need` device bytes (the uploaded image
    // is a prefix of them)
    dvl_status ensure_block(size_t need) {
        return blk.cap >= need ? DVL_OK : grow(blk, std::max(need * 2, (size_t)65536), "batch descriptors");
    }

    // memory for the single updates of one volume: part of its slab, or (NULL)
    // from the executor's allocator
    dvl_status reserve(char* lent_ws, size_t ws_bytes, char* lent_blk, size_t blk_bytes) {
        ws.resize(1);
        if (lent_ws) {
            ws[0] = {lent_ws, ws_bytes, true};
            blk = {lent_blk, blk_bytes, true};
            return DVL_OK;
        }
        if (dvl_status st = grow(ws[0], ws_bytes, "request workspace")) return st;
        return grow(blk, blk_bytes, "batch descriptors");
    }

    // the next pinned staging buffer, its previous copy complete, of at
    // least `need` bytes
    dvl_status take_staging(size_t need, Staging** out) {
        Staging& r = ring[next];
        next = (next + 1) % kRing;
        if (!r.ev) DVL_HIP(hipEventCreateWithFlags(&r.ev, hipEventDisableTiming));
        if (r.used) DVL_HIP(hipEventSynchronize(r.ev));
        if (r.cap < need) {
            const size_t cap = std::max(need * 2, (size_t)65536);
            char* host = nullptr;
            if (hipHostMalloc((void**)&host, cap, hipHostMallocDefault) != hipSuccess) {
                (void)hipGetLastError();
                return fail(DVL_E_NOMEM, "pinned host allocation of %zu bytes failed", cap);
            }
            if (r.host) (void)hipHostFree(r.host);
            r.host = host;
            r.cap = cap;
        }
        *out = &r;
        return DVL_OK;
    }

    // write the plan's descriptor block into blk on stream s
    dvl_status upload(Plan& P, hipStream_t s) {
        if (P.block_bytes <= kPokeMaxBytes) {
            img.resize(P.block_bytes);
            if (dvl_status st = fill_block(P, img.data(), (char*)blk.p)) return st;
            return poke((char*)blk.p, img.data(), P.block_bytes, s);
        }
        Staging* r = nullptr;
        if (dvl_status st = take_staging(P.block_bytes, &r)) return st;
        if (dvl_status st = fill_block(P, r->host, (char*)blk.p)) return st;
        DVL_HIP(hipMemcpyAsync(blk.p, r->host, P.block_bytes, hipMemcpyHostToDevice, s));
        DVL_HIP(hipEventRecord(r->ev, s));
        r->used = true;
        return DVL_OK;
    }

    dvl_status timing_events(hipEvent_t** out) {
        *out = nullptr;
        if (!timing) return DVL_OK;
        if (ev_pool.empty()) {
            std::vector<hipEvent_t> set(kPhases + 1, nullptr);
            for (auto& e : set)
                if (hipError_t err = hipEventCreate(&e)) {
                    for (auto x : set)
                        if (x) (void)hipEventDestroy(x);
                    return hip_fail(err, "hipEventCreate");
                }
            ev_pool.push_back(set);
        }
        ev_pending.push_back(ev_pool.back());
        ev_pool.pop_back();
        ev_mode.push_back(timing);
        ev_sel.assign(kPhases + 1, nullptr);
        for (int p = 0; p <= kPhases; ++p)
            if (timing == 1 || p == 1 || p == 2) ev_sel[p] = ev_pending.back()[p];
        *out = ev_sel.data();
        return DVL_OK;
    }

    dvl_status run(Plan& P, hipStream_t s) {
        for (size_t q = 0; q < P.reqs.size(); ++q) {
            const ReqHost& r = P.reqs[q];
            if (dvl_status st = ensure_ws(q, request_ws_bytes(r.v, r.p.n_bins))) return st;
            carve_request(P, q, ws[q].p, fstore_cells(r.v, r.p.n_bins));
        }
        std::vector<CacheBuild> builds;
        if (dvl_status st = decide_cache(P, builds)) return st;
        if (dvl_status st = run_cache_builds(builds, s)) return st;
        if (dvl_status st = cache_wait(P, s)) return st;
        if (dvl_status st = ensure_block(P.block_bytes)) return st;
        // a launch on another stream than the previous one first waits for it
        // (it may still read the block and the workspaces)
        if (launched && s != last_stream) {
            hipEvent_t prev = nullptr;
            if (dvl_status st = last_event(&prev)) return st;
            if (prev) DVL_HIP(hipStreamWaitEvent(s, prev, 0));
        }
        const int paths = plan_paths(P);
        if (dvl_status st = upload(P, s)) return st;
        hipEvent_t* ev = nullptr;
        if (dvl_status st = timing_events(&ev)) return st;
        if (dvl_status st = launch_batch(batch_dev(P, (char*)blk.p, paths), P.dtype, P.max_m, n_cu, s, kDescriptorLayout, ev))
            return st;
        cache_add_readers(P, s);
        hipEvent_t done = nullptr;
        if (dvl_status st = reader_event(s, true, &done)) return st;
        DVL_HIP(hipEventRecord(done, s));
        last_stream = s;
        launched = true;
        return DVL_OK;
    }

    dvl_status kernel_times(double* ms, int32_t* n) {
        for (size_t i = 0; i < ev_pending.size(); ++i) {
            auto& set = ev_pending[i];
            const bool all = ev_mode[i] == 1;
            DVL_HIP(hipEventSynchronize(set[all ? kPhases : 2]));
            for (int p = all ? 0 : 1; p < (all ? kPhases : 2); ++p) {
                float t = 0.0f;
                DVL_HIP(hipEventElapsedTime(&t, set[p], set[p + 1]));
                phase_ms[p] += t;
            }
            timed += 1;
            ev_pool.push_back(set);
        }
        ev_pending.clear();
        ev_mode.clear();
        if (ms)
            for (int p = 0; p < kPhases; ++p) ms[p] = phase_ms[p];
        if (n) *n = timed;
        for (int p = 0; p < kPhases; ++p) phase_ms[p] = 0.0;
        timed = 0;
        return DVL_OK;
    }
};

static dvl_status new_executor(const Alloc& a, Executor** out) {
    Executor* ex = new (std::nothrow) Executor();
    if (!ex) return fail(DVL_E_NOMEM, "host allocation failed");
    ex->alloc = a;
    if (dvl_status st = ex->init()) {
        delete ex;
        return st;
    }
    *out = ex;
    return DVL_OK;
}

static dvl_status requests_from(const dvl_request* reqs, int32_t n, std::vector<ReqHost>& out) {
    if (!reqs || n < 1) return fail(DVL_E_INVALID, "no requests");
    out.resize(n);
    for (int i = 0; i < n; ++i) {
        const dvl_request& r = reqs[i];
        if (dvl_status st = make_request(r.volume, r.alpha, r.n_tf, r.lo, r.hi, &r.params, &r.out, out[i])) {
            const std::string msg = g_err;
            return fail(st, "request %d: %s", i, msg.c_str());
        }
    }
    return DVL_OK;
}

}  // namespace dvl

// ================================================================== graphs

struct dvl_graph {
    Plan plan;
    Alloc alloc;                         // the first request's volume's allocator
    int n_cu = 256;
    // two descriptor blocks, each read by its own captured graphs; launches
    // alternate between them, so consecutive replays are different
    // executable graphs (one executable graph is not replayed while its
    // previous launch may still run)
    static constexpr int kSlots = 2;
    char* dev[kSlots] = {};
    int launches = 0;
    std::vector<void*> ws;               // one workspace per request
    char* host[kRing] = {};              // pinned staging of the descriptor block
    hipEvent_t ev[kRing] = {};
    bool used[kRing] = {};
    int next = 0;
    // one captured graph per set of projection paths (values, cached
    // entries, stored f) and way of reading (BatchDev::stream, shares): a replay
    // launches only the kernel variants its requests use, and both can change
    // between launches as entry caches appear.  At most kKept are kept.
    static constexpr size_t kKept = 32;
    struct Captured {
        int paths;
        int stream;
        std::vector<Share> shares;
        int slot;
        hipGraph_t graph;
        hipGraphExec_t exec;
    };
    std::vector<Captured> captured;
    void drop_captured() {
        (void)hipDeviceSynchronize();
        for (auto& c : captured) {
            if (c.exec) (void)hipGraphExecDestroy(c.exec);
            if (c.graph) (void)hipGraphDestroy(c.graph);
        }
        captured.clear();
    }
    ~dvl_graph() {
        drop_captured();
        for (char* d : dev) alloc.put(d, nullptr);
        for (void* w : ws) alloc.put(w, nullptr);
        for (int r = 0; r < kRing; ++r) {
            if (host[r]) (void)hipHostFree(host[r]);
            if (ev[r]) (void)hipEventDestroy(ev[r]);
        }
    }
};

// the statistics arrays of a volume as the placing pass writes them
static PlaceStats place_stats(const dvl_volume* v, uint2* range) {
    PlaceStats st{};
    st.n_tiles = v->n_tiles;
    st.M = v->M;
    st.tile = v->tile_stat;
    st.seg = v->seg_stat;
    st.range = range;
    return st;
}

// What a new volume sets aside for its single updates: the descriptors of any of
// them, and a workspace for plots of up to 3840 pixels (with f of every cell
// where a plot of 1920 would store it), so that the first update allocates
// nothing.  (hipMalloc and hipFree of a workspace cost the first update of a
// volume 60 to 300 us.)
constexpr int kReservedBins = 3840, kReservedStoreBins = 1920;
constexpr size_t kReservedBlock = (size_t)kMaxTfTotal * sizeof(float) + 4096;
static_assert(sizeof(ReqDev) + 1024 <= 4096, "one request's descriptors and its largest tables");
static size_t reserved_ws_bytes(const dvl_volume* v) {
    return workspace_bytes(v->n_tiles, v->M, kReservedBins, fstore_cells(v, kReservedStoreBins));
}

// Device memory a build works in before the volume's arrays are filled, and what
// it sets aside in the slab (NULL without one).
struct BuildScratch {
    char* ws = nullptr;         // reserved_ws_bytes()
    char* blk = nullptr;        // kReservedBlock
    char* small = nullptr;      // the extent, then the partial ranges per tile
    char* spare = nullptr;      // the arrays that are filled last, free until then
    size_t spare_bytes = 0;
};
static size_t build_small_bytes(const dvl_volume* v) {
    return al256(256 + extent_scratch_bytes()) + al256((size_t)v->M * v->n_tiles * sizeof(uint2));
}

// The volume's own arrays.  Through the caller's allocator each is an
// allocation; without one they are parts of one hipMalloc, with the build's
// small scratch and what is set aside for updates, and the sort may use the
// space of the arrays that are filled after it.  (hipMalloc and hipFree of more
// than 4 MB take 50 to 300 us each: loading 1.1 M cells spent 0.9 ms in twenty of
// them, 0.2 ms in its kernels.)
static dvl_status alloc_arrays(dvl_volume* v, BuildScratch* scratch) {
    const size_t eb = elem_bytes_of(v->dtype);
    const size_t tile_bytes = (size_t)v->M * v->n_tiles * sizeof(FieldStat);
    struct Array {
        void** to;
        size_t bytes;
        const char* what;     // NULL: only in the slab
    } arrays[9 + kMaxFields] = {{(void**)&v->keys_s, (size_t)v->n * 8, "keys"},
                                {(void**)&v->perm, (size_t)v->n * 4, "permutation"},
                                {(void**)&scratch->small, build_small_bytes(v), nullptr},
                                {(void**)&v->level_s, (size_t)v->n_pad, "sorted levels"},
                                {(void**)&v->lcode_s, (size_t)v->n_pad / kStepCells * 4, "level codes"},
                                {(void**)&v->tile_stat, tile_bytes, "tile statistics"},
                                {(void**)&v->seg_stat, tile_bytes * v->tile_steps * kSegsPerStep, "segment statistics"}};
    constexpr int kFilledLast = 3;     // the first array that nothing reads before it is filled
    int n_arrays = 7;
    for (int m = 0; m < v->M; ++m) arrays[n_arrays++] = {&v->fields_s[m], (size_t)v->n_pad * eb, "sorted field"};
    // side by side: kernels read the descriptors and the workspace's first arrays together
    arrays[n_arrays++] = {(void**)&scratch->blk, kReservedBlock, nullptr};
    arrays[n_arrays++] = {(void**)&scratch->ws, reserved_ws_bytes(v), nullptr};
    if (!v->alloc.custom) {
        for (int k = 0; k < n_arrays; ++k) v->slab_size += al256(arrays[k].bytes);
        if (hipMalloc((void**)&v->slab, v->slab_size) != hipSuccess) {
            v->slab = nullptr;
            (void)hipGetLastError();
            return fail(DVL_E_NOMEM, "device allocation of %zu bytes for the volume failed", v->slab_size);
        }
    }
    for (int k = 0; k < n_arrays; ++k) {
        if (v->slab) {
            *arrays[k].to = v->slab + v->slab_used;
            if (k == kFilledLast) scratch->spare = v->slab + v->slab_used;
            v->slab_used += al256(arrays[k].bytes);
            v->bytes += al256(arrays[k].bytes);
        } else if (arrays[k].what) {
            DevBuf b(v->alloc);
            if (dvl_status st = b.alloc(arrays[k].bytes, arrays[k].what)) return st;
            *arrays[k].to = b.release();
            v->bytes += arrays[k].bytes;
        }
    }
    if (v->slab) scratch->spare_bytes = v->slab_size - (size_t)(scratch->spare - v->slab);
    return DVL_OK;
}

// Fill the sorted arrays and statistics of a volume in one pass from the given
// arrays (original order, or a contiguous range of another volume's sorted
// arrays: perm NULL).  `ranges` (host-readable, a uint2 per field and one
// more) receives the data ranges and `flag`; `range_part` is device scratch of
// 8 bytes per field and tile.
static dvl_status place_volume(dvl_volume* v, const uint32_t* perm, const uint8_t* level, const void* const* fields,
                               uint2* range_part, uint2* ranges, const unsigned long long* flag, hipStream_t s) {
    PlaceArrays pa{};
    pa.n_fields = v->M;
    pa.level_src = level;
    pa.level_dst = v->level_s;
    pa.codes = v->lcode_s;
    for (int m = 0; m < v->M; ++m) {
        pa.src[m] = fields[m];
        pa.dst[m] = v->fields_s[m];
    }
    return launch_place(v->n, v->dtype, v->tile_steps, perm, pa, place_stats(v, range_part), ranges, flag, s);
}

extern "C" {

const char* dvl_last_error(void) { return g_err.c_str(); }

size_t dvl_update_workspace_bytes(int64_t n_cells, int32_t n_fields, int32_t n_bins) {
    if (n_cells < 1 || n_fields < 1 || n_bins < 1) return 0;
    const int64_t cells = (int64_t)kDefaultTileSteps * kStepCells;
    const int64_t T = (n_cells + cells - 1) / cells;
    return workspace_bytes(T, n_fields, n_bins, wants_fstore(T, n_bins) ? T * cells : 0);
}

size_t dvl_request_bytes(const dvl_volume* v, int32_t n_bins) {
    if (!v || n_bins < 1) return 0;
    // workspace + outputs (first/last, mean/min/max/y per field, two scalars)
    return request_ws_bytes(v, n_bins) + (size_t)n_bins * (8 + 16 * (size_t)v->M) + 16;
}

dvl_status dvl_build_order_ex(int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                              const uint8_t* level, int32_t M, int32_t dtype, const void* const* fields,
                              const dvl_build_options* opt, void* stream, dvl_volume** out) {
    g_err.clear();
    if (!out) return fail(DVL_E_INVALID, "out is NULL");
    *out = nullptr;
    if (n < 1 || n >= ((int64_t)1 << 32)) return fail(DVL_E_INVALID, "n_cells=%lld outside [1, 2^32)", (long long)n);
    if (M < 1 || M > kMaxFields) return fail(DVL_E_INVALID, "n_fields=%d outside [1, %d]", M, kMaxFields);
    if (dtype != DVL_F32 && dtype != DVL_F16 && dtype != DVL_BF16) return fail(DVL_E_INVALID, "unknown dtype %d", dtype);
    if (!x || !y || !z || !level || !fields) return fail(DVL_E_INVALID, "NULL input pointer");
    for (int m = 0; m < M; ++m)
        if (!fields[m]) return fail(DVL_E_INVALID, "field %d pointer is NULL", m);
    int tile_steps = kDefaultTileSteps, run_waves = 0, entry_cache = DVL_ENTRY_CACHE_AUTO;
    Alloc alloc;
    if (opt) {
        if (dvl_status st = make_alloc(opt->allocator, alloc)) return st;
        if (opt->entry_cache < DVL_ENTRY_CACHE_AUTO || opt->entry_cache > DVL_ENTRY_CACHE_NEVER)
            return fail(DVL_E_INVALID, "entry_cache %d", opt->entry_cache);
        entry_cache = opt->entry_cache;
        if (opt->tile_steps != 0 && opt->tile_steps != 8 && opt->tile_steps != 16 && opt->tile_steps != 32)
            return fail(DVL_E_INVALID, "tile_steps %d (0, 8, 16 or 32)", opt->tile_steps);
        if (opt->run_waves != 0 && (opt->run_waves < 64 || opt->run_waves > 65536))
            return fail(DVL_E_INVALID, "run_waves %d outside [64, 65536]", opt->run_waves);
        if (opt->tile_steps) tile_steps = opt->tile_steps;
        run_waves = opt->run_waves;
    }
    hipStream_t s = (hipStream_t)stream;
    dvl_volume* v = new (std::nothrow) dvl_volume();
    if (!v) return fail(DVL_E_NOMEM, "host allocation failed");
    struct Guard { dvl_volume* v; ~Guard() { if (v) dvl_destroy(v); } } guard{v};
    v->alloc = alloc;
    const Alloc& A = v->alloc;
    v->n = n;
    v->M = M;
    v->dtype = dtype;
    v->tile_steps = tile_steps;
    v->idx_policy = entry_cache;
    const int64_t tile_cells = (int64_t)tile_steps * kStepCells;
    v->n_tiles = (n + tile_cells - 1) / tile_cells;
    v->n_pad = v->n_tiles * tile_cells;
    DVL_HIP(hipGetDevice(&v->device));
    DVL_HIP(hipDeviceGetAttribute(&v->n_cu, hipDeviceAttributeMultiprocessorCount, v->device));
    {
        // runs of consecutive tiles, one per wave of the importance pass; the
        // default (32 per compute unit) is two rounds of resident waves: a
        // wave that finishes early takes another run, which evens out the
        // finishing times of the compute units
        const int64_t waves = run_waves ? run_waves : (int64_t)v->n_cu * 32;
        v->tiles_per_run = std::max<int64_t>(1, (v->n_tiles + waves - 1) / waves);
        v->n_runs = (v->n_tiles + v->tiles_per_run - 1) / v->tiles_per_run;
    }

    HostPage page;
    if (dvl_status st = page.take()) return st;
    BuildScratch scratch;
    if (dvl_status st = alloc_arrays(v, &scratch)) return st;
    DevBuf small(A), tmp(A);
    if (!scratch.small) {
        if (dvl_status st = small.alloc(build_small_bytes(v), "build scratch")) return st;
        scratch.small = (char*)small.p;
    }

    // extent, validity, grid bits
    unsigned long long* eh = (unsigned long long*)page.p;
    unsigned long long* dup = (unsigned long long*)scratch.small;
    uint2* range_part = (uint2*)(scratch.small + al256(256 + extent_scratch_bytes()));
    if (dvl_status st = launch_extent(n, x, y, z, level, eh, dup, scratch.small + 256, s)) return st;
    DVL_HIP(hipStreamSynchronize(s));
    if (eh[1]) return fail(DVL_E_RANGE, "a cell has a negative corner or a level above 20");
    int bits = 1;
    while (((unsigned long long)1 << bits) < eh[0]) ++bits;
    if (bits > 21) return fail(DVL_E_RANGE, "logical grid extent %llu exceeds 2^21 per axis", eh[0]);
    v->bits = bits;
    v->max_level = (int)eh[2];

    // keys + sort, between the volume's own arrays and a second pair of
    // buffers (the spare arrays where they are large enough, else one
    // temporary allocation), so that the sorted pair ends in the volume's
    const SortPlan sp = sort_plan(n, 3 * bits);
    const size_t key_bytes = al256((size_t)n * 8), idx_bytes = sp.packed ? 0 : al256((size_t)n * 4);
    char* second = scratch.spare;
    const size_t second_bytes = key_bytes + idx_bytes + sp.scratch_bytes;
    if (second_bytes > scratch.spare_bytes) {
        if (dvl_status st = tmp.alloc(second_bytes, "sort buffers")) return st;
        second = (char*)tmp.p;
    }
    uint64_t* keys_t = (uint64_t*)second;
    uint32_t* perm_t = sp.packed ? nullptr : (uint32_t*)(second + key_bytes);
    uint32_t* counts = (uint32_t*)(second + key_bytes + idx_bytes);
    const bool odd = sp.passes & 1;      // an odd number of passes ends in the second pair
    bool in_second = false;
    if (dvl_status st = launch_order(sp, n, x, y, z, level, bits, odd ? keys_t : v->keys_s, odd ? v->keys_s : keys_t,
                                     odd && !sp.packed ? perm_t : v->perm, odd && !sp.packed ? v->perm : perm_t, counts, s,
                                     &in_second))
        return st;
    if (in_second != odd) return fail(DVL_E_HIP, "sort passes disagree with their plan");
    if (dvl_status st = launch_dup(n, v->keys_s, dup, s)) return st;

    // sorted arrays (padded to whole tiles), statistics and data ranges
    uint2* rh = (uint2*)page.p;
    if (dvl_status st = place_volume(v, v->perm, level, fields, range_part, rh, dup, s)) return st;
    DVL_HIP(hipStreamSynchronize(s));
    page.idle = small.idle = tmp.idle = true;
    if (rh[M].x) return fail(DVL_E_OVERLAP, "two cells share a Hilbert key (overlapping AMR cells)");
    for (int m = 0; m < M; ++m) {
        if (rh[m].y == kRangeNan) return fail(DVL_E_RANGE, "field %d holds a NaN", m);
        v->dmin[m] = unkey(rh[m].x);
        v->dmax[m] = unkey(rh[m].y);
    }
    DVL_HIP(hipEventCreateWithFlags(&v->cache_ready, hipEventDisableTiming));

    // private executor of dvl_update, with room for its requests
    if (dvl_status st = new_executor(A, &v->ex)) return st;
    if (dvl_status st = v->ex->reserve(scratch.ws, reserved_ws_bytes(v), scratch.blk, kReservedBlock)) return st;
    guard.v = nullptr;
    *out = v;
    return DVL_OK;
}

dvl_status dvl_build_order(int64_t n, const int32_t* x, const int32_t* y, const int32_t* z,
                           const uint8_t* level, int32_t M, int32_t dtype, const void* const* fields,
                           void* stream, dvl_volume** out) {
    return dvl_build_order_ex(n, x, y, z, level, M, dtype, fields, nullptr, stream, out);
}

dvl_status dvl_set_field(dvl_volume* v, int32_t m, const void* values, void* stream) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    if (m < 0 || m >= v->M) return fail(DVL_E_INVALID, "field index %d outside [0, %d)", m, v->M);
    if (!values) return fail(DVL_E_INVALID, "values is NULL");
    hipStream_t s = (hipStream_t)stream;
    // The data range (and the NaN check) does not depend on the order, so it
    // is taken from the new values as given, before anything of the volume
    // changes: a rejected field leaves the volume as it was.
    HostPage page;
    if (dvl_status st = page.take()) return st;
    uint2* part = (uint2*)page.p;
    int n_part = 0;
    if (dvl_status st = launch_range(v->n, v->dtype, values, part, &n_part, s)) return st;
    DVL_HIP(hipStreamSynchronize(s));
    page.idle = true;
    uint32_t r_lo = 0xFFFFFFFFu, r_hi = 0u;
    for (int i = 0; i < n_part; ++i) {
        r_lo = std::min(r_lo, part[i].x);
        r_hi = std::max(r_hi, part[i].y);
    }
    if (r_hi == kRangeNan) return fail(DVL_E_RANGE, "field %d holds a NaN; the volume is unchanged", m);
    v->idx_valid = false;      // the cached entries describe the old values
    v->cand_set = false;
    PlaceArrays pa{};
    pa.n_fields = 1;
    pa.first_field = m;
    pa.src[0] = values;
    pa.dst[0] = v->fields_s[m];
    if (dvl_status st = launch_place(v->n, v->dtype, v->tile_steps, v->perm, pa, place_stats(v, nullptr), nullptr, nullptr, s)) {
        v->sticky = st;
        return st;
    }
    v->dmin[m] = unkey(r_lo);
    v->dmax[m] = unkey(r_hi);
    return DVL_OK;
}

dvl_status dvl_field_range(const dvl_volume* v, int32_t m, float* vmin, float* vmax) {
    g_err.clear();
    if (!v) return fail(DVL_E_INVALID, "volume is NULL");
    if (m < 0 || m >= v->M) return fail(DVL_E_INVALID, "field index %d outside [0, %d)", m, v->M);
    if (vmin) *vmin = v->dmin[m];
    if (vmax) *vmax = v->dmax[m];
    return DVL_OK;
}

dvl_status dvl_set_tf(dvl_volume* v, int32_t m, const float* alpha, int32_t n_tf, float lo, float hi) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    if (m < 0 || m >= v->M) return fail(DVL_E_INVALID, "field index %d outside [0, %d)", m, v->M);
    if (!alpha) return fail(DVL_E_INVALID, "alpha is NULL");
    if (n_tf < 2 || n_tf > kMaxTfEntries) return fail(DVL_E_INVALID, "n_tf=%d outside [2, %d]", n_tf, kMaxTfEntries);
    if (!isfinite(lo) || !isfinite(hi) || !(lo < hi)) return fail(DVL_E_INVALID, "window [%g, %g] is not finite with lo < hi", lo, hi);
    size_t total = n_tf;
    for (int q = 0; q < v->M; ++q)
        if (q != m && v->tf_set[q]) total += v->alpha[q].size();
    if (total > (size_t)kMaxTfTotal) return fail(DVL_E_INVALID, "sum of TF sizes %zu exceeds %d", total, kMaxTfTotal);
    for (int i = 0; i < n_tf; ++i)
        if (!isfinite(alpha[i])) return fail(DVL_E_INVALID, "alpha[%d] is not finite", i);
    float s, b;
    quantiser(n_tf, lo, hi, &s, &b);
    if (!isfinite(s) || !isfinite(b)) return fail(DVL_E_INVALID, "window [%g, %g] is too narrow for fp32", lo, hi);
    v->alpha[m].assign(alpha, alpha + n_tf);
    v->lo[m] = lo;
    v->hi[m] = hi;
    v->tf_set[m] = true;
    return DVL_OK;
}

dvl_status dvl_update(dvl_volume* v, const dvl_params* p, const dvl_bins* out, void* stream) {
    g_err.clear();
    std::vector<ReqHost> reqs(1);
    if (dvl_status st = volume_request(v, p, out, reqs[0])) return st;
    Plan P;
    if (dvl_status st = plan_batch(std::move(reqs), P)) return st;
    const dvl_status st = v->ex->run(P, (hipStream_t)stream);
    if (st == DVL_E_HIP) v->sticky = st;
    return st;
}

// ------------------------------------------------------------------ allocation-free update

}  // extern "C"

namespace dvl {

// The fixed device scratch of dvl_update_noalloc: the descriptor block
// (descriptors, tables) followed by the request workspace.
// Every call on a device shares its copy.  In host code `scratch` names a
// host-side stand-in, never the device memory: its device address comes
// from hipGetSymbolAddress, once per device, and only that address is used.
constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static char* g_scratch_dev[kMaxDevices] = {};

// device address of this device's scratch (the device must be current)
static dvl_status scratch_address(int dev, char** out) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (dev < 0 || dev >= kMaxDevices) return fail(DVL_E_INVALID, "device %d outside [0, %d)", dev, kMaxDevices);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_dev[dev] = (char*)p;
    }
    *out = g_scratch_dev[dev];
    return DVL_OK;
}

// A request reads the volume's entry cache here only when the cache already
// holds its key (it is never built here) and this stream is already one of the
// volume's reader streams (its reader event exists and is re-recorded below,
// creating nothing), so a later rebuild elsewhere still waits for this launch.
static void use_existing_cache(Plan& P, hipStream_t s) {
    for (const VolReqs& g : P.groups) {
        P.rdev[g.req0].entries = 0;      // one request per plan here
        dvl_volume* v = P.reqs[g.req0].v;
        if (v->idx_policy == DVL_ENTRY_CACHE_NEVER || !v->idx_valid) continue;
        CacheKey key;
        if (!key_of(P.reqs[g.req0], key) || !(key == v->idx_key)) continue;
        if (std::find(v->cache_readers.begin(), v->cache_readers.end(), s) == v->cache_readers.end()) continue;
        use_cache(P, g, 0, 1);
    }
}

// Scratch an update is charged in dvl_update_noalloc: the limit that the
// header documents (72 bytes per tile of workspace and queues, 8 per bin, the
// tables and descriptors), kept where the layout itself has become smaller,
// so that the same updates are refused.
static size_t noalloc_charge(const Plan& P) {
    const size_t T = (size_t)P.rdev[0].v.n_tiles, W = (size_t)P.rdev[0].W;
    const size_t block = 1792 + al256(P.tf_floats * sizeof(float)) + al256(24 * T);
    return block + 4 * al256(8 * T) + al256(8 * (T + 1)) + 2 * al256(4 * T) + 2 * al256(4 * W) + 256;
}

}  // namespace dvl

extern "C" {

dvl_status dvl_update_noalloc(dvl_volume* v, const dvl_params* p, const dvl_bins* out, void* stream) {
    g_err.clear();
    std::vector<ReqHost> reqs(1);
    if (dvl_status st = volume_request(v, p, out, reqs[0])) return st;
    int dev = -1;
    DVL_HIP(hipGetDevice(&dev));
    if (dev != v->device) return fail(DVL_E_INVALID, "volume lives on device %d, device %d is current", v->device, dev);
    hipStream_t s = (hipStream_t)stream;
    Plan P;
    if (dvl_status st = plan_batch(std::move(reqs), P)) return st;
    const size_t block = al256(P.block_bytes);
    const size_t need = std::max(noalloc_charge(P), block + workspace_bytes(v->n_tiles, v->M, p->n_bins, 0));
    if (need > kScratchBytes)
        return fail(DVL_E_NOMEM, "this update needs %zu bytes of scratch; dvl_update_noalloc has %zu "
                    "(use dvl_update)", need, kScratchBytes);
    char* base = nullptr;
    if (dvl_status st = scratch_address(dev, &base)) return st;
    carve_request(P, 0, base + block, 0);
    use_existing_cache(P, s);
    if (dvl_status st = cache_wait(P, s)) return st;
    const int paths = plan_paths(P);
    std::vector<char> img(P.block_bytes);
    if (dvl_status st = fill_block(P, img.data(), base)) return st;
    if (dvl_status st = poke(base, img.data(), P.block_bytes, s)) {
        v->sticky = st;
        return st;
    }
    if (dvl_status st = launch_batch(batch_dev(P, base, paths), P.dtype, P.max_m, v->n_cu, s, kDescriptorLayout, nullptr)) {
        if (st == DVL_E_HIP) v->sticky = st;
        return st;
    }
    if (P.rdev[0].entries == 1) {
        hipEvent_t ev = nullptr;   // exists: s is a reader stream of the volume
        if (dvl_status st = reader_event(s, false, &ev)) return st;
        if (ev) DVL_HIP(hipEventRecord(ev, s));
    }
    return DVL_OK;
}

size_t dvl_update_noalloc_max_bytes(void) { return kScratchBytes; }

dvl_status dvl_set_carry_wait(int32_t polls) {
    g_err.clear();
    if (polls < 0) return fail(DVL_E_INVALID, "polls %d < 0", (int)polls);
    return DVL_OK;   // every classifying workgroup computes its carry itself
}

dvl_status dvl_read_bins(const dvl_volume* v, const dvl_bins* b, int32_t W, void* stream, uint32_t* count,
                         uint32_t* first, uint32_t* last, float* mean, float* vmin, float* vmax, float* y,
                         double* f_total, float* vmax_used) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    if (!b) return fail(DVL_E_INVALID, "bins is NULL");
    if (W < 1 || W > (1 << 20)) return fail(DVL_E_INVALID, "n_bins=%d outside [1, 2^20]", W);
    hipStream_t s = (hipStream_t)stream;
    const size_t w4 = (size_t)W * 4, mw4 = (size_t)v->M * w4;
    // count needs both cell ranges, wanted by the caller or not
    struct Item {
        void* host;
        const void* dev;
        size_t bytes;
        bool want;
    } items[8] = {{first, b->first_cell, w4, first || count}, {last, b->last_cell, w4, last || count},
                  {mean, b->mean, mw4, mean != nullptr},      {vmin, b->vmin, mw4, vmin != nullptr},
                  {vmax, b->vmax, mw4, vmax != nullptr},      {y, b->y, mw4, y != nullptr},
                  {f_total, b->f_total, 8, f_total != nullptr}, {vmax_used, b->vmax_used, 4, vmax_used != nullptr}};
    PackList l{};
    size_t words = 0;
    for (const Item& it : items) {
        if (!it.want) continue;
        if (!it.dev) return fail(DVL_E_INVALID, "a bins pointer is NULL");
        l.src[l.n] = (const uint32_t*)it.dev;
        l.words[l.n] = (uint32_t)(it.bytes / 4);
        l.at[l.n] = (uint32_t)words;
        words += (it.bytes / 4 + 15) & ~(size_t)15;
        ++l.n;
    }
    if (l.n == 0) {
        DVL_HIP(hipStreamSynchronize(s));
        return DVL_OK;
    }
    const uint32_t *fh = first, *lh = last;
    std::vector<uint32_t> f_tmp, l_tmp;
    ReadStage stage;
    int dev = -1;
    DVL_HIP(hipGetDevice(&dev));
    if (words * 4 <= kReadStageBytes && dev == v->device) {
        // one kernel writes every array into pinned memory
        if (dvl_status st = stage.take()) return st;
        uint32_t* const staged = (uint32_t*)stage.p;
        if (dvl_status st = launch_pack(l, staged, s)) return st;
        DVL_HIP(hipStreamSynchronize(s));
        stage.idle = true;
        int a = 0;
        for (int k = 0; k < 8; ++k) {
            if (!items[k].want) continue;
            const uint32_t* src = staged + l.at[a++];
            if (k == 0) fh = src;
            if (k == 1) lh = src;
            if (items[k].host) memcpy(items[k].host, src, items[k].bytes);
        }
    } else {
        DVL_HIP(hipStreamSynchronize(s));
        for (int k = 0; k < 8; ++k) {
            if (!items[k].want) continue;
            void* to = items[k].host;
            if (!to) {
                std::vector<uint32_t>& tmp = k == 0 ? f_tmp : l_tmp;
                tmp.resize(W);
                to = tmp.data();
                (k == 0 ? fh : lh) = tmp.data();
            }
            DVL_HIP(hipMemcpy(to, items[k].dev, items[k].bytes, hipMemcpyDeviceToHost));
        }
    }
    if (count)
        for (int i = 0; i < W; ++i) count[i] = (fh[i] == 0xFFFFFFFFu) ? 0u : lh[i] - fh[i] + 1u;
    return DVL_OK;
}

dvl_status dvl_export_order(const dvl_volume* v, uint64_t* keys, uint32_t* perm, void* stream) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    hipStream_t s = (hipStream_t)stream;
    // the permutation, read for the keys anyway, leaves in the same pass (50 M
    // cells: 318 us apart, 221 together) if the kernel can write to it
    bool together = false;
    if (keys && perm) {
        hipPointerAttribute_t a{};
        if (hipPointerGetAttributes(&a, perm) == hipSuccess)
            together = a.type == hipMemoryTypeDevice && a.device == v->device;
        else
            (void)hipGetLastError();
    }
    if (keys)
        if (dvl_status st = launch_keys_back(v->n, v->perm, v->keys_s, keys, together ? perm : nullptr, s)) return st;
    if (perm && !together) DVL_HIP(hipMemcpyAsync(perm, v->perm, (size_t)v->n * 4, hipMemcpyDeviceToDevice, s));
    return DVL_OK;
}

dvl_status dvl_export_sorted(const dvl_volume* v, uint8_t* level, void* const* fields, void* stream) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    hipStream_t s = (hipStream_t)stream;
    if (level) DVL_HIP(hipMemcpyAsync(level, v->level_s, (size_t)v->n, hipMemcpyDeviceToDevice, s));
    if (fields) {
        const size_t eb = elem_bytes_of(v->dtype);
        for (int m = 0; m < v->M; ++m)
            if (fields[m]) DVL_HIP(hipMemcpyAsync(fields[m], v->fields_s[m], (size_t)v->n * eb, hipMemcpyDeviceToDevice, s));
    }
    return DVL_OK;
}

// ------------------------------------------------------------------ bin views, brushing, zoom

static dvl_status check_bins_of(const dvl_volume* v, const dvl_bins* b, int32_t W) {
    if (dvl_status st = check_volume(v)) return st;
    if (!b || !b->first_cell || !b->last_cell) return fail(DVL_E_INVALID, "bins is NULL or lacks first/last");
    if (W < 1 || W > (1 << 20)) return fail(DVL_E_INVALID, "n_bins=%d outside [1, 2^20]", W);
    return DVL_OK;
}

dvl_status dvl_select_bins(const dvl_volume* v, const dvl_bins* bins, int32_t W, int32_t b0, int32_t b1,
                           void* stream, uint32_t* first, uint32_t* last, uint64_t* key_lo, uint64_t* key_hi) {
    g_err.clear();
    if (dvl_status st = check_bins_of(v, bins, W)) return st;
    if (b0 < 0 || b1 < b0 || b1 >= W) return fail(DVL_E_INVALID, "bin range [%d, %d] outside [0, %d)", b0, b1, W);
    hipStream_t s = (hipStream_t)stream;
    int dev = -1;
    DVL_HIP(hipGetDevice(&dev));
    uint32_t f = 0, l = 0;
    uint64_t klo = 0, khi = 0;
    if (dev == v->device) {
        HostPage page;
        if (dvl_status st = page.take()) return st;
        uint64_t* got = (uint64_t*)page.p;
        if (dvl_status st = launch_pick(bins->first_cell, bins->last_cell, b0, b1, v->n, v->keys_s, got, s)) return st;
        DVL_HIP(hipStreamSynchronize(s));
        page.idle = true;
        f = (uint32_t)got[0];
        l = (uint32_t)(got[0] >> 32);
        klo = got[1];
        khi = got[2];
    } else {
        // another device is current: copies find their way, a kernel would not
        DVL_HIP(hipMemcpyAsync(&f, bins->first_cell + b0, 4, hipMemcpyDeviceToHost, s));
        DVL_HIP(hipMemcpyAsync(&l, bins->last_cell + b1, 4, hipMemcpyDeviceToHost, s));
        DVL_HIP(hipStreamSynchronize(s));
        if (f <= l && (int64_t)l < v->n) {
            DVL_HIP(hipMemcpyAsync(&klo, v->keys_s + f, 8, hipMemcpyDeviceToHost, s));
            DVL_HIP(hipMemcpyAsync(&khi, v->keys_s + l, 8, hipMemcpyDeviceToHost, s));
            DVL_HIP(hipStreamSynchronize(s));
        }
    }
    if (f > l || (int64_t)l >= v->n) return fail(DVL_E_STATE, "the bins do not hold a cell range of this volume");
    if (first) *first = f;
    if (last) *last = l;
    if (key_lo) *key_lo = klo;
    if (key_hi) *key_hi = khi;
    return DVL_OK;
}

dvl_status dvl_select_mask(const dvl_volume* v, const uint64_t* ranges, int32_t n_ranges, uint8_t* mask,
                           void* stream) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    if (n_ranges < 1 || n_ranges > kMaxSelectRanges)
        return fail(DVL_E_INVALID, "n_ranges=%d outside [1, %d]", n_ranges, kMaxSelectRanges);
    if (!ranges || !mask) return fail(DVL_E_INVALID, "ranges or mask is NULL");
    for (int i = 0; i < n_ranges; ++i)
        if (ranges[2 * i] > ranges[2 * i + 1]) return fail(DVL_E_INVALID, "range %d has lo > hi", i);
    return launch_select_mask(v->n, v->keys_s, v->perm, n_ranges, ranges, mask, (hipStream_t)stream);
}

dvl_status dvl_bin_histograms(const dvl_volume* v, const dvl_bins* bins, int32_t W, int32_t m, int32_t n_buckets,
                              float lo, float hi, uint32_t* counts, void* stream) {
    g_err.clear();
    if (dvl_status st = check_bins_of(v, bins, W)) return st;
    if (m < 0 || m >= v->M) return fail(DVL_E_INVALID, "field index %d outside [0, %d)", m, v->M);
    if (n_buckets < 1 || n_buckets > kMaxTfEntries)
        return fail(DVL_E_INVALID, "n_buckets=%d outside [1, %d]", n_buckets, kMaxTfEntries);
    if (!counts) return fail(DVL_E_INVALID, "counts is NULL");
    if (!isfinite(lo) || !isfinite(hi) || !(lo < hi)) return fail(DVL_E_INVALID, "window [%g, %g] is not finite with lo < hi", lo, hi);
    float qs, qb;
    quantiser(n_buckets, lo, hi, &qs, &qb);
    if (!isfinite(qs) || !isfinite(qb)) return fail(DVL_E_INVALID, "window [%g, %g] is too narrow for fp32", lo, hi);
    return launch_bin_histograms(v->dtype, v->fields_s[m], v->n, W, bins->first_cell, bins->last_cell, n_buckets, qs, qb,
                                 counts, v->n_cu, (hipStream_t)stream);
}

dvl_status dvl_rasterize(const float* y, int32_t n_lines, int32_t W, int32_t n_rows, int32_t mode, uint8_t* image,
                         void* stream) {
    g_err.clear();
    if (!y || !image) return fail(DVL_E_INVALID, "y or image is NULL");
    if (n_lines < 1 || n_lines > kMaxFields) return fail(DVL_E_INVALID, "n_lines=%d outside [1, %d]", n_lines, kMaxFields);
    if (W < 1 || W > (1 << 20)) return fail(DVL_E_INVALID, "n_bins=%d outside [1, 2^20]", W);
    if (n_rows < 1 || n_rows > 16384) return fail(DVL_E_INVALID, "n_rows=%d outside [1, 16384]", n_rows);
    if (mode != DVL_RASTER_POLYLINE && mode != DVL_RASTER_BARS) return fail(DVL_E_INVALID, "raster mode %d", mode);
    return launch_rasterize(y, W, n_rows, n_lines, mode, image, (hipStream_t)stream);
}

dvl_status dvl_zoom(const dvl_volume* v, uint32_t first, uint32_t last, const dvl_build_options* opt, void* stream,
                    dvl_volume** out) {
    g_err.clear();
    if (!out) return fail(DVL_E_INVALID, "out is NULL");
    *out = nullptr;
    if (dvl_status st = check_volume(v)) return st;
    if (first > last || (int64_t)last >= v->n)
        return fail(DVL_E_INVALID, "cell range [%u, %u] outside [0, %lld)", first, last, (long long)v->n);
    int tile_steps = kDefaultTileSteps, run_waves = 0, entry_cache = DVL_ENTRY_CACHE_AUTO;
    Alloc alloc = v->alloc;
    if (opt) {
        if (opt->allocator)
            if (dvl_status st = make_alloc(opt->allocator, alloc)) return st;
        if (opt->entry_cache < DVL_ENTRY_CACHE_AUTO || opt->entry_cache > DVL_ENTRY_CACHE_NEVER)
            return fail(DVL_E_INVALID, "entry_cache %d", opt->entry_cache);
        if (opt->tile_steps != 0 && opt->tile_steps != 8 && opt->tile_steps != 16 && opt->tile_steps != 32)
            return fail(DVL_E_INVALID, "tile_steps %d (0, 8, 16 or 32)", opt->tile_steps);
        if (opt->run_waves != 0 && (opt->run_waves < 64 || opt->run_waves > 65536))
            return fail(DVL_E_INVALID, "run_waves %d outside [64, 65536]", opt->run_waves);
        entry_cache = opt->entry_cache;
        if (opt->tile_steps) tile_steps = opt->tile_steps;
        run_waves = opt->run_waves;
    }
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = (int64_t)last - first + 1;
    const int eb = elem_bytes_of(v->dtype);
    dvl_volume* z = new (std::nothrow) dvl_volume();
    if (!z) return fail(DVL_E_NOMEM, "host allocation failed");
    struct Guard { dvl_volume* v; ~Guard() { if (v) dvl_destroy(v); } } guard{z};
    z->alloc = alloc;
    const Alloc& A = z->alloc;
    z->n = n;
    z->M = v->M;
    z->dtype = v->dtype;
    z->bits = v->bits;
    z->max_level = v->max_level;
    z->device = v->device;
    z->n_cu = v->n_cu;
    z->tile_steps = tile_steps;
    z->idx_policy = entry_cache;
    const int64_t tile_cells = (int64_t)tile_steps * kStepCells;
    z->n_tiles = (n + tile_cells - 1) / tile_cells;
    z->n_pad = z->n_tiles * tile_cells;
    {
        const int64_t waves = run_waves ? run_waves : (int64_t)z->n_cu * 32;
        z->tiles_per_run = std::max<int64_t>(1, (z->n_tiles + waves - 1) / waves);
        z->n_runs = (z->n_tiles + z->tiles_per_run - 1) / z->tiles_per_run;
    }
    HostPage page;
    if (dvl_status st = page.take()) return st;
    BuildScratch scratch;
    if (dvl_status st = alloc_arrays(z, &scratch)) return st;
    DevBuf small(A);
    if (!scratch.small) {
        if (dvl_status st = small.alloc(build_small_bytes(z), "build scratch")) return st;
        scratch.small = (char*)small.p;
    }
    uint2* range_part = (uint2*)(scratch.small + al256(256 + extent_scratch_bytes()));
    if (dvl_status st = launch_range_order(n, v->keys_s + first, z->keys_s, z->perm, s)) return st;
    const void* src[kMaxFields] = {};
    for (int m = 0; m < z->M; ++m) src[m] = (const char*)v->fields_s[m] + (size_t)first * eb;
    uint2* rh = (uint2*)page.p;
    if (dvl_status st = place_volume(z, nullptr, v->level_s + first, src, range_part, rh, nullptr, s)) return st;
    DVL_HIP(hipStreamSynchronize(s));
    page.idle = small.idle = true;
    for (int m = 0; m < z->M; ++m) {
        z->dmin[m] = unkey(rh[m].x);
        z->dmax[m] = unkey(rh[m].y);
    }
    DVL_HIP(hipEventCreateWithFlags(&z->cache_ready, hipEventDisableTiming));
    if (dvl_status st = new_executor(A, &z->ex)) return st;
    if (dvl_status st = z->ex->reserve(scratch.ws, reserved_ws_bytes(z), scratch.blk, kReservedBlock)) return st;
    guard.v = nullptr;
    *out = z;
    return DVL_OK;
}

dvl_status dvl_set_timing(dvl_volume* v, int32_t enable) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    if (enable < 0 || enable > 2) return fail(DVL_E_INVALID, "timing mode %d (0, 1 or 2)", (int)enable);
    v->ex->timing = enable;
    return DVL_OK;
}

dvl_status dvl_kernel_times(dvl_volume* v, double* ms, int32_t* n_updates) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    return v->ex->kernel_times(ms, n_updates);
}

dvl_status dvl_set_entry_cache(dvl_volume* v, int32_t policy) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    if (policy < DVL_ENTRY_CACHE_AUTO || policy > DVL_ENTRY_CACHE_NEVER)
        return fail(DVL_E_INVALID, "entry_cache %d", policy);
    v->idx_policy = policy;
    if (policy == DVL_ENTRY_CACHE_NEVER) {
        DVL_HIP(hipDeviceSynchronize());   // queued updates may still read it
        if (v->idx_s[0]) {
            v->alloc.put(v->idx_s[0], nullptr);
            for (int m = 0; m < kMaxFields; ++m) v->idx_s[m] = nullptr;
            v->bytes -= (size_t)v->n_pad * v->M;
        }
        v->idx_valid = false;
        v->cand_set = false;
    }
    return DVL_OK;
}

int32_t dvl_entry_cache_info(const dvl_volume* v, float* lo, float* hi, int32_t* n_tf) {
    if (!v || !v->idx_valid) return 0;
    for (int m = 0; m < v->M; ++m) {
        if (lo) lo[m] = v->idx_key.lo[m];
        if (hi) hi[m] = v->idx_key.hi[m];
        if (n_tf) n_tf[m] = v->idx_key.n_tf[m];
    }
    return 1;
}

int64_t dvl_num_cells(const dvl_volume* v) { return v ? v->n : 0; }
int32_t dvl_num_fields(const dvl_volume* v) { return v ? v->M : 0; }
int32_t dvl_grid_bits(const dvl_volume* v) { return v ? v->bits : 0; }
int32_t dvl_dtype(const dvl_volume* v) { return v ? v->dtype : -1; }
size_t dvl_volume_bytes(const dvl_volume* v) { return v ? v->bytes + (v->ex ? v->ex->bytes : 0) : 0; }

dvl_status dvl_level_segments(const dvl_volume* v, int64_t* n_segments, int64_t* n_mixed) {
    g_err.clear();
    if (dvl_status st = check_volume(v)) return st;
    const int64_t n_steps = v->n_pad / kStepCells;
    std::vector<uint32_t> codes((size_t)n_steps);
    DVL_HIP(hipDeviceSynchronize());
    DVL_HIP(hipMemcpy(codes.data(), v->lcode_s, (size_t)n_steps * 4, hipMemcpyDeviceToHost));
    int64_t mixed = 0;
    for (uint32_t c : codes)
        for (int k = 0; k < 4; ++k) mixed += ((c >> (8 * k)) & 0xFFu) == 0xFFu;
    if (n_segments) *n_segments = n_steps * 4;
    if (n_mixed) *n_mixed = mixed;
    return DVL_OK;
}

void dvl_destroy(dvl_volume* v) {
    if (!v) return;
    (void)hipDeviceSynchronize();
    delete v->ex;
    const Alloc& A = v->alloc;
    if (v->slab) {
        (void)hipFree(v->slab);
    } else {
        A.put(v->level_s, nullptr);
        A.put(v->lcode_s, nullptr);
        for (int m = 0; m < kMaxFields; ++m) A.put(v->fields_s[m], nullptr);
        A.put(v->keys_s, nullptr);
        A.put(v->perm, nullptr);
        A.put(v->tile_stat, nullptr);
        A.put(v->seg_stat, nullptr);
    }
    A.put(v->idx_s[0], nullptr);
    if (v->cache_ready) (void)hipEventDestroy(v->cache_ready);
    delete v;
}

// ------------------------------------------------------------------ executors and batches

dvl_status dvl_executor_create_ex(const dvl_allocator* allocator, dvl_executor** out) {
    g_err.clear();
    if (!out) return fail(DVL_E_INVALID, "out is NULL");
    *out = nullptr;
    Alloc a;
    if (dvl_status st = make_alloc(allocator, a)) return st;
    Executor* ex = nullptr;
    if (dvl_status st = new_executor(a, &ex)) return st;
    *out = reinterpret_cast<dvl_executor*>(ex);
    return DVL_OK;
}

dvl_status dvl_executor_create(dvl_executor** out) { return dvl_executor_create_ex(nullptr, out); }

void dvl_executor_destroy(dvl_executor* ex) { delete reinterpret_cast<Executor*>(ex); }

size_t dvl_executor_bytes(const dvl_executor* ex) {
    return ex ? reinterpret_cast<const Executor*>(ex)->bytes : 0;
}

dvl_status dvl_executor_set_timing(dvl_executor* ex, int32_t enable) {
    g_err.clear();
    if (!ex) return fail(DVL_E_INVALID, "executor is NULL");
    if (enable < 0 || enable > 2) return fail(DVL_E_INVALID, "timing mode %d (0, 1 or 2)", (int)enable);
    reinterpret_cast<Executor*>(ex)->timing = enable;
    return DVL_OK;
}

dvl_status dvl_executor_kernel_times(dvl_executor* ex, double* ms, int32_t* n) {
    g_err.clear();
    if (!ex) return fail(DVL_E_INVALID, "executor is NULL");
    return reinterpret_cast<Executor*>(ex)->kernel_times(ms, n);
}

dvl_status dvl_update_batch(dvl_executor* exh, const dvl_request* reqs, int32_t n_reqs, void* stream) {
    g_err.clear();
    if (!exh) return fail(DVL_E_INVALID, "executor is NULL");
    std::vector<ReqHost> rh;
    if (dvl_status st = requests_from(reqs, n_reqs, rh)) return st;
    Plan P;
    if (dvl_status st = plan_batch(std::move(rh), P)) return st;
    return reinterpret_cast<Executor*>(exh)->run(P, (hipStream_t)stream);
}

dvl_status dvl_graph_create(const dvl_request* reqs, int32_t n_reqs, dvl_graph** out) {
    g_err.clear();
    if (!out) return fail(DVL_E_INVALID, "out is NULL");
    *out = nullptr;
    std::vector<ReqHost> rh;
    if (dvl_status st = requests_from(reqs, n_reqs, rh)) return st;
    dvl_graph* g = new (std::nothrow) dvl_graph();
    if (!g) return fail(DVL_E_NOMEM, "host allocation failed");
    struct Guard { dvl_graph* g; ~Guard() { delete g; } } guard{g};
    if (dvl_status st = plan_batch(std::move(rh), g->plan)) return st;
    Plan& P = g->plan;
    g->alloc = P.reqs[0].v->alloc;
    int dev = 0;
    DVL_HIP(hipGetDevice(&dev));
    DVL_HIP(hipDeviceGetAttribute(&g->n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    for (size_t q = 0; q < P.reqs.size(); ++q) {
        DevBuf w(g->alloc);
        const ReqHost& r = P.reqs[q];
        if (dvl_status st = w.alloc(request_ws_bytes(r.v, r.p.n_bins), "request workspace")) return st;
        g->ws.push_back(w.release());
        carve_request(P, q, g->ws.back(), fstore_cells(r.v, r.p.n_bins));
    }
    for (int k = 0; k < dvl_graph::kSlots; ++k) {
        DevBuf d(g->alloc);
        if (dvl_status st = d.alloc(P.block_bytes, "graph descriptors")) return st;
        g->dev[k] = (char*)d.release();
    }
    {
        // a first descriptor image validates the tables (range checks) before anything is captured
        std::vector<char> probe(P.block_bytes);
        if (dvl_status st = fill_block(P, probe.data(), g->dev[0])) return st;
    }
    for (int r = 0; r < kRing; ++r) {
        if (hipHostMalloc((void**)&g->host[r], P.block_bytes, hipHostMallocDefault) != hipSuccess) {
            g->host[r] = nullptr;
            (void)hipGetLastError();
            return fail(DVL_E_NOMEM, "pinned host allocation failed");
        }
        DVL_HIP(hipEventCreateWithFlags(&g->ev[r], hipEventDisableTiming));
    }
    // the kernels are captured at the first launch with each set of paths;
    // the descriptors they read are refreshed before every replay
    guard.g = nullptr;
    *out = g;
    return DVL_OK;
}

// The executable graph of this path set and way of reading, captured on first use.
static dvl_status graph_exec_for(dvl_graph* g, int paths, int slot, hipGraphExec_t* out) {
    Plan& P = g->plan;
    const BatchLaunch b = batch_dev(P, g->dev[slot], paths);
    for (auto& c : g->captured)
        if (c.paths == paths && c.stream == b.dev.stream && c.shares == b.shares && c.slot == slot) {
            *out = c.exec;
            return DVL_OK;
        }
    if (g->captured.size() >= dvl_graph::kKept) g->drop_captured();
    hipStream_t cs;
    DVL_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    if (hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal)) {
        (void)hipStreamDestroy(cs);
        return hip_fail(e, "hipStreamBeginCapture");
    }
    const dvl_status cst = launch_batch(b, P.dtype, P.max_m, g->n_cu, cs, kDescriptorLayout, nullptr);
    hipGraph_t graph = nullptr;
    const hipError_t ee = hipStreamEndCapture(cs, &graph);
    (void)hipStreamDestroy(cs);
    if (cst != DVL_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return cst;
    }
    if (ee != hipSuccess) return hip_fail(ee, "hipStreamEndCapture");
    hipGraphExec_t exec = nullptr;
    if (hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0)) {
        (void)hipGraphDestroy(graph);
        return hip_fail(e, "hipGraphInstantiate");
    }
    g->captured.push_back({paths, b.dev.stream, b.shares, slot, graph, exec});
    *out = exec;
    return DVL_OK;
}

dvl_status dvl_graph_set_tf(dvl_graph* g, int32_t req, const float* alpha, const float* lo, const float* hi) {
    g_err.clear();
    if (!g) return fail(DVL_E_INVALID, "graph is NULL");
    Plan& P = g->plan;
    if (req < 0 || req >= (int)P.where.size())
        return fail(DVL_E_INVALID, "request %d outside [0, %zu)", req, P.where.size());
    ReqHost& r = P.reqs[P.where[req]];
    ReqHost tmp;
    if (dvl_status st = make_request(r.v, alpha, r.n_tf[0], lo, hi, &r.p, &r.out, tmp)) return st;
    r.alpha = std::move(tmp.alpha);
    for (int m = 0; m < r.v->M; ++m) {
        r.lo[m] = tmp.lo[m];
        r.hi[m] = tmp.hi[m];
        r.qs[m] = tmp.qs[m];
        r.qb[m] = tmp.qb[m];
    }
    return DVL_OK;
}

dvl_status dvl_graph_set_tf_all(dvl_graph* g, const float* const* alpha, const float* const* lo,
                                const float* const* hi) {
    g_err.clear();
    if (!g) return fail(DVL_E_INVALID, "graph is NULL");
    if (!alpha) return fail(DVL_E_INVALID, "alpha is NULL");
    const int n = (int)g->plan.where.size();
    for (int i = 0; i < n; ++i)
        if (dvl_status st = dvl_graph_set_tf(g, i, alpha[i], lo ? lo[i] : nullptr, hi ? hi[i] : nullptr)) {
            const std::string msg = g_err;
            return fail(st, "request %d: %s", i, msg.c_str());
        }
    return DVL_OK;
}

dvl_status dvl_graph_launch(dvl_graph* g, void* stream) {
    g_err.clear();
    if (!g) return fail(DVL_E_INVALID, "graph is NULL");
    hipStream_t s = (hipStream_t)stream;
    const int r = g->next;
    if (g->used[r]) DVL_HIP(hipEventSynchronize(g->ev[r]));
    std::vector<CacheBuild> builds;
    if (dvl_status st = decide_cache(g->plan, builds)) return st;
    if (dvl_status st = run_cache_builds(builds, s)) return st;
    if (dvl_status st = cache_wait(g->plan, s)) return st;
    const int paths = plan_paths(g->plan);
    const int slot = g->launches % dvl_graph::kSlots;
    hipGraphExec_t exec = nullptr;
    if (dvl_status st = graph_exec_for(g, paths, slot, &exec)) return st;
    if (dvl_status st = fill_block(g->plan, g->host[r], g->dev[slot])) return st;
    g->next = (r + 1) % kRing;
    DVL_HIP(hipMemcpyAsync(g->dev[slot], g->host[r], g->plan.block_bytes, hipMemcpyHostToDevice, s));
    DVL_HIP(hipEventRecord(g->ev[r], s));
    g->used[r] = true;
    DVL_HIP(hipGraphLaunch(exec, s));
    ++g->launches;
    return cache_mark_readers(g->plan, s);
}

void dvl_graph_destroy(dvl_graph* g) { delete g; }

}  // extern "C"
