// Device code of the per-update kernels that depend on the field storage
// type and field count (K0 exact max V, K1 importance and tile sums, K3b rescan,
// K4 bin statistics), their helpers, and the templated launcher.  Each pair of
// them is instantiated in a generated translation unit of its own; the other
// kernels and the overview of all are in update.hip.
#pragma once

#include "update.hpp"

#include <algorithm>
#include <atomic>
#include <climits>
#include <type_traits>

namespace dvl {

// ------------------------------------------------------------------ unit lookup

struct Unit {
    int req;                  // request
    int local;                // unit of that request
    int left;                 // units of the request from it on
};

// The request and its unit of importance-pass unit u: by one load of 64
// requests' first units at a time (a binary search is a chain of dependent
// loads).
__device__ __forceinline__ Unit find_unit(const BatchDev& b, int64_t u) {
    Unit r;
    r.req = 0;
    int64_t first = 0, end = b.k1_units;
    if (b.n_reqs > 1) {
        for (int base = 0; base < b.n_reqs; base += kWave) {
            const int i = base + lane_id();
            const uint64_t below = __ballot(i < b.n_reqs && gload<int64_t>(b.unit0, min(i, b.n_reqs - 1)) <= u);
            r.req = base + (int)__popcll(below) - 1;
            if (below != ~0ull) break;
        }
        r.req = uni(r.req);
        first = uni(gload<int64_t>(b.unit0, r.req));
        if (r.req + 1 < b.n_reqs) end = uni(gload<int64_t>(b.unit0, r.req + 1));
    }
    r.local = (int)(u - first);
    r.left = (int)(end - u);
    return r;
}

// ------------------------------------------------------------------ per-cell math

struct ImpCtx {
    float inv_vmax;
    bool scalable;   // inv_vmax times the largest level scale (2^60) is finite
    float fmin;
    float p;
    int exp_is_one;
    int clamp_mode;
    int lshift;
};

// In two steps: what the descriptor holds, read with a kernel's first loads,
// and max V, whose load hangs behind them; a kernel issues it early too and
// takes the value once its cells are on their way (read after the barrier that
// follows the tables, both cost every workgroup two cold loads in a row).
__device__ __forceinline__ ImpCtx ctx_params(const ReqDev& q) {
    ImpCtx c;
    c.fmin = uni(q.fmin);
    c.p = uni(q.exponent);
    c.exp_is_one = uni(q.exp_is_one);
    c.clamp_mode = uni(q.clamp_mode);
    c.lshift = uni(q.level_shift);
    return c;
}
__device__ __forceinline__ void ctx_vmax(ImpCtx& c, float vmax) {
    const float vm = uni(vmax);
    c.inv_vmax = vm > 0.0f ? 1.0f / vm : 0.0f;
    c.scalable = uni((int)(ldexpf(c.inv_vmax, 60) <= 3.0e38f)) != 0;
}

// TF entry: clamp(floor(fma(x, s, b)), 0, n_tf - 1); the clamp is one
// median-of-three (nmax >= 1), the floor the truncation of a value >= 0
__device__ __forceinline__ int tf_entry(float x, float s, float b, float nmax) {
    return (int)__builtin_amdgcn_fmed3f(fmaf(x, s, b), 0.0f, nmax);
}

// A request's quantisers and table offsets: in scalar registers for up to 8
// fields (a load inside a streaming loop would be the youngest in flight, and
// waiting for it would drain the prefetched steps), in the descriptor beyond.
template <int MT, bool REGS = (MT <= 8)>
struct Quant {
    float s[MT], b[MT], nmax[MT];
    int off[MT];
    __device__ __forceinline__ void load(const ReqDev& q) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            s[m] = uni(q.s[m]);
            b[m] = uni(q.b[m]);
            nmax[m] = uni(q.nmax[m]);
            off[m] = uni(q.tf_off[m]);
        }
    }
};
template <int MT>
struct Quant<MT, false> {
    const float *s, *b, *nmax;
    const int* off;
    __device__ __forceinline__ void load(const ReqDev& q) {
        s = q.s;
        b = q.b;
        nmax = q.nmax;
        off = q.tf_off;
    }
};

// Eq. 1: V = max_m alpha_m(x_m) - min_m alpha_m(x_m); `tf` is the request's block
template <int MT>
__device__ __forceinline__ float variation(const float (&x)[MT], int M, const float* __restrict__ tf,
                                           const Quant<MT>& q) {
    float amax = -INFINITY, amin = INFINITY;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if (m < M) {
            const int e = tf_entry(x[m], q.s[m], q.b[m], q.nmax[m]);
            const float al = tf[q.off[m] + e];
            amax = fmaxf(amax, al);
            amin = fminf(amin, al);
        }
    }
    return amax - amin;
}

// Eq. 3 with the minimum importance
__device__ __forceinline__ float importance_from_v(float v, uint32_t L, const ImpCtx& c) {
    const float r = v * c.inv_vmax;
    const int e = (int)(((uint32_t)c.lshift & 0xFFu) * (L & 0xFFu));   // 8 x 8 bits: a 24-bit multiply
    float f;
    if (c.clamp_mode == 0) {
        const float g = ldexpf(r, e);
        f = c.exp_is_one ? g : powf(g, c.p);
        f = fmaxf(f, c.fmin);
    } else {
        const float g = ldexpf(fmaxf(r, c.fmin), e);
        f = c.exp_is_one ? g : powf(g, c.p);
    }
    return f;
}

// Eq. 3 for P = 1 with the minimum importance on f (the paper's setting):
// the same operations as importance_from_v takes for it
__device__ __forceinline__ float importance_p1(float v, uint32_t L, const ImpCtx& c) {
    const float r = v * c.inv_vmax;
    const int e = (int)(((uint32_t)c.lshift & 0xFFu) * (L & 0xFFu));   // 8 x 8 bits: a 24-bit multiply
    return fmaxf(ldexpf(r, e), c.fmin);
}

// Field count of a volume: the variants MT = 1 .. 8 run batches whose
// volumes all have exactly MT fields (a compile-time count); MT = 16 reads it
// per volume.
template <int MT>
__device__ __forceinline__ int fields_of(int M) {
    return MT <= 8 ? MT : M;
}

// A wave's streams over one run of a volume: scalar base pointers advanced to
// the run's first cell, so every load is a scalar base plus a 32-bit lane
// offset (a run holds at most 1/64 of a volume, well below 2^32 bytes), and
// the level codes of the run's steps.
template <int MT>
struct RunView {
    const char* base[MT];
    const char* lev;
    const uint32_t* lcode;
};

// Levels of the 4 cells of a lane.  The per-step level code says for every
// 64 cells whether they share one level; lanes in such a segment take it from
// the code and point their level load at the run's first word (a cached
// line), so only segments of mixed levels fetch level bytes.
struct LaneLevels {
    uint32_t lv;   // loaded levels (meaningful for code 0xFF only)
    uint32_t lc;   // the lane's segment code
    __device__ __forceinline__ void load(const char* lev, uint32_t qd, uint32_t code) {
        lc = (code >> ((lane_id() >> 4) << 3)) & 0xFFu;
        lv = gload_at<uint32_t>(lev, lc == 0xFFu ? qd * 4u : 0u);
    }
    // the 4 levels as the bytes of one word: the loaded ones, or the code's
    // level in every byte (one select per step instead of one per cell)
    __device__ __forceinline__ uint32_t word() const {
        return lc == 0xFFu ? lv : __builtin_amdgcn_perm(0u, lc, 0u);
    }
    __device__ __forceinline__ uint32_t get(int k) const { return (word() >> (8 * k)) & 0xFFu; }
};

// values of the 4 cells of this lane in the given step
template <int MT, typename S>
struct StepData {
    static constexpr uint32_t kQuadBytes = Quad<S>::kBytes;
    Quad<S> q[MT];
    LaneLevels lv;
    __device__ static const void* source(const VolDev& v, int m) { return v.fields[m]; }
    // step: index from the run's first step; code: its level code; STREAM: a
    // volume too large for the caches (common.hpp)
    template <bool STREAM>
    __device__ __forceinline__ void load(const RunView<MT>& v, int M, int step, uint32_t code) {
        const uint32_t qd = (uint32_t)(step * kWave + lane_id());
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if (m >= M) continue;
            if constexpr (STREAM)
                q[m].stream_at(v.base[m], qd * kQuadBytes);
            else
                q[m].load_at(v.base[m], qd * kQuadBytes);
        }
        lv.load(v.lev, qd, code);
    }
};

// TF entries of the 4 cells of this lane in the given step, from the
// volume's entry cache (one byte per cell and field)
template <int MT>
struct StepIdx {
    static constexpr uint32_t kQuadBytes = 4;
    uint32_t e[MT];
    LaneLevels lv;
    __device__ static const void* source(const VolDev& v, int m) { return v.idx[m]; }
    template <bool STREAM>
    __device__ __forceinline__ void load(const RunView<MT>& v, int M, int step, uint32_t code) {
        const uint32_t qd = (uint32_t)(step * kWave + lane_id());
#pragma unroll
        for (int m = 0; m < MT; ++m)
            if (m < M) e[m] = STREAM ? gstream_at<uint32_t>(v.base[m], qd * 4u) : gload_at<uint32_t>(v.base[m], qd * 4u);
        lv.load(v.lev, qd, code);
    }
};

// The rescan's forms of both: levels loaded as they are (a quarter more bytes
// of few tiles, one dependent load less than through the level codes).
struct PlainLevels {
    uint32_t lv;
    __device__ __forceinline__ uint32_t get(int k) const { return (lv >> (8 * k)) & 0xFFu; }
};
template <int MT, typename S>
struct BinData {
    static constexpr uint32_t kQuadBytes = Quad<S>::kBytes;
    Quad<S> q[MT];
    PlainLevels lv;
    __device__ static const void* source(const VolDev& v, int m) { return v.fields[m]; }
    __device__ __forceinline__ void load(const RunView<MT>& v, int M, int step) {
        const uint32_t qd = (uint32_t)(step * kWave + lane_id());
#pragma unroll
        for (int m = 0; m < MT; ++m)
            if (m < M) q[m].load_at(v.base[m], qd * kQuadBytes);
        lv.lv = gload_at<uint32_t>(v.lev, qd * 4u);
    }
};
template <int MT>
struct BinIdx {
    static constexpr uint32_t kQuadBytes = 4;
    uint32_t e[MT];
    PlainLevels lv;
    __device__ static const void* source(const VolDev& v, int m) { return v.idx[m]; }
    __device__ __forceinline__ void load(const RunView<MT>& v, int M, int step) {
        const uint32_t qd = (uint32_t)(step * kWave + lane_id());
#pragma unroll
        for (int m = 0; m < MT; ++m)
            if (m < M) e[m] = gload_at<uint32_t>(v.base[m], qd * 4u);
        lv.lv = gload_at<uint32_t>(v.lev, qd * 4u);
    }
};

// the importance of the 4 cells of this lane, as the importance pass stored
// it (view.base[0]: the request's stored f)
template <int MT>
struct StepF {
    static constexpr uint32_t kQuadBytes = 16;
    f32x4 fv;
    __device__ static const void* source(const VolDev&, int) { return nullptr; }
    __device__ __forceinline__ void load(const RunView<MT>& v, int M, int step) {
        fv = gload_at<f32x4>(v.base[0], (uint32_t)(step * kWave + lane_id()) * kQuadBytes);
    }
};

template <int MT, typename D>
__device__ __forceinline__ RunView<MT> run_view(const VolDev& vol, int M, int64_t c_begin) {
    RunView<MT> v;
    const int64_t quad0 = c_begin >> 2;
#pragma unroll
    for (int m = 0; m < MT; ++m)
        v.base[m] = m < M ? uni(reinterpret_cast<const char*>(D::source(vol, m))) + quad0 * D::kQuadBytes : nullptr;
    v.lev = uni(reinterpret_cast<const char*>(vol.level)) + quad0 * 4;
    v.lcode = uni(vol.lcode) + (c_begin >> 8);
    return v;
}

// V of cell k of this lane, from values or from cached entries; tf: the
// request's tables in LDS (values: as uploaded; entries: table m at
// m * kIdxTable)
template <int MT, typename S>
__device__ __forceinline__ float values_v(const Quad<S> (&v)[MT], int k, int M, const float* tf, const Quant<MT>& q) {
    float xk[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) xk[m] = m < M ? v[m].get(k) : 0.0f;
    return variation<MT>(xk, M, tf, q);
}
template <int MT, typename S>
__device__ __forceinline__ float cell_v(const StepData<MT, S>& d, int k, int M, const float* tf, const Quant<MT>& q) {
    return values_v<MT, S>(d.q, k, M, tf, q);
}
template <int MT, typename S>
__device__ __forceinline__ float cell_v(const BinData<MT, S>& d, int k, int M, const float* tf, const Quant<MT>& q) {
    return values_v<MT, S>(d.q, k, M, tf, q);
}
// 4 x byte k of w (the byte offset of an entry in its table), one
// instruction through the byte operand select of the SDWA encoding
__device__ __forceinline__ uint32_t entry_x4(uint32_t w, int k) {
    uint32_t a;
    switch (k) {
    case 0:
        asm("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0"
            : "=v"(a) : "v"(w));
        break;
    case 1:
        asm("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1"
            : "=v"(a) : "v"(w));
        break;
    case 2:
        asm("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2"
            : "=v"(a) : "v"(w));
        break;
    default:
        asm("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3"
            : "=v"(a) : "v"(w));
        break;
    }
    return a;
}

typedef __attribute__((address_space(3))) const float lds_f32;

// The tables start at LDS address 0 (the kernels that take this path have no
// static LDS; their launcher checks), so an entry's LDS address is its byte
// offset in the table plus the table's compile-time offset, which lands in the
// instruction's immediate.
template <int MT>
__device__ __forceinline__ float entries_v(const uint32_t (&e)[MT], int k, int M) {
    float amax = -INFINITY, amin = INFINITY;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if (m < M) {
            const uint32_t a = entry_x4(e[m], k) + (uint32_t)(m * kIdxTable * sizeof(float));
            const float al = *reinterpret_cast<lds_f32*>((uintptr_t)a);
            amax = fmaxf(amax, al);
            amin = fminf(amin, al);
        }
    }
    return amax - amin;
}
template <int MT>
__device__ __forceinline__ float cell_v(const StepIdx<MT>& d, int k, int M, const float* tf, const Quant<MT>& q) {
    return entries_v<MT>(d.e, k, M);
}
template <int MT>
__device__ __forceinline__ float cell_v(const BinIdx<MT>& d, int k, int M, const float* tf, const Quant<MT>& q) {
    return entries_v<MT>(d.e, k, M);
}

// How many steps one loop iteration loads ahead: one 4-vector per field is
// enough to keep HBM busy; 16-bit values are half of that and cached entries
// a quarter, so two or four steps go together (tiles hold a multiple of four
// steps and are padded, so the loads of a group stay inside the volume's
// buffers).
template <typename D> struct Group { static constexpr int n = 1; };
#ifndef DVL_ENTRY_GROUP
#define DVL_ENTRY_GROUP 4
#endif
template <int MT> struct Group<StepIdx<MT>> { static constexpr int n = DVL_ENTRY_GROUP; };
#ifndef DVL_HALF_GROUP
#define DVL_HALF_GROUP 2
#endif
template <int MT> struct Group<StepData<MT, F16>> { static constexpr int n = DVL_HALF_GROUP; };
template <int MT> struct Group<StepData<MT, BF16>> { static constexpr int n = DVL_HALF_GROUP; };

// level codes of the G steps of a group (step: its first, a multiple of G),
// through vector loads (every lane the same words): they are waited for in
// order with the stream loads (a scalar load would be waited for with the
// LDS lookups, and all outstanding scalar loads at once)
template <int G>
struct StepCodes {
    uint32_t c[G];
};
template <int G>
__device__ __forceinline__ StepCodes<G> load_codes(const uint32_t* lcode, int step) {
    StepCodes<G> r;
    if constexpr (G == 4) {
        const u32x4 w = gload<u32x4>(lcode + step, 0);
        r.c[0] = w.x;
        r.c[1] = w.y;
        r.c[2] = w.z;
        r.c[3] = w.w;
    } else {
#pragma unroll
        for (int g = 0; g < G; ++g) r.c[g] = gload<uint32_t>(lcode, step + g);
    }
    return r;
}

// ------------------------------------------------------------------ tables

// n LDS floats dst[i] = value(i), i < n, by the whole workgroup of kThreads:
// each thread issues the loads of eight of its elements before it stores any,
// so a round costs one memory latency (a load-store loop waits for each load
// alone)
template <int kThreads, typename F>
__device__ __forceinline__ void stage_lds(float* dst, int n, F value) {
    const int tid = thread_x();
    for (int i0 = tid; i0 < n; i0 += 8 * kThreads) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = i0 + k * kThreads < n ? value(i0 + k * kThreads) : 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (i0 + k * kThreads < n) dst[i0 + k * kThreads] = v[k];
    }
}

// The request's tables into LDS, for the importance pass (kUpdThreads = one
// thread per entry of a kIdxTable table).  Requests that read values keep the
// block as uploaded; requests that read cached entries (tables of <= 256
// entries) place table m at m * kIdxTable floats, so that every lookup address
// is the entry times 4 plus a compile-time offset.  Two dependent rounds of
// loads in all: the tables' places, then every table at once.
template <int MT, bool IDX>
__device__ __forceinline__ void load_tables(const ReqDev& q, int M, float* tf_lds) {
    if constexpr (IDX) {
        static_assert(kUpdThreads == kIdxTable, "a thread per entry");
        const float* tf = uni(q.tf);
        const int e = thread_x();
        float v[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            v[m] = 0.0f;
            if (m < M && e <= (int)uni(q.nmax[m])) v[m] = gload<float>(tf, uni(q.tf_off[m]) + e);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
            if (m < M) tf_lds[m * kIdxTable + e] = v[m];
    } else {
        const float* tf = uni(q.tf);
        stage_lds<kUpdThreads>(tf_lds, uni(q.tf_total), [&](int i) { return gload<float>(tf, i); });
    }
}

// Floats of LDS the tables take in the importance pass and K0 (the
// partial results of the waves follow, 8-byte aligned).
template <bool IDX>
__host__ __device__ __forceinline__ int sums_lds(const BatchDev& b) {
    return IDX ? b.max_fields * kIdxTable : (b.max_req_tf + 1) & ~1;
}


// ------------------------------------------------------------------ K0

constexpr int kMaxStreamSteps = 1 << 20;    // steps of one wave's stream: its offsets stay below 2^32 bytes

// max V over nsteps steps from cell c_begin, by one wave (per lane): two groups
// of steps in flight, the first ones while `tables()` waits for the tables
// (called once, by a wave without work too)
template <int MT, typename D, bool STREAM, typename Tables>
__device__ __forceinline__ float vmax_run(const ReqDev& q, int64_t c_begin, int nsteps, const float* tf_lds,
                                          Tables tables) {
    constexpr int G = Group<D>::n;
    if (nsteps <= 0) {
        tables();
        return 0.0f;
    }
    const int lane = lane_id();
    const VolDev& vol = q.v;
    const int M = uni(fields_of<MT>(vol.M));
    const int64_t n = uni(vol.n);
    Quant<MT> qn;
    qn.load(q);
    float vmax = 0.0f;
    const RunView<MT> view = run_view<MT, D>(vol, M, c_begin);
    D A[G], B[G];
    auto load = [&](D (&d)[G], int s) {
#pragma unroll
        for (int g = 0; g < G; ++g) d[g].template load<STREAM>(view, M, min(s + g, nsteps - 1), 0u);   // levels unused
    };
    auto process = [&](const D (&d)[G], int s) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (s + g >= nsteps) break;
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = cell_v<MT>(d[g], k, M, tf_lds, qn);
            const int64_t c0 = c_begin + (int64_t)(s + g) * kStepCells;
            if (c0 + kStepCells <= n) {
                vmax = fmaxf(vmax, fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (c0 + 4 * lane + k < n) vmax = fmaxf(vmax, v[k]);
            }
        }
    };
    load(A, 0);
    load(B, G);
    tables();
    for (int s = 0; s < nsteps; s += 2 * G) {
        process(A, s);
        load(A, s + 2 * G);
        if (s + G >= nsteps) break;
        process(B, s + G);
        load(B, s + 3 * G);
    }
    return vmax;
}

// A workgroup takes b.chain consecutive units, the cells of one request among
// them as one stretch in four parts, and publishes the request's maximum with
// one atomic (atomics on one word follow each other at 12 ns: 5.2 M cells took
// 24 us with one per wave, 19 with one for each of 1024 workgroups, 13 with
// 316 workgroups).
// IDX: this instance serves the requests that read cached entries (1) or values (0)
template <int MT, typename S, int IDX>
__global__ __launch_bounds__(kUpdThreads) void k_vmax_exact(BatchDev b) {
    extern __shared__ float tf_lds[];
    float* part = tf_lds + sums_lds<IDX != 0>(b);   // a maximum per wave behind the tables
    const int wv = uni((int)(thread_x() / kWave));
    int loaded = -1;
    float vmax = 0.0f;
    auto publish = [&]() {
        const float v = wave_highest_f(vmax);
        if (lane_id() == 0) part[wv] = v;
        __syncthreads();
        if (thread_x() == 0) {
            float m = part[0];
            for (int k = 1; k < kUpdWaves; ++k) m = fmaxf(m, part[k]);
            if (m > 0.0f) atomicMax(reinterpret_cast<unsigned int*>(b.reqs[loaded].vmax_dev), __float_as_uint(m));
        }
        __syncthreads();
        vmax = 0.0f;
    };
    using D = typename std::conditional<IDX != 0, StepIdx<MT>, StepData<MT, S>>::type;
    const int64_t u1 = min((block_x() + 1) * b.chain, b.k1_units);
    for (int64_t u = block_x() * b.chain; u < u1;) {
        const Unit un = find_unit(b, u);
        const ReqDev& q = b.reqs[un.req];
        int k = (int)min(u1 - u, (int64_t)un.left);
        if ((uni(q.entries) == 1) != (IDX == 1) || !uni(q.vmax_exact)) {
            u += k;
            continue;
        }
        auto tables = [&]() {
            if (un.req == loaded) return;
            load_tables<MT, IDX != 0>(q, uni(fields_of<MT>(q.v.M)), tf_lds);
            __syncthreads();
            loaded = un.req;
        };
        if (un.req != loaded && loaded >= 0) publish();      // also: every wave is done with the tables
        const int unit_steps = uni(q.v.tile_steps) * (uni(q.v.split) ? 1 : kUpdWaves * uni(q.v.tiles_per_run));
        k = max(1, min(k, kUpdWaves * kMaxStreamSteps / unit_steps));
        const int64_t n_steps = (uni(q.v.n) + kStepCells - 1) / kStepCells;
        const int64_t s0 = (int64_t)un.local * unit_steps, s1 = min(n_steps, s0 + (int64_t)k * unit_steps);
        const int64_t steps = (s1 - s0 + kUpdWaves - 1) / kUpdWaves;     // of each wave
        const int64_t w0 = s0 + wv * steps, w1 = min(s1, w0 + steps);
        vmax = fmaxf(vmax, b.stream ? vmax_run<MT, D, true>(q, w0 * kStepCells, (int)(w1 - w0), tf_lds, tables)
                                    : vmax_run<MT, D, false>(q, w0 * kStepCells, (int)(w1 - w0), tf_lds, tables));
        u += k;
    }
    if (loaded >= 0) publish();
}

// ------------------------------------------------------------------ K1

// Error-free sum of two floats: s + e == a + b exactly (Knuth's TwoSum).
__device__ __forceinline__ void two_sum_f(float a, float b, float& s, float& e) {
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// A sum kept in the arithmetic of the scan mode: fp64 (d), compensated fp32
// (the unevaluated pair hi + lo) or plain fp32 (hi).  Used for the per-lane
// tile partials and the running sum of tile sums along a run; the mode is
// the same in every lane (a scalar branch).
struct ModeSum {
    double d;
    float hi, lo;
    __device__ void init() { d = 0.0; hi = 0.0f; lo = 0.0f; }
    __device__ double value(int mode) const {
        return mode == DVL_SCAN_FP64 ? d : (mode == DVL_SCAN_KAHAN_FP32 ? (double)hi + (double)lo : (double)hi);
    }
    __device__ void add_f(int mode, float x) {
        if (mode == DVL_SCAN_FP64) {
            d += (double)x;
        } else if (mode == DVL_SCAN_KAHAN_FP32) {
            float s, e;
            two_sum_f(hi, x, s, e);
            const float l = lo + e;
            hi = s + l;
            lo = l - (hi - s);
        } else {
            hi += x;
        }
    }
    // add another sum of the same mode
    __device__ void add(int mode, const ModeSum& o) {
        if (mode == DVL_SCAN_FP64) {
            d += o.d;
        } else if (mode == DVL_SCAN_KAHAN_FP32) {
            float s, e;
            two_sum_f(hi, o.hi, s, e);
            const float l = (lo + o.lo) + e;
            hi = s + l;
            lo = l - (hi - s);
        } else {
            hi += o.hi;
        }
    }
    // the same total in every lane (butterfly; each combine is symmetric in
    // its two operands, so every lane computes the same bits)
    __device__ void wave_total(int mode) {
        if (mode == DVL_SCAN_FP64) {
            d = wave_total_d(d);
            return;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const int src = (lane_id() ^ o) << 2;
            ModeSum x;
            x.hi = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(hi)));
            x.lo = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(lo)));
            add(mode, x);
        }
    }
};

// One wave's part of the importance pass: `nsteps` steps of one request.  Not
// split: consecutive, whole runs from run `first` (tile t_begin) on; the sum of
// every run, and per tile the non-decreasing sum of the earlier tiles of its
// run, are recorded.  Split: `part` steps of every tile from tile `first` on
// (c_begin: the wave's first cell there); the wave's sum of tile first + k goes
// to part_sums[k * kUpdWaves].  Either way the cells are one stream: the next
// steps are on their way while a tile ends and the next begins.
// f of the cells is evaluated from values or cached entries (the same bits) and
// summed over each tile per lane, 4 cells per step as (f0 + f1) + (f2 + f3) in
// fp32, accumulated over the tile's steps and then over the wave in the
// request's scan arithmetic: fp64, compensated fp32 or plain fp32.  `tables()`
// puts the tables into LDS after the first loads are on their way; it is called
// exactly once, by every wave (also one without work, nsteps <= 0).
//
// kRunPlain, kRunSplit: fp64 sums, P = 1 with the importance clamp, f not
// stored, every cell inside the volume (whole groups of steps): nothing is
// tested per step but whether its levels are mixed.  In a step without mixed
// segments a lane's four cells share a level, so the level scale is folded into
// 1 / max V (a power of two: the product has the same bits unless V / max V is
// subnormal and loses some: requests where that can show run kRunP1, see kNoFold).  75 vector and 30
// scalar instructions per step became 62 and 8, and a step's 16 lookups are in
// flight together: 432 -> 417 us for 501 M cells of 4 fields (vector units now
// busy 52 % of the time, LDS 26 %, no bank conflicts; 5 TB/s; 346 us at 6.0 TB/s
// since the cells are read as non-temporal streams).
// kRunSplitAny: fp64 sums; kRunP1, kRunPow: anything.
// kRunStream, kRunP1Stream: kRunPlain and kRunP1 over a volume too large for the
// caches (BatchDev::stream).
enum RunKind { kRunPlain, kRunStream, kRunP1, kRunP1Stream, kRunPow, kRunSplit, kRunSplitAny };
template <int MT, typename D, int KIND, typename Tables>
__device__ __forceinline__ void tile_sums_run(const ReqDev& q, int first, int t_begin, int64_t c_begin, int nsteps,
                                              int part, double* part_sums, const float* tf_lds, Tables tables) {
    constexpr int G = Group<D>::n;
    constexpr bool kSplit = KIND == kRunSplit || KIND == kRunSplitAny;
    constexpr bool kStream = KIND == kRunStream || KIND == kRunP1Stream;
    constexpr bool kPlain = KIND == kRunPlain || KIND == kRunStream || KIND == kRunSplit;
    constexpr bool kP1 = KIND == kRunP1 || KIND == kRunP1Stream;
    if (nsteps <= 0) {
        tables();
        return;
    }
    const int lane = lane_id();
    const VolDev& vol = q.v;
    const int M = uni(fields_of<MT>(vol.M));
    const int tile_steps = uni(vol.tile_steps);
    const int tile_shift = __builtin_ctz((unsigned)tile_steps), part_shift = kSplit ? __builtin_ctz((unsigned)part) : 0;
    const int tpr = uni(vol.tiles_per_run);
    const int64_t n = uni(vol.n);
    const int last_group = (nsteps - 1) / G * G;
    const RunView<MT> view = run_view<MT, D>(vol, M, c_begin);
    // where step s of the stream lies, counted from c_begin
    auto at = [&](int s) { return kSplit ? ((s >> part_shift) << tile_shift) + (s & (part - 1)) : s; };
    const float vmax = gload<float>(q.vmax_dev, 0);
    ImpCtx ctx = ctx_params(q);
    float* const fst = uni(q.ws.fstore);      // where f of every cell is kept for the projection, or NULL
    double* const lpre = uni(q.ws.local_prefix);
    double* const run_total = uni(q.ws.run_total);
    const int mode = uni(q.scan_mode);
    Quant<MT> qn;
    qn.load(q);
    // Two groups in flight, in buffers A and B that take turns: a buffer is
    // loaded again (unconditionally; past the run's end the last step is
    // reloaded) right after its group was used, so no loaded value is ever
    // moved and every wait is for the older of the two groups only.  The
    // level codes a reload needs were fetched before the buffer's previous
    // load, so they have arrived.
    D A[G], B[G];
    StepCodes<G> cA, cB;
    {
        const StepCodes<G> c0 = load_codes<G>(view.lcode, 0);
        const StepCodes<G> c1 = load_codes<G>(view.lcode, at(min(G, last_group)));
        cA = load_codes<G>(view.lcode, at(min(2 * G, last_group)));
#pragma unroll
        for (int g = 0; g < G; ++g) A[g].template load<kStream>(view, M, g, c0.c[g]);
        cB = load_codes<G>(view.lcode, at(min(3 * G, last_group)));
#pragma unroll
        for (int g = 0; g < G; ++g) B[g].template load<kStream>(view, M, at(min(G + g, nsteps - 1)), c1.c[g]);
    }
    tables();
    ctx_vmax(ctx, vmax);
    ModeSum run, tacc;
    run.init();
    tacc.init();
    double prev = 0.0;
    int t = t_begin, r = first;               // tile, and run (split: the tile again)
    int in_tile = 0, in_run = 0;
    auto end_run = [&]() {
        if (lane == 0) gstore<double>(run_total, r, fmax(prev, kPlain ? run.d : run.value(mode)));
        run.init();
        prev = 0.0;
        in_run = 0;
        ++r;
    };
    auto end_tile = [&]() {
        if constexpr (kPlain || kSplit)
            tacc.d = wave_total_d(tacc.d);
        else
            tacc.wave_total(mode);
        if constexpr (kSplit) {
            if (lane == 0) *part_sums = tacc.d;
            part_sums += kUpdWaves;
        } else {
            prev = fmax(prev, kPlain ? run.d : run.value(mode));
            if (lane == 0) gstore<double>(lpre, t, prev);
            if constexpr (kPlain)
                run.d += tacc.d;
            else
                run.add(mode, tacc);
            ++t;
            if (++in_run == tpr) end_run();
        }
        tacc.init();
        in_tile = 0;
    };

    // the steps s .. s + G - 1 of the stream, loaded into `cur`
    auto process = [&](const D (&cur)[G], int s) {
        if constexpr (kPlain) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float f[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = cell_v<MT>(cur[g], k, M, tf_lds, qn);
                if (ctx.scalable && __ballot(cur[g].lv.lc == 0xFFu) == 0ull) {
                    const float scale = ldexpf(ctx.inv_vmax, (int)(((uint32_t)ctx.lshift & 0xFFu) * cur[g].lv.lc));
#pragma unroll
                    for (int k = 0; k < 4; ++k) f[k] = fmaxf(f[k] * scale, ctx.fmin);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) f[k] = importance_p1(f[k], cur[g].lv.get(k), ctx);
                }
                tacc.d += (double)((f[0] + f[1]) + (f[2] + f[3]));
            }
            in_tile += G;
            if (in_tile == (kSplit ? part : tile_steps)) end_tile();
            return;
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (s + g >= nsteps) break;
            const int64_t c0 = c_begin + (int64_t)at(s + g) * kStepCells;
            const int64_t quad = (c0 >> 2) + lane;
            const bool full = c0 + kStepCells <= n;   // no cell past the end
            float f[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t L = cur[g].lv.get(k);
                const float v = cell_v<MT>(cur[g], k, M, tf_lds, qn);
                f[k] = kP1 ? importance_p1(v, L, ctx) : importance_from_v(v, L, ctx);
            }
            if (!full) {
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = ((quad << 2) + k < n) ? f[k] : 0.0f;
            }
            if (fst) {
                f32x4 fv;
                fv.x = f[0];
                fv.y = f[1];
                fv.z = f[2];
                fv.w = f[3];
                gstore<f32x4>(fst, quad, fv);
            }
            const float sum = (f[0] + f[1]) + (f[2] + f[3]);
            if constexpr (kSplit)
                tacc.d += (double)sum;
            else
                tacc.add_f(mode, sum);
            if (++in_tile == (kSplit ? part : tile_steps) || s + g + 1 == nsteps) end_tile();
        }
    };

    for (int s = 0; s < nsteps; s += 2 * G) {
        process(A, s);
        {
            const StepCodes<G> c2 = load_codes<G>(view.lcode, at(min(s + 4 * G, last_group)));
#pragma unroll
            for (int g = 0; g < G; ++g) A[g].template load<kStream>(view, M, at(min(s + 2 * G + g, nsteps - 1)), cA.c[g]);
            cA = c2;
        }
        if (s + G >= nsteps) break;
        process(B, s + G);
        {
            const StepCodes<G> c3 = load_codes<G>(view.lcode, at(min(s + 5 * G, last_group)));
#pragma unroll
            for (int g = 0; g < G; ++g) B[g].template load<kStream>(view, M, at(min(s + 3 * G + g, nsteps - 1)), cB.c[g]);
            cB = c3;
        }
    }
    if constexpr (!kSplit)
        if (in_run > 0) end_run();                // the volume's last run may have fewer tiles
}

// A unit is 4 runs of a request, a wave each; run r owns the tiles [r k,
// (r + 1) k).  When the volume is so small that a run is one tile and the tiles
// do not fill the chip (VolDev::split), a unit is one tile, a quarter of its
// steps each wave, and their fp64 sums are added in order (sums of fp32 values
// over a tile are exact in fp64 unless f spans more than about 2^20, so the
// split changes no bit then).  A workgroup takes b.chain consecutive units, and
// those that belong to one request as one stream: the tables are staged once
// and only the first loads are waited for.  Eight requests on two 20 M-cell
// volumes 131 -> 119 us, eight volumes of 2.3 M cells and 8 fields 60.5 -> 45
// against unit by unit, the requests in turns.
//
// A share (values, several requests on one volume; BatchDev::share): the units
// are those of one request, a workgroup takes one chain of one request, and the
// chains of the same cells for the share's requests go to workgroups b, b + 8,
// b + 16, ...: to one XCD at about the same time, which reads them from HBM
// once and finds them in its L2 for the others (who runs ahead waits for HBM,
// who follows catches up).  Past the caches (non-temporal) they would not be
// found.  Importance pass and rest of 8 requests, W = 64, request after request
// / shared / shared with non-temporal loads: 300 M fp32 cells of 4 fields 5854
// / 2780 / 4574 us, 50 M of 8 fields 1976 / 844 / 1362, 50 M bf16 cells of 4
// fields 539 / 436 / 441, 2 M fp32 cells of 8 fields 147 / 105 / 105.
constexpr int kMaxChain = 16;           // units of one stream
constexpr size_t kSumsPartBytes = (size_t)kMaxChain * kUpdWaves * sizeof(double);
template <int MT, typename S, int IDX>
__global__ __launch_bounds__(kUpdThreads) void k_tile_sums(BatchDev b) {
    extern __shared__ float tf_lds[];
    double* const part_sums = reinterpret_cast<double*>(tf_lds + sums_lds<IDX != 0>(b));   // [kMaxChain][kUpdWaves]
    const int wv = uni((int)(thread_x() / kWave));
    int loaded = -1;
    int64_t u0 = block_x() * b.chain, next = grid_dim_x() * b.chain;
    int shared = -1;                        // the workgroup's request of a share
    if (IDX == 0 && b.share > 0) {
        const int g = block_x(), row = kXcds * b.share;
        shared = g % row / kXcds;
        u0 = (int64_t)(g / row * kXcds + g % kXcds) * b.chain;
        next = b.k1_units;
    }
    for (; u0 < b.k1_units; u0 += next) {
        const int64_t u1 = min(u0 + b.chain, b.k1_units);
        for (int64_t u = u0; u < u1;) {
            const Unit un = IDX == 0 && shared >= 0 ? Unit{shared, (int)u, (int)(b.k1_units - u)} : find_unit(b, u);
            const ReqDev& q = b.reqs[un.req];
            int k = (int)min(u1 - u, (int64_t)un.left);
            if (uni(q.entries) != (shared >= 0 ? kValuesShared : IDX)) {     // another launch's
                u += k;
                continue;
            }
            const VolDev& vol = q.v;
            const int tile_steps = uni(vol.tile_steps), tpr = uni(vol.tiles_per_run), n_runs = uni(vol.n_runs);
            const int64_t n = uni(vol.n), tile_cells = (int64_t)tile_steps * kStepCells;
            const bool split = uni(vol.split) != 0;
            auto tables = [&]() {
                if (un.req == loaded) return;
                if (loaded >= 0) __syncthreads();   // the other waves are done with the previous tables
                load_tables<MT, IDX != 0>(q, uni(fields_of<MT>(vol.M)), tf_lds);
                __syncthreads();
                loaded = un.req;
            };
            using D = typename std::conditional<IDX != 0, StepIdx<MT>, StepData<MT, S>>::type;
            // P = 1 with the importance clamp: no pow
            const bool p1 = uni((int)(q.exp_is_one && q.clamp_mode == 0)) != 0;
            const bool fold = uni(q.level_shift) < kNoFold;
            const bool stored = uni(q.ws.fstore) != nullptr;
            k = max(1, min(min(k, kMaxChain), kMaxStreamSteps / (tpr * tile_steps)));
            if (!split) {
                const int r0 = un.local * kUpdWaves + wv * k, r1 = min(r0 + k, n_runs);
                const int64_t c_begin = (int64_t)r0 * tpr * tile_cells;
                const int64_t c_end = min(n, (int64_t)r1 * tpr * tile_cells);
                const int nsteps = r1 > r0 ? (int)((c_end - c_begin + kStepCells - 1) / kStepCells) : 0;
                const bool plain = p1 && fold && uni(q.scan_mode) == DVL_SCAN_FP64 && !stored &&
                                   c_begin + (int64_t)nsteps * kStepCells <= n && nsteps % tile_steps == 0;
                if (plain && b.stream)
                    tile_sums_run<MT, D, kRunStream>(q, r0, r0 * tpr, c_begin, nsteps, 0, nullptr, tf_lds, tables);
                else if (plain)
                    tile_sums_run<MT, D, kRunPlain>(q, r0, r0 * tpr, c_begin, nsteps, 0, nullptr, tf_lds, tables);
                else if (p1 && b.stream)
                    tile_sums_run<MT, D, kRunP1Stream>(q, r0, r0 * tpr, c_begin, nsteps, 0, nullptr, tf_lds, tables);
                else if (p1)
                    tile_sums_run<MT, D, kRunP1>(q, r0, r0 * tpr, c_begin, nsteps, 0, nullptr, tf_lds, tables);
                else
                    tile_sums_run<MT, D, kRunPow>(q, r0, r0 * tpr, c_begin, nsteps, 0, nullptr, tf_lds, tables);
            } else {
                // whole tiles as one stream, a ragged last tile by itself
                const int t0 = un.local, part = tile_steps / kUpdWaves;
                const int whole = min(k, (int)(n / tile_cells) - t0);
                k = max(1, whole);
                const int64_t c_begin = ((int64_t)t0 * tile_steps + wv * part) * kStepCells;
                const int64_t here = n - c_begin;       // cells left in the volume
                const int nsteps = whole > 0 ? k * part : (int)max((int64_t)0, min((int64_t)part, (here + kStepCells - 1) / kStepCells));
                if (nsteps == 0 && lane_id() == 0) part_sums[wv] = 0.0;
                if (whole > 0 && p1 && fold && !stored)
                    tile_sums_run<MT, D, kRunSplit>(q, t0, t0, c_begin, nsteps, part, part_sums + wv, tf_lds, tables);
                else
                    tile_sums_run<MT, D, kRunSplitAny>(q, t0, t0, c_begin, nsteps, part, part_sums + wv, tf_lds, tables);
                __syncthreads();
                if ((int)thread_x() < k) {
                    const double* p = part_sums + thread_x() * kUpdWaves;
                    double sum = p[0];
                    for (int w = 1; w < kUpdWaves; ++w) sum += p[w];
                    gstore<double>(q.ws.local_prefix, t0 + thread_x(), 0.0);
                    gstore<double>(q.ws.run_total, t0 + thread_x(), fmax(0.0, sum));
                }
                __syncthreads();
            }
            u += k;
        }
    }
}

// ------------------------------------------------------------------ K3

constexpr int kBinThreads = 256;  // one workgroup of four waves per rescanned (request, tile)

// The in-step prefix of one 256-cell step, per lane (4 cells): the wave's
// exclusive prefix before the lane (Bex), the lane's own partial sums p1..p3
// and the inclusive prefix B through the lane (running maximum: never
// decreasing).
struct StepPrefix {
    f32x4 ex_p;   // Bex, p1, p2, p3
    float B;
};

// LDS of the staged prefixes of one tile: [steps][64] (Bex, p1, p2, p3).
// B is not stored: B of a lane is Bex of the next lane, and B of the last
// lane (the step total) is kept in the Bex slot of lane 0, whose Bex is 0 by
// definition.  16 bytes per lane and step.
struct Stage {
    f32x4* ex_p;
    __device__ void put(int s, float B, float p1, float p2, float p3) {
        f32x4 v;
        v.x = wave_shr1(B, readlane(B, kWave - 1));
        v.y = p1;
        v.z = p2;
        v.w = p3;
        ex_p[s * kWave + lane_id()] = v;
    }
    __device__ StepPrefix get(int s) const {
        StepPrefix p;
        p.ex_p = ex_p[s * kWave + lane_id()];
        p.B = __int_as_float(
            __builtin_amdgcn_ds_bpermute(((lane_id() + 1) & (kWave - 1)) << 2, __float_as_int(p.ex_p.x)));
        if (lane_id() == 0) p.ex_p.x = 0.0f;
        return p;
    }
};

constexpr int kBinWaves = kBinThreads / kWave;
constexpr int kMaxTileSteps = 32;
constexpr size_t kStageBytesPerStep = (size_t)kWave * sizeof(f32x4);

// Phase 1 of the rescan, for the steps s = w, w + kBinWaves, ... of tile t
// taken by wave w: f of every cell again (from values, cached entries or the
// stored f, bit for bit as in K1; 1 when the total importance is 0) and the
// step's monotone prefix, into LDS.  A wave's loads go out in groups of kAhead
// steps, all four of a 16-step tile's wave at once (values of four or more
// 4-byte fields: two, which keeps six waves a SIMD); `tables()` waits for the request's tables, whose loads
// went out before them.
// POW: the importance needs powf or the other clamp; its steps go one after
// another in a rolled loop (six copies of four powf were 20 KB of code, run
// cold by every workgroup).
// One branch a step for the two special cases (total importance 0, cells past
// the end): a test per cell kept each cell's lookups in a block of their own,
// waited for one after another.
template <int MT, typename D, bool POW, typename Tables>
__device__ __forceinline__ void rescan_stage(const ReqDev& q, int t, float vmax, double degenerate_d,
                                             const float* tf_lds, Stage stage, Tables tables) {
    const int lane = lane_id();
    const int w = uni((int)(thread_x() / kWave));
    const VolDev& vol = q.v;
    const int M = uni(fields_of<MT>(vol.M));
    const int64_t n = uni(vol.n);
    const int tile_steps = uni(vol.tile_steps);
    const int64_t tbase = (int64_t)t * tile_steps * kStepCells;
    const int here = (int)min((int64_t)tile_steps * kStepCells, n - tbase);    // cells of the tile
    const int nsteps = (here + kStepCells - 1) / kStepCells;
    constexpr bool kStored = std::is_same<D, StepF<MT>>::value;
    RunView<MT> view = run_view<MT, D>(vol, kStored ? 0 : M, tbase);
    if constexpr (kStored) view.base[0] = reinterpret_cast<const char*>(uni(q.ws.fstore)) + tbase * 4;
    ImpCtx c;
    Quant<MT> qn;
    if constexpr (!kStored) {
        c = ctx_params(q);
        qn.load(q);
    }
    bool degenerate = false;
    auto process = [&](const D& cur, int s) {
        float f[4];
        if (degenerate) {
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = 1.0f;
        } else if constexpr (kStored) {
            f[0] = cur.fv.x;
            f[1] = cur.fv.y;
            f[2] = cur.fv.z;
            f[3] = cur.fv.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = cell_v<MT>(cur, k, M, tf_lds, qn);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                f[k] = POW ? importance_from_v(f[k], cur.lv.get(k), c) : importance_p1(f[k], cur.lv.get(k), c);
        }
        if ((s + 1) * kStepCells > here) {
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = s * kStepCells + 4 * lane + k < here ? f[k] : 0.0f;
        }
        // monotone in-tile prefix: lane-serial over 4 cells, wave sum scan,
        // running max to undo rounding steps back
        const float p1 = f[0], p2 = p1 + f[1], p3 = p2 + f[2], tl = p3 + f[3];
        stage.put(s, wave_incl_max(wave_incl_sum(tl)), p1, p2, p3);
    };
    constexpr int kAhead = POW ? 1 : (MT * D::kQuadBytes >= 64 ? 2 : 4);
    const int cnt = nsteps > w ? (nsteps - w + kBinWaves - 1) / kBinWaves : 0;
    bool first = true;
#pragma unroll 1
    for (int k0 = 0; k0 < cnt || first; k0 += kAhead) {
        D buf[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (k0 + k < cnt) buf[k].load(view, M, w + (k0 + k) * kBinWaves);
        if (first) {
            tables();
            degenerate = uni((int)(degenerate_d != 0.0)) != 0;
            if constexpr (!kStored) ctx_vmax(c, vmax);
            first = false;
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (k0 + k < cnt) process(buf[k], w + (k0 + k) * kBinWaves);
    }
}

// Phase 2, by every wave: the cells' pixel intervals and bins from the staged
// prefixes.  Along the sorted order the first and the last bin of a cell
// never decrease, every bin has a cell, and the next cell starts in the bin
// where this one ends or in the one after.  So each cell settles alone, from
// its own bins [blo, bhi], the last bin `prev_hi` of the cell before it and
// the first bin `next_lo` of the cell after it, which bins start with it,
// (prev_hi, bhi], and which end with it, [blo, next_lo): no walk from bin to
// bin.  (One wave walking the open bin through the steps, three wave
// reductions per bin, made the kernel take 36 us for the 64 tiles of a 64^3 grid
// plotted 1024 wide, 60 us for 50 M cells from values and 34 us for the 1900
// tiles of 501 M cells at W = 1920; settled like this 16, 45 and 33 us, most of it
// the loads before, which now leave 8.4, 29 and 16 us: see k_bin.)  Bins inside the
// tile are written as outputs; the tile's first bin
// (Bh) and last bin (O) go to its head and tail records,
// merged across tiles by K4.
struct TileBins {
    int Bh, O;              // bins of the tile's first and last cell
    bool one;               // the whole tile in one bin
    // the outputs, and this tile's tail first and head last (descriptor fields
    // in registers: behind a store they would be loaded again)
    uint32_t *first_cell, *last_cell, *tail_first, *head_last;
};

__device__ __forceinline__ void bin_start(const TileBins& tb, int b, uint32_t cell) {
    gstore<uint32_t>(b == tb.O ? tb.tail_first : tb.first_cell + b, 0, cell);
}
__device__ __forceinline__ void bin_end(const TileBins& tb, int b, uint32_t cell) {
    gstore<uint32_t>(b == tb.Bh ? tb.head_last : tb.last_cell + b, 0, cell);
}
__device__ __forceinline__ void bin_starts(const TileBins& tb, int from, int to, uint32_t cell) {
    for (int b = from; b <= to; ++b) bin_start(tb, b, cell);
}
__device__ __forceinline__ void bin_ends(const TileBins& tb, int from, int before, uint32_t cell) {
    for (int b = from; b < before; ++b) bin_end(tb, b, cell);
}

// FAR: more bins than kFarBins of one lane's cells are written by the wave
// (see far_bins).
constexpr int kFarBins = 64;

template <bool FAR>
__device__ __forceinline__ void rescan_bins(const ReqDev& q, int64_t t, float X0, float X1, float scale_f,
                                            const Stage stage) {
    const int lane = lane_id();
    const int w = uni((int)(thread_x() / kWave));
    const int64_t T = uni(q.v.n_tiles);
    const int64_t n = uni(q.v.n);
    const int W1 = uni(q.W) - 1;
    const int tile_steps = uni(q.v.tile_steps);
    TileBins tb;
    tb.first_cell = uni(q.first_cell);
    tb.last_cell = uni(q.last_cell);
    uint32_t* const rec_first = uni(q.ws.rec_first) + t;
    uint32_t* const rec_last = uni(q.ws.rec_last) + t;
    tb.tail_first = rec_first + T;
    tb.head_last = rec_last;
    int32_t* const head_bin = uni(q.ws.head_bin) + t;
    int32_t* const tail_bin = uni(q.ws.tail_bin) + t;
    const int64_t tile_cells = (int64_t)tile_steps * kStepCells;
    const int64_t tbase = t * tile_cells;
    const int64_t tend = min(tbase + tile_cells, n);
    const uint32_t last_valid = (uint32_t)(tend - 1);
    const int nsteps = (int)((tend - tbase + kStepCells - 1) / kStepCells);

    // Every step at once (lane s: step s; lanes past the last step repeat
    // it): its running base (the fp32 sum of the earlier steps' totals, in
    // step order), the first bin of its first cell and the last bin of its
    // last cell.
    const int ls = min(lane, nsteps - 1);
    const float total = stage.ex_p[ls * kWave].x;         // the step total (lane 0's Bex slot): B of lane 63
    float run_v = 0.0f;
    for (int k = 0; k < nsteps - 1; ++k) {
        const float st_k = readlane(total, k);
        run_v = k < ls ? run_v + st_k : run_v;
    }
    int key0_v, key_end_v;
    {
        const int64_t c0 = tbase + (int64_t)ls * kStepCells;
        const float B0 = stage.ex_p[ls * kWave + 1].x;    // B of lane 0: Bex of lane 1
        const float x_first = fminf(fmaf(run_v + fminf(0.0f, B0), scale_f, X0), X1);
        key0_v = max(0, min((int)floorf(x_first), W1));
        // the step's last valid cell: cell kl of lane ll
        const int r = (int)(min(c0 + kStepCells, n) - 1 - c0), ll = r >> 2, kl = r & 3;
        const f32x4 e = stage.ex_p[ls * kWave + ll];
        const float Bex = ll == 0 ? 0.0f : e.x;
        const float B = ll == kWave - 1 ? total : stage.ex_p[ls * kWave + ll + 1].x;
        const float p = kl == 0 ? 0.0f : (kl == 1 ? e.y : (kl == 2 ? e.z : e.w));
        const float x3 = fminf(fmaf(run_v + fminf(Bex + p, B), scale_f, X0), X1);
        const float x4 = (uint32_t)(c0 + r) == last_valid ? X1 : fminf(fmaf(run_v + B, scale_f, X0), X1);
        const int lo3 = max(0, min((int)floorf(x3), W1));
        key_end_v = max(lo3, min((int)ceilf(x4) - 1, W1));
    }
    tb.Bh = readlane(key0_v, 0);
    tb.O = readlane(key_end_v, nsteps - 1);
    tb.one = tb.Bh == tb.O;
    // last bin of the cell before the step, first bin of the cell after it
    // (the tile's own first and last bin stand in at its ends: those bins are
    // its records)
    const int before_v = shfl_i(key_end_v, max(lane - 1, 0)), after_v = shfl_i(key0_v, min(lane + 1, kWave - 1));
    const int prev_v = lane == 0 ? tb.Bh : before_v, next_v = lane >= nsteps - 1 ? tb.O : after_v;

    if (w == 0) {
        if (lane == 0) {
            gstore<int32_t>(head_bin, 0, tb.Bh);
            gstore<int32_t>(tail_bin, 0, tb.O);
            gstore<uint32_t>(rec_first, 0, (uint32_t)tbase);
            gstore<uint32_t>(rec_last, tb.one ? 0 : T, last_valid);
        }
        // steps inside one bin, a lane each
        if (!tb.one && lane < nsteps && key0_v == key_end_v) {
            const int64_t c0 = tbase + (int64_t)lane * kStepCells;
            bin_starts(tb, prev_v + 1, key_end_v, (uint32_t)c0);
            bin_ends(tb, key0_v, next_v, (uint32_t)(min(c0 + kStepCells, n) - 1));
        }
    }
    if (tb.one) return;

    // steps holding a bin edge, a wave each
    for (int s = w; s < nsteps; s += kBinWaves) {
        const int key0 = readlane(key0_v, s), key_end = readlane(key_end_v, s);
        if (key0 == key_end) continue;
        const int64_t c0 = tbase + (int64_t)s * kStepCells;
        const float run = readlane(run_v, s);
        // read in uniform control flow: under a lane's own branch the compiler
        // may compute the source register for that lane alone
        const int step_prev = readlane(prev_v, s), step_next = readlane(next_v, s);
        const int64_t quad = (c0 >> 2) + lane;
        const StepPrefix pr = stage.get(s);
        const float Bex = pr.ex_p.x, p1 = pr.ex_p.y, p2 = pr.ex_p.z, p3 = pr.ex_p.w, B = pr.B;
        float xs[5];
        xs[0] = fminf(fmaf(run + fminf(Bex, B), scale_f, X0), X1);
        xs[1] = fminf(fmaf(run + fminf(Bex + p1, B), scale_f, X0), X1);
        xs[2] = fminf(fmaf(run + fminf(Bex + p2, B), scale_f, X0), X1);
        xs[3] = fminf(fmaf(run + fminf(Bex + p3, B), scale_f, X0), X1);
        xs[4] = fminf(fmaf(run + B, scale_f, X0), X1);
        // pixel bins of each cell: [floor(x1), ceil(x2) - 1], clamped
        int blo[4], bhi[4];
        bool last[4];                     // the tile's last cell
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            last[k] = (uint32_t)((quad << 2) + k) == last_valid;
            const float en = last[k] ? X1 : xs[k + 1];
            blo[k] = max(0, min((int)floorf(xs[k]), W1));
            bhi[k] = max(blo[k], min((int)ceilf(en) - 1, W1));
        }
        int prev_hi = shfl_i(bhi[3], max(lane - 1, 0)), next_lo = shfl_i(blo[0], min(lane + 1, kWave - 1));
        prev_hi = lane == 0 ? step_prev : prev_hi;
        next_lo = lane == kWave - 1 ? step_next : next_lo;
        bool far = false;
        if (FAR && key_end - key0 > kFarBins) {     // such lanes one after another
            far = bhi[3] - prev_hi > kFarBins;
            for (uint64_t m = __ballot(far); m; m &= m - 1) {
                const int l = __builtin_ctzll(m);
                int from = readlane(prev_hi, l);
#pragma unroll 1
                for (int k = 0; k < 4; ++k) {
                    const uint32_t g = (uint32_t)(c0 + 4 * l + k);
                    if (g > last_valid) break;
                    const int lo = readlane(k < 2 ? (k == 0 ? blo[0] : blo[1]) : (k == 2 ? blo[2] : blo[3]), l);
                    const int hi = readlane(k < 2 ? (k == 0 ? bhi[0] : bhi[1]) : (k == 2 ? bhi[2] : bhi[3]), l);
                    const int next = readlane(k < 2 ? (k == 0 ? blo[1] : blo[2]) : (k == 2 ? blo[3] : next_lo), l);
                    const int end = g == last_valid ? tb.O : next;
                    for (int b = from + 1 + lane; b <= hi; b += kWave) bin_start(tb, b, g);
                    for (int b = lo + lane; b < end; b += kWave) bin_end(tb, b, g);
                    from = hi;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t g = (uint32_t)((quad << 2) + k);
            if (g <= last_valid && !far) {
                bin_starts(tb, (k == 0 ? prev_hi : bhi[k - 1]) + 1, bhi[k], g);
                bin_ends(tb, blo[k], last[k] ? tb.O : (k == 3 ? next_lo : blo[k + 1]), g);
            }
        }
    }
}

// The first and last bin of a tile's pixel interval.
__device__ __forceinline__ int bin_of(float x, int W1) { return max(0, min((int)floorf(x), W1)); }

// K3b: the tiles that hold a bin edge, one workgroup each (grid: x, request
// y).  With more tiles than bins a workgroup takes a bin edge and its tile,
// unless an earlier edge of the same tile has it (EdgeRec::tile < 0); else it
// takes a tile.  Its waves stage the prefixes of the tile's steps in LDS
// together (phase 1; the loads of all waves in flight), then settle the bins
// of the steps that hold an edge (phase 2).  Bound by latency on a large
// volume (a chain of kernel arguments, descriptor, edge and cells), by the
// arithmetic of phase 1 when most tiles are rescanned.  From cached entries:
// 64^3 cells W 1024 13.6 -> 8.4 us, 11.8 M cells 21 -> 16.2, 501 M 22.4 -> 19.2,
// eight requests on two 20 M-cell volumes 102 -> 78 us, eight volumes of 8
// fields 48 -> 42; 16-bit values 33 -> 26: three waves a tile found their tile
// through the per-bin bounds, and tests per cell held the lookups apart.
// IDX: this instance serves the requests whose projection reads values (0),
// cached entries (1) or the f the importance pass stored (2).  LDS: the
// request's tables (as in the importance pass; none for stored f), then the
// staged prefixes.
template <int MT, typename S, int IDX, bool FAR>
__global__ __launch_bounds__(kBinThreads) void k_bin(BatchDev bd) {
    extern __shared__ f32x4 bin_lds[];
    const ReqDev& q = bd.reqs[block_y()];
    if (uni(q.bin_path) != IDX) return;
    const int W1 = uni(q.W) - 1;
    const double* const scal = uni(q.ws.scal);
    const double degenerate_d = gload<double>(scal, 1), scale_d = gload<double>(scal, 2);
    float vmax = 0.0f;
    if constexpr (IDX != 2) vmax = gload<float>(q.vmax_dev, 0);
    int t = block_x();
    float X0, X1;
    if (uni(q.by_tile)) {
        if (t >= uni(q.v.n_tiles)) return;
        X0 = uni(gload<float>(q.ws.x0, t));
        X1 = uni(gload<float>(q.ws.x0, t + 1));
        if (bin_of(X0, W1) == bin_of(X1, W1)) return;
    } else {
        if (t >= W1) return;
        const u32x4 e = gload<u32x4>(q.ws.edge, t + 1);   // edge t + 1
        t = uni((int)e.x);
        if (t < 0) return;
        X0 = uni(__uint_as_float(e.y));
        X1 = uni(__uint_as_float(e.z));
    }
    float* tf_lds = reinterpret_cast<float*>(bin_lds);
    Stage stage;
    stage.ex_p = IDX == 2 ? bin_lds : bin_lds + ((IDX == 1 ? bd.max_fields * kIdxTable : bd.max_req_tf) + 3) / 4;
    static_assert(kBinThreads == kUpdThreads, "load_tables");
    if constexpr (IDX != 2) load_tables<MT, IDX == 1>(q, uni(fields_of<MT>(q.v.M)), tf_lds);
    auto tables = [&]() {
        if constexpr (IDX != 2) __syncthreads();
    };
    const bool pow = uni((int)!(q.exp_is_one && q.clamp_mode == 0)) != 0;
    using D = typename std::conditional<IDX == 1, BinIdx<MT>, BinData<MT, S>>::type;
    if constexpr (IDX == 2)
        rescan_stage<MT, StepF<MT>, false>(q, t, vmax, degenerate_d, tf_lds, stage, tables);
    else if (pow)
        rescan_stage<MT, D, true>(q, t, vmax, degenerate_d, tf_lds, stage, tables);
    else
        rescan_stage<MT, D, false>(q, t, vmax, degenerate_d, tf_lds, stage, tables);
    __syncthreads();
    rescan_bins<FAR>(q, t, X0, X1, uni((float)scale_d), stage);
}

// ------------------------------------------------------------------ K4

// Lanes of a wave's classes: lane l serves field l % P, P the power of two not
// below the field count (a function of M alone, so that the sums of a volume
// associate alike in every variant).
__host__ __device__ constexpr int stat_classes(int M) { return M <= 1 ? 1 : (M <= 2 ? 2 : (M <= 4 ? 4 : (M <= 8 ? 8 : 16))); }

// v combined over the lanes of each class, in every lane: rotations inside the
// rows of 16, then across the rows
template <int P, int N, typename Op>
__device__ __forceinline__ void class_reduce(uint32_t (&v)[N], Op op) {
    auto with = [&](auto move) {
        uint32_t o[N];
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = move(v[i]);
        op(v, o);
    };
    if constexpr (P <= 1) with([](uint32_t x) { return dpp_move<0x121, 0xF>(x, x); });    // row_ror:1
    if constexpr (P <= 2) with([](uint32_t x) { return dpp_move<0x122, 0xF>(x, x); });
    if constexpr (P <= 4) with([](uint32_t x) { return dpp_move<0x124, 0xF>(x, x); });
    if constexpr (P <= 8) with([](uint32_t x) { return dpp_move<0x128, 0xF>(x, x); });
    const int l = lane_id();
    with([l](uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_bpermute((l ^ 16) << 2, (int)x); });
    with([l](uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_bpermute((l ^ 32) << 2, (int)x); });
}

// Field statistics of the sorted cells [first, last], by one wave, field l % P
// by lane l (`field`: its values; `act`: the volume has it): the stored values
// of the partial 64-cell segments at the two ends, the statistics of the whole
// segments next to them and of the whole tiles in between (a segment or tile is
// whole when the range holds all of its cells below n).  A stretch's statistics
// lie field after field, so a load covers 64 / P neighbouring stretches in one
// piece and every lane sums one field.  (A field after another, 64 lanes each,
// left three lanes of four idle on dense bins and reduced every field over the
// whole wave, some 2700 instructions a bin of 8 fields: eight volumes of 8
// fields, W 2048, 39 us against 21; eight requests on two 20 M-cell volumes 29
// against 22; 64^3 cells 5.7 against 4.6; 501 M, W 1920, 13.3 against 12.2.)
// Bound by the latency of cold loads, above all their address translation, on
// few or large bins.  All loads of a round are issued before the first is used.  Sums are fp64; every lane
// ends with its class's result.
template <int P, typename S>
__device__ __forceinline__ FieldStat bin_range_stats(const VolDev& j, int M, bool act, const char* field,
                                                     uint32_t first, uint32_t last) {
    constexpr int L = kWave / P;                      // lanes of a class
    constexpr int KQ = L >= 32 ? 1 : 32 / L;          // 4-cell vectors of the two end segments per lane
    constexpr int KS = P < 4 ? 2 : 4;                 // stretches of each kind per lane and round
    const int lane = lane_id(), li = lane / P, m = lane % P;
    const int64_t n = uni(j.n);
    const int shift = __builtin_ctz((unsigned)uni(j.tile_steps)) + 2;     // segments per tile: a power of two
    const int64_t f = first, l = last;
    auto whole = [&](int64_t sg) { return f <= sg * kSegCells && l >= min(n, sg * kSegCells + kSegCells) - 1; };
    const int64_t sf = f / kSegCells, sl = l / kSegCells;
    const bool wf = whole(sf), wl = whole(sl) || sl == sf;
    // whole segments [a, b]; whole tiles [ta, tb] among them; the segments
    // outside whole tiles: [a, a + n0) and [s2, s2 + n1)
    const int a = (int)(wf ? sf : sf + 1), b = (int)(whole(sl) ? sl : sl - 1);
    int ta = 1, tb = 0, s2 = 0, n0 = 0, n1 = 0;
    if (a <= b) {
        ta = (a + (1 << shift) - 1) >> shift;
        tb = ((b + 1) >> shift) - 1;
        if (ta <= tb) {
            n0 = (ta << shift) - a;
            s2 = (tb + 1) << shift;
            n1 = b + 1 - s2;
        } else {
            n0 = b + 1 - a;             // less than two tiles
        }
    }
    const int ns = n0 + n1, nt = tb - ta + 1;
    const FieldStat* const tile_stat = uni(j.tile_stat) + m;
    const FieldStat* const seg_stat = uni(j.seg_stat) + m;
    auto segment = [&](int i) { return i < n0 ? a + i : s2 + (i - n0); };
    auto stat = [](const FieldStat* p, int64_t i) {
        return __builtin_bit_cast(FieldStat, gload<u32x4>(p + i, 0));
    };
    FieldStat r{0.0, INFINITY, -INFINITY};
    auto add = [&](double sum, float mn, float mx) {
        r.sum += sum;
        r.mn = fminf(r.mn, mn);
        r.mx = fmaxf(r.mx, mx);
    };
    Quad<S> qd[KQ];
    uint32_t c[KQ];
    bool need[KQ];
    FieldStat ss[KS], ts[KS];
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
        const int e = li + k * L;                     // vectors 0-15: the first segment's, 16-31: the last's
        c[k] = (uint32_t)(e < 16 ? sf : sl) * kSegCells + 4 * (e & 15);
        need[k] = act && e < 32 && !(e < 16 ? wf : wl) && c[k] + 3 >= first && c[k] <= last;
        if (need[k]) qd[k].load(field, c[k] >> 2);
    }
    int i0 = 0;
    for (; i0 == 0 || i0 < ns; i0 += KS * L) {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int i = i0 + li + k * L;
            if (act && i < ns) ss[k] = stat(seg_stat, (int64_t)segment(i) * M);
            if (act && i < nt) ts[k] = stat(tile_stat, (int64_t)(ta + i) * M);
        }
        if (i0 == 0) {
#pragma unroll
            for (int k = 0; k < KQ; ++k) {
                if (!need[k]) continue;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const bool in = c[k] + x - first <= last - first;
                    const float v = qd[k].get(x);
                    add(in ? (double)v : 0.0, in ? v : INFINITY, in ? v : -INFINITY);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int i = i0 + li + k * L;
            if (act && i < ns) add(ss[k].sum, ss[k].mn, ss[k].mx);
            if (act && i < nt) add(ts[k].sum, ts[k].mn, ts[k].mx);
        }
    }
    // the tiles of a long range: twice as many in flight
    for (; i0 < nt; i0 += 2 * KS * L) {
        FieldStat t2[2 * KS];
#pragma unroll
        for (int k = 0; k < 2 * KS; ++k)
            if (act && i0 + li + k * L < nt) t2[k] = stat(tile_stat, (int64_t)(ta + i0 + li + k * L) * M);
#pragma unroll
        for (int k = 0; k < 2 * KS; ++k)
            if (act && i0 + li + k * L < nt) add(t2[k].sum, t2[k].mn, t2[k].mx);
    }
    uint32_t w[4];
    {
        const u32x4 u = __builtin_bit_cast(u32x4, r);
        w[0] = u.x;
        w[1] = u.y;
        w[2] = u.z;
        w[3] = u.w;
    }
    class_reduce<P>(w, [](uint32_t (&x)[4], const uint32_t (&o)[4]) {
        auto d = [](const uint32_t (&y)[4]) { return __longlong_as_double(((uint64_t)y[1] << 32) | y[0]); };
        const uint64_t sum = (uint64_t)__double_as_longlong(d(x) + d(o));
        x[0] = (uint32_t)sum;
        x[1] = (uint32_t)(sum >> 32);
        x[2] = __float_as_uint(fminf(__uint_as_float(x[2]), __uint_as_float(o[2])));
        x[3] = __float_as_uint(fmaxf(__uint_as_float(x[3]), __uint_as_float(o[3])));
    });
    u32x4 u;
    u.x = w[0];
    u.y = w[1];
    u.z = w[2];
    u.w = w[3];
    return __builtin_bit_cast(FieldStat, u);
}

// K4: one wave per (request, bin).  The bin's cell range: written by the
// rescan when the bin starts and ends inside one rescanned tile; else the
// smallest first and largest last cell over the records of the tiles it
// touches (a tile inside one bin is that bin's record whole, a rescanned
// tile holds records of its first and last bin).  Then the statistics of the
// range and the height of the mean.
template <int MT, typename S>
__global__ __launch_bounds__(kUpdThreads) void k_bin_stats(BatchDev bd) {
    const int lane = lane_id();
    const ReqDev& q = bd.reqs[block_y()];
    const VolDev& j = q.v;
    const int b = uni(block_x() * kUpdWaves + (int)(thread_x() / kWave));
    if (b >= uni(q.W)) return;   // the whole wave
    const int M = uni(fields_of<MT>(j.M));
    if (b == 0 && lane == 0) {
        gstore<double>(q.f_total, 0, gload<double>(q.ws.scal, 0));
        gstore<float>(q.vmax_used, 0, gload<float>(q.vmax_dev, 0));
    }
    // the lane's field: its values, quantiser and table (P divides the wave, so
    // lanes below M serve the field of their number)
    const int mine = min(lane % stat_classes(M), M - 1);
    const char* const field = reinterpret_cast<const char*>(gload<uint64_t>(j.fields, mine));
    const float qs = gload<float>(q.s, mine), qb = gload<float>(q.b, mine), qn = gload<float>(q.nmax, mine);
    const int qo = gload<int32_t>(q.tf_off, mine);
    const int64_t T = uni(j.n_tiles);
    const int32_t* hb = q.ws.head_bin;
    const int32_t* tb = q.ws.tail_bin;
    // tiles touching bin b: t0 = first with tail >= b, t1 = last with head <= b
    // (K3a wrote both per bin; t0 is its candidate ta or the next tile)
    const int64_t t1 = uni(gload<int32_t>(q.ws.bin_t1, b));
    const int64_t ta = uni(gload<int32_t>(q.ws.bin_ta, b));
    // then one round of loads: the candidate's tail bin, the last tile's head
    // and tail bins, the bin's own outputs (written by the rescan when the
    // bin starts and ends inside one tile) and, per lane, the head and tail
    // bins and both records of the tiles [ta, t1].  When t0 = ta + 1, tile
    // ta's bins are all below b and it adds nothing.
    const int ea = gload<int32_t>(tb, ta);
    const int h1 = gload<int32_t>(hb, t1), e1 = gload<int32_t>(tb, t1);
    const uint32_t in_first = gload<uint32_t>(q.first_cell, b), in_last = gload<uint32_t>(q.last_cell, b);
    uint32_t first = 0xFFFFFFFFu, last = 0u;
    for (int64_t t = ta + lane; t <= t1; t += kWave) {
        const int h = gload<int32_t>(hb, t), e = gload<int32_t>(tb, t);
        const uint32_t f0 = gload<uint32_t>(q.ws.rec_first, t), l0 = gload<uint32_t>(q.ws.rec_last, t);
        const uint32_t f1 = gload<uint32_t>(q.ws.rec_first, T + t), l1 = gload<uint32_t>(q.ws.rec_last, T + t);
        if (h == b) {
            first = min(first, f0);
            last = max(last, l0);
        } else if (e == b) {
            first = min(first, f1);
            last = max(last, l1);
        }
    }
    const int64_t t0 = (ea >= b || ta + 1 >= T) ? ta : ta + 1;
    const bool inside = t0 == t1 && h1 < b && b < e1;
    if (inside) {
        first = in_first;
        last = in_last;
    } else {
        first = wave_lowest_u(first);
        last = wave_highest_u(last);
    }
    // no cell (cannot happen with a positive total width); a range outside
    // the volume is treated the same way, so no statistic reads past it
    if (first == 0xFFFFFFFFu || first > last || (int64_t)last >= uni(j.n)) {
        if (lane == 0) {
            gstore<uint32_t>(q.first_cell, b, 0xFFFFFFFFu);
            gstore<uint32_t>(q.last_cell, b, 0xFFFFFFFEu);
        }
        if (lane < M) {
            const int64_t o = (int64_t)lane * q.W + b;
            gstore<float>(q.mean, o, 0.0f);
            gstore<float>(q.vmin, o, INFINITY);
            gstore<float>(q.vmax, o, -INFINITY);
            gstore<float>(q.y, o, 0.0f);
        }
        return;
    }
    if (lane == 0 && !inside) {
        gstore<uint32_t>(q.first_cell, b, first);
        gstore<uint32_t>(q.last_cell, b, last);
    }
    first = uni(first);
    last = uni(last);
    auto stats = [&](auto classes) {
        constexpr int P = decltype(classes)::value;
        return bin_range_stats<P, S>(j, M, lane % P < M, field, first, last);
    };
    FieldStat r;
    if constexpr (MT <= 8) {
        r = stats(std::integral_constant<int, stat_classes(MT)>{});
    } else {
        switch (stat_classes(M)) {
            case 1: r = stats(std::integral_constant<int, 1>{}); break;
            case 2: r = stats(std::integral_constant<int, 2>{}); break;
            case 4: r = stats(std::integral_constant<int, 4>{}); break;
            case 8: r = stats(std::integral_constant<int, 8>{}); break;
            default: r = stats(std::integral_constant<int, 16>{}); break;
        }
    }
    if (lane < M) {
        const float mean = (float)(r.sum / (double)(last - first + 1u));
        const int e = tf_entry(mean, qs, qb, qn);
        const int64_t o = (int64_t)lane * q.W + b;
        gstore<float>(q.mean, o, mean);
        gstore<float>(q.vmin, o, r.mn);
        gstore<float>(q.vmax, o, r.mx);
        gstore<float>(q.y, o, gload<float>(q.tf, qo + e));
    }
}

// ------------------------------------------------------------------ launcher

// launchers of the kernels that do not depend on the storage type (update.hip)
dvl_status launch_carry_classify(const BatchDev& b, bool far, hipStream_t s);

// The cached-entry importance kernels address their tables from LDS address
// 0 (the start of the dynamic LDS array): they must hold no static LDS.
template <void (*Kernel)(BatchDev)>
static dvl_status check_no_static_lds(const char* name) {
    static int checked = 0;   // one flag per kernel instance
    if (checked == 1) return DVL_OK;
    hipFuncAttributes fa;
    DVL_HIP(hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(Kernel)));
    if (fa.sharedSizeBytes != 0) {
        set_error("%s holds %zu bytes of static LDS; its table addressing needs none", name, (size_t)fa.sharedSizeBytes);
        return DVL_E_HIP;
    }
    checked = 1;
    return DVL_OK;
}

// Grid of the importance pass.  Units of several requests go in equal chains to
// as many workgroups as fit the chip at once.  One large request: as many workgroups as fit when that splits them evenly (or
// there are no more); a workgroup that finishes its unit takes the next one
// with its tables in LDS, 5 % faster for 501 M cells from cached entries than a
// second round starting cold.  Else 8 workgroups per compute unit, whose later
// rounds the hardware hands to whichever compute unit frees a slot (a fixed
// uneven split, 2048 units over 1280 resident workgroups of the value path, was
// 3 % slower).  A share: chains so long that the workgroups of all its
// requests fit the chip at once.  The occupancy is queried once per kernel and LDS size; any grid
// gives the same results.
template <void (*Kernel)(BatchDev)>
static dvl_status launch_sums(const BatchDev& b, size_t lds, int n_cu, hipStream_t s) {
    static std::atomic<uint64_t> cache{0};   // (lds << 8) | blocks per compute unit, 0: none
    uint64_t c = cache.load(std::memory_order_relaxed);
    int nb = (c >> 8) == (uint64_t)lds && c != 0 ? (int)(c & 0xFF) : 0;
    if (nb == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(Kernel), kUpdThreads,
                                                         lds) != hipSuccess || nb < 1) {
            (void)hipGetLastError();
            nb = 8;
        }
        nb = std::min(nb, 255);
        cache.store(((uint64_t)lds << 8) | (uint64_t)nb, std::memory_order_relaxed);
    }
    const int64_t resident = (int64_t)n_cu * nb, units = b.k1_units;
    BatchDev d = b;
    int64_t grid = units;
    if (b.share > 0) {
        const int64_t row = (int64_t)kXcds * b.share, slots = std::max<int64_t>(1, resident / row) * kXcds;
        d.chain = (units + slots - 1) / slots;
        const int64_t chains = (units + d.chain - 1) / d.chain;
        grid = (chains + kXcds - 1) / kXcds * row;
    } else if (units > resident) {
        if (b.n_reqs > 1) {
            d.chain = (units + resident - 1) / resident;
            grid = (units + d.chain - 1) / d.chain;
        } else {
            grid = units % resident == 0 ? resident : std::min<int64_t>(units, (int64_t)n_cu * 8);
        }
    }
    hipLaunchKernelGGL(Kernel, dim3((unsigned)std::max<int64_t>(1, grid)), dim3(kUpdThreads), lds, s, d);
    DVL_HIP(hipGetLastError());
    return DVL_OK;
}

// Kernels with a request per grid row: at most kMaxGridY rows a launch.
constexpr int kMaxGridY = 32768;
template <void (*Kernel)(BatchDev)>
static dvl_status launch_rows(const BatchDev& b, int64_t blocks, int threads, size_t lds, hipStream_t s) {
    for (int q0 = 0; q0 < b.n_reqs; q0 += kMaxGridY) {
        BatchDev part = b;
        part.reqs = b.reqs + q0;
        const int rows = std::min(kMaxGridY, b.n_reqs - q0);
        hipLaunchKernelGGL(Kernel, dim3((unsigned)std::max<int64_t>(1, blocks), rows), dim3(threads), lds, s, part);
        DVL_HIP(hipGetLastError());
    }
    return DVL_OK;
}

template <int MT, typename S>
static dvl_status launch_typed(const BatchLaunch& batch, int n_cu, hipStream_t s, hipEvent_t* ev) {
    const BatchDev& b = batch.dev;
    if (b.paths & kPathEntries) {
        if (dvl_status st = check_no_static_lds<k_tile_sums<MT, S, 1>>("k_tile_sums")) return st;
        if (dvl_status st = check_no_static_lds<k_vmax_exact<MT, S, 1>>("k_vmax_exact")) return st;
        if (dvl_status st = check_no_static_lds<k_bin<MT, S, 1, false>>("k_bin")) return st;
        if (dvl_status st = check_no_static_lds<k_bin<MT, S, 1, true>>("k_bin")) return st;
    }
    auto mark = [&](int i) -> dvl_status {
        if (ev && ev[i]) DVL_HIP(hipEventRecord(ev[i], s));
        return DVL_OK;
    };
    const size_t lds1 = (size_t)sums_lds<false>(b) * sizeof(float) + kSumsPartBytes;
    const size_t lds1i = (size_t)sums_lds<true>(b) * sizeof(float) + kSumsPartBytes;
    if (dvl_status st = mark(0)) return st;
    if (b.any_exact) {
        // 16 steps a wave, so that the atomics on one word stay a few us, but a
        // workgroup for every compute unit; at most four, whose loads in flight
        // fill the memory
        const int64_t want = std::min<int64_t>(std::max<int64_t>(b.n_steps / (16 * kUpdWaves), n_cu), (int64_t)n_cu * 4);
        BatchDev d = b;
        d.chain = std::max<int64_t>(1, (b.k1_units + want - 1) / want);
        const dim3 g((unsigned)std::max<int64_t>(1, (b.k1_units + d.chain - 1) / d.chain));
        if (b.paths & kPathValues) {
            hipLaunchKernelGGL((k_vmax_exact<MT, S, 0>), g, dim3(kUpdThreads), lds1, s, d);
            DVL_HIP(hipGetLastError());
        }
        if (b.paths & kPathEntries) {
            hipLaunchKernelGGL((k_vmax_exact<MT, S, 1>), g, dim3(kUpdThreads), lds1i, s, d);
            DVL_HIP(hipGetLastError());
        }
    }
    if (dvl_status st = mark(1)) return st;
    for (const Share& sh : batch.shares) {
        BatchDev d = b;
        d.reqs = b.reqs + sh.req0;
        d.n_reqs = d.share = sh.n_req;
        d.k1_units = sh.units;
        d.stream = 0;
        if (dvl_status st = launch_sums<k_tile_sums<MT, S, 0>>(d, lds1, n_cu, s)) return st;
    }
    if (b.paths & kPathAlone) {
        if (dvl_status st = launch_sums<k_tile_sums<MT, S, 0>>(b, lds1, n_cu, s)) return st;
    }
    if (b.paths & kPathEntries) {
        if (dvl_status st = launch_sums<k_tile_sums<MT, S, 1>>(b, lds1i, n_cu, s)) return st;
    }
    if (dvl_status st = mark(2)) return st;
    if (dvl_status st = launch_carry_classify(b, batch.far, s)) return st;
    if (dvl_status st = mark(3)) return st;
    const size_t stage = (size_t)b.max_tile_steps * kStageBytesPerStep;
    const size_t tables = ((size_t)b.max_req_tf * sizeof(float) + 15) & ~(size_t)15;
    const size_t tables_i = (size_t)b.max_fields * kIdxTable * sizeof(float);
    auto rescan = [&](auto far) -> dvl_status {
        constexpr bool FAR = decltype(far)::value;
        if (b.paths & kPathBinValues)
            if (dvl_status st = launch_rows<k_bin<MT, S, 0, FAR>>(b, b.max_bin_units, kBinThreads, stage + tables, s)) return st;
        if (b.paths & kPathBinEntries)
            if (dvl_status st = launch_rows<k_bin<MT, S, 1, FAR>>(b, b.max_bin_units, kBinThreads, stage + tables_i, s)) return st;
        if (b.paths & kPathBinStoredF)
            if (dvl_status st = launch_rows<k_bin<MT, S, 2, FAR>>(b, b.max_bin_units, kBinThreads, stage, s)) return st;
        return DVL_OK;
    };
    if (dvl_status st = batch.far ? rescan(std::true_type{}) : rescan(std::false_type{})) return st;
    if (dvl_status st = mark(4)) return st;
    if (dvl_status st = launch_rows<k_bin_stats<MT, S>>(b, (b.max_w + kUpdWaves - 1) / kUpdWaves, kUpdThreads, 0, s)) return st;
    return mark(5);
}

// One storage type and field count.  Each (S, MT) pair is instantiated in a
// translation unit of its own, generated by the build (they compile in
// parallel); elsewhere the declarations below keep the compiler from
// instantiating them.
template <typename S, int MT>
dvl_status launch_sm(const BatchLaunch& b, int n_cu, hipStream_t s, uint64_t layout, hipEvent_t* ev) {
    if (layout != kDescriptorLayout) {
        set_error("descriptor layout mismatch between library objects (%llx vs %llx): rebuild the library",
                  (unsigned long long)layout, (unsigned long long)kDescriptorLayout);
        return DVL_E_INVALID;
    }
    return launch_typed<MT, S>(b, n_cu, s, ev);
}

#define DVL_FOR_EACH_COUNT(X, S) X(S, 1) X(S, 2) X(S, 3) X(S, 4) X(S, 5) X(S, 6) X(S, 7) X(S, 8) X(S, 16)
#define DVL_EXTERN_LAUNCH(S, MT) \
    extern template dvl_status launch_sm<S, MT>(const BatchLaunch&, int, hipStream_t, uint64_t, hipEvent_t*);
DVL_FOR_EACH_COUNT(DVL_EXTERN_LAUNCH, F32)
DVL_FOR_EACH_COUNT(DVL_EXTERN_LAUNCH, F16)
DVL_FOR_EACH_COUNT(DVL_EXTERN_LAUNCH, BF16)
#undef DVL_EXTERN_LAUNCH

// Field-count variants: batches whose volumes all have the same 1 to 8 fields
// run the variant with that count fixed at compile time; others (mixed counts,
// more than 8 fields) the general variant, which reads M per volume and keeps
// the per-field scalars of 16 fields, more than the scalar registers hold.
// Importance pass of 20 M fp32 cells, own variant / general: 3 fields from
// entries 24.5 / 118 us, from values 64 / 171; 6 fields 38 / 145 and 118 / 253.
template <typename S>
static dvl_status launch_s(const BatchLaunch& b, int max_m, int n_cu, hipStream_t s, uint64_t layout, hipEvent_t* ev) {
    switch (max_m) {
        case 1: return launch_sm<S, 1>(b, n_cu, s, layout, ev);
        case 2: return launch_sm<S, 2>(b, n_cu, s, layout, ev);
        case 3: return launch_sm<S, 3>(b, n_cu, s, layout, ev);
        case 4: return launch_sm<S, 4>(b, n_cu, s, layout, ev);
        case 5: return launch_sm<S, 5>(b, n_cu, s, layout, ev);
        case 6: return launch_sm<S, 6>(b, n_cu, s, layout, ev);
        case 7: return launch_sm<S, 7>(b, n_cu, s, layout, ev);
        case 8: return launch_sm<S, 8>(b, n_cu, s, layout, ev);
        default: return launch_sm<S, 16>(b, n_cu, s, layout, ev);
    }
}

}  // namespace dvl
