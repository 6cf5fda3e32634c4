// A HIP runtime without a device, for tests of the library's host code on the
// CPU: device memory is host memory, streams and events are names, launches
// are recorded instead of run.  Three kernels whose results the host waits for
// are stood in for (data ranges, grid extent, the packing of bins).  Loaded
// into the global scope before libdvl.so, whose HIP symbols then resolve here.
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

struct Dim3 { uint32_t x, y, z; };
struct Launch { std::string name; Dim3 grid, block; size_t lds; void* stream; };

static std::mutex mu;
static std::map<const void*, std::string> names;
static std::vector<Launch> launches;
static int n_malloc, n_free, n_host_malloc, n_instantiate, n_fail_malloc;
static bool fail_new, fail_attribute;
static int sync_parties, sync_here;            // hipStreamSynchronize waits for so many threads
static pthread_cond_t sync_cv = PTHREAD_COND_INITIALIZER;
static pthread_mutex_t sync_mu = PTHREAD_MUTEX_INITIALIZER;

struct Pack {                                   // the argument of k_pack
    int n;
    const uint32_t* src[8];
    uint32_t words[8], at[8];
};

void* operator new(size_t n) {
    if (fail_new) throw std::bad_alloc();
    return malloc(n ? n : 1);
}

void* operator new(size_t n, const std::nothrow_t&) noexcept { return malloc(n ? n : 1); }

static void stand_in(const std::string& name, Dim3 grid, void** args) {
    auto has = [&](const char* s) { return name.find(s) != std::string::npos; };
    if (has("k_extent_fold")) {
        unsigned long long* out = *(unsigned long long**)args[2];
        out[0] = 64;
        out[1] = out[2] = 0;
    } else if (has("k_range_fold")) {           // every field's data range: [0, 1]
        uint32_t* out = *(uint32_t**)args[2];
        for (uint32_t m = 0; m <= grid.x; ++m) {
            out[2 * m] = m < grid.x ? 0x80000000u : 0u;
            out[2 * m + 1] = m < grid.x ? 0xBF800000u : 0u;
        }
    } else if (has("k_pack")) {
        const Pack* l = (const Pack*)args[0];
        uint32_t* out = *(uint32_t**)args[1];
        for (int a = 0; a < l->n; ++a) memcpy(out + l->at[a], l->src[a], (size_t)l->words[a] * 4);
    }
}

extern "C" {

// ------------------------------------------------------------ seen by the tests
void fake_reset() {
    std::lock_guard<std::mutex> lk(mu);
    launches.clear();
    n_malloc = n_free = n_host_malloc = n_instantiate = 0;
}
int fake_launches() { return (int)launches.size(); }
const char* fake_name(int i) { return launches[i].name.c_str(); }
uint32_t fake_grid(int i, int d) { return d == 0 ? launches[i].grid.x : (d == 1 ? launches[i].grid.y : launches[i].grid.z); }
int fake_mallocs() { return n_malloc; }
int fake_frees() { return n_free; }
int fake_host_mallocs() { return n_host_malloc; }
int fake_instantiated() { return n_instantiate; }
void fake_fail_mallocs(int n) { n_fail_malloc = n; }
void fake_fail_new(int on) { fail_new = on != 0; }
void fake_fail_attribute(int on) { fail_attribute = on != 0; }
void fake_sync_parties(int n) { sync_parties = n; sync_here = 0; }

// ------------------------------------------------------------ the runtime
static thread_local struct { Dim3 grid, block; size_t lds; void* stream; } config;
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    config = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    std::lock_guard<std::mutex> lk(mu);
    names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t lds, void* stream) {
    std::lock_guard<std::mutex> lk(mu);
    const std::string name = names[f];
    launches.push_back({name, grid, block, lds, stream});
    stand_in(name, grid, args);
    return 0;
}
int hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> lk(mu);
    if (n_fail_malloc > 0) {
        --n_fail_malloc;
        return 2;
    }
    ++n_malloc;
    return posix_memalign(p, 4096, n) ? 2 : 0;
}
int hipFree(void* p) {
    std::lock_guard<std::mutex> lk(mu);
    ++n_free;
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    std::lock_guard<std::mutex> lk(mu);
    ++n_host_malloc;
    return posix_memalign(p, 4096, n) ? 2 : 0;
}
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipStreamSynchronize(void*) {
    if (sync_parties < 2) return 0;
    pthread_mutex_lock(&sync_mu);
    if (++sync_here >= sync_parties)
        pthread_cond_broadcast(&sync_cv);
    else
        while (sync_here < sync_parties) pthread_cond_wait(&sync_cv, &sync_mu);
    pthread_mutex_unlock(&sync_mu);
    return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) {                               // compute units
    *v = 256;
    return fail_attribute ? 1 : 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 5; return 0; }
int hipFuncGetAttributes(void* a, const void*) { memset(a, 0, 56); return 0; }
int hipPointerGetAttributes(void*, const void*) { return 1; }
int hipGetSymbolAddress(void** p, const void*) { *p = malloc((size_t)64 << 20); return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "error"; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = malloc(1); return 0; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { ++n_instantiate; *x = malloc(1); return 0; }
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void* g) { free(g); return 0; }
int hipGraphExecDestroy(void* g) { free(g); return 0; }

}  // extern "C"
