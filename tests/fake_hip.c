/* A stand-in for the HIP runtime, so that the host side of libbps.so runs without a GPU: "device" memory is host
 * memory, streams run everything at once, and a kernel launch appends one line to a log.  The two kernels that move
 * work items (k_unpack_items, k_dispatch_order: here the items as they are) are carried out, and a k_raster line tells
 * what the kernel would find in its item array.  Load it RTLD_GLOBAL before libbps.so: it is then found first. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t env, scene, split_of, tile; } item;

static struct { const void* host; char name[256]; } g_kernels[256];
static int g_n_kernels;
static struct { void* var; void* memory; size_t size; } g_vars[16];
static int g_n_vars;
static char g_log[1 << 20];
static size_t g_log_at;

static const void* g_scenes;      /* the scene table of the last k_raster */
const void* fake_scenes(void) { return g_scenes; }
const char* fake_log(void) { return g_log; }
void fake_clear_log(void) { g_log[g_log_at = 0] = 0; }
/* kernels and records of events in the order they were enqueued, a line each; events by their numbers */
static char g_ops[1 << 16];
static size_t g_ops_at;
const char* fake_ops(void) { return g_ops; }
void fake_clear_ops(void) { g_ops[g_ops_at = 0] = 0; }
typedef struct { long held; int number; } event;
static const char* kernel_name(const void* f);
static void op(const char* what, hipEvent_t e) {
    const size_t room = sizeof(g_ops) - g_ops_at;
    const int n = e ? snprintf(g_ops + g_ops_at, room, "%s event=%d\n", what, ((event*)e)->number) : snprintf(g_ops + g_ops_at, room, "%s\n", what);
    if (n < 0 || (size_t)n >= room) abort();
    g_ops_at += (size_t)n;
}

void** __hipRegisterFatBinary(const void* data) { (void)data; static void* handle; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device_function, const char* name, unsigned limit, void* tid,
                           void* bid, dim3* block, dim3* grid, int* wsize) {
    (void)modules; (void)device_function; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (g_n_kernels == 256) abort();
    g_kernels[g_n_kernels].host = host;
    strncpy(g_kernels[g_n_kernels++].name, name, 255);
}
void __hipRegisterVar(void** modules, void* var, char* host_name, char* device_name, int ext, size_t size, int constant, int global) {
    (void)modules; (void)host_name; (void)device_name; (void)ext; (void)constant; (void)global;
    if (g_n_vars == 16) abort();
    g_vars[g_n_vars].var = var;
    g_vars[g_n_vars].size = size;
    g_vars[g_n_vars++].memory = calloc(1, size);
}

static struct { dim3 grid, block; size_t shared; hipStream_t stream; } g_config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    g_config.grid = grid; g_config.block = block; g_config.shared = shared; g_config.stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    *grid = g_config.grid; *block = g_config.block; *shared = g_config.shared; *stream = g_config.stream;
    return hipSuccess;
}

#define ARG(type, k) (*(type*)args[k])

static const char* kernel_name(const void* f) {
    for (int k = 0; k < g_n_kernels; ++k)
        if (g_kernels[k].host == f) return g_kernels[k].name;
    return "?";
}
static hipError_t run(const void* f, dim3 grid, dim3 block, void** args, size_t shared, hipStream_t stream) {
    (void)stream;
    const char* name = kernel_name(f);
    char* out = g_log + g_log_at;
    const size_t room = sizeof(g_log) - g_log_at;
    int n;
    if (strstr(name, "k_unpack_items")) {            /* (packed words, first, count, items) */
        const uint32_t first = ARG(uint32_t, 1), count = ARG(uint32_t, 2);
        item* items = ARG(item*, 3);
        for (uint32_t k = 0; k < count; ++k) {
            const uint32_t w = ((const uint32_t*)args[0])[k];
            const item it = {w & 0x3FFFu, (w >> 14) & 0xFFFu, 1u << 16, w >> 26};
            items[first + k] = it;
        }
        n = snprintf(out, room, "k_unpack_items\n");
    } else if (strstr(name, "k_dispatch_order")) {   /* (cost, n_items, items, ordered) */
        memcpy(ARG(item*, 3), ARG(const item*, 2), ARG(uint32_t, 1) * sizeof(item));
        n = snprintf(out, room, "k_dispatch_order\n");
    } else if (strstr(name, "k_raster")) {           /* (scenes, items, view_proj, ...) */
        /* shared: work-groups whose item names no share of the scene, or one drawn by another group already */
        const item* items = ARG(const item*, 1);
        g_scenes = ARG(const void*, 0);
        uint32_t envs = 0, tiles = 0, wrong = 0;
        uint8_t* seen = (uint8_t*)calloc(1, 65536u * 64u);
        for (uint32_t k = 0; k < grid.x; ++k) {
            if (items[k].env >= envs) envs = items[k].env + 1;
            if (items[k].tile >= tiles) tiles = items[k].tile + 1;
            if (items[k].split_of != 1u << 16 || items[k].env > 0xFFFFu || items[k].tile > 63u || seen[64u * items[k].env + items[k].tile]++) ++wrong;
        }
        free(seen);
        n = snprintf(out, room, "k_raster groups=%u envs=%u tiles=%u wrong=%u threads=%u lds=%zu\n", grid.x, envs, tiles, wrong, block.x, shared);
    } else {
        n = snprintf(out, room, "%s\n", name);
    }
    if (n < 0 || (size_t)n >= room) abort();
    g_log_at += (size_t)n;
    return hipSuccess;
}

/* Capture: launches are kept, with copies of the arguments the logged kernels have, and carried out by fake_replay. */
typedef struct { const void* f; dim3 grid, block; void* args[4]; } captured;
static captured g_graph[64];
static int g_capturing, g_n_graph, g_unknown;
void fake_capture_unknown(int on) { g_unknown = on; }      /* whether a stream is being captured cannot be told */
void fake_capture(int on) { g_capturing = on; if (on) g_n_graph = 0; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
    (void)s;
    if (g_unknown) return hipErrorStreamCaptureImplicit;
    *status = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
static hipError_t launch(const void* f, dim3 grid, dim3 block, void** args, size_t shared, hipStream_t stream) {
    if (!g_capturing) return run(f, grid, block, args, shared, stream);
    if (g_n_graph == 64) abort();
    captured* c = &g_graph[g_n_graph++];
    c->f = f; c->grid = grid; c->block = block;
    const char* name = kernel_name(f);
    const size_t unpack[4] = {3840, 4, 4, 8}, order[4] = {8, 4, 8, 8}, raster[4] = {8, 8, 8, 0}, none[4] = {0, 0, 0, 0};
    const size_t* size = strstr(name, "k_unpack_items") ? unpack : strstr(name, "k_dispatch_order") ? order : strstr(name, "k_raster") ? raster : none;
    for (int k = 0; k < 4; ++k) c->args[k] = memcpy(malloc(size[k] + 1), size[k] ? args[k] : "", size[k]);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shared, hipStream_t stream) {
    op(kernel_name(f), NULL);
    return launch(f, grid, block, args, shared, stream);
}
/* an event that is the end of a kernel; a kernel of a graph has none */
static long g_held, g_holds;
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shared, hipStream_t stream, hipEvent_t start,
                              hipEvent_t stop, int flags) {
    if (g_capturing || start || !stop || flags) return hipErrorNotSupported;
    op(kernel_name(f), stop);
    ((event*)stop)->held = g_held;
    return launch(f, grid, block, args, shared, stream);
}
void fake_replay(void) {
    for (int k = 0; k < g_n_graph; ++k) run(g_graph[k].f, g_graph[k].grid, g_graph[k].block, g_graph[k].args, 0, NULL);
}

static int g_units = 256;
void fake_compute_units(int n) { g_units = n; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int device) {
    (void)device;
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = g_units;
    p->sharedMemPerBlock = 163840;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int device) { (void)a; (void)device; *v = 163840; return hipSuccess; }
hipError_t hipSetDevice(int device) { (void)device; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "fake error"; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v) { (void)f; (void)a; (void)v; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
    for (int k = 0; k < g_n_vars; ++k)
        if (g_vars[k].var == symbol) { *p = g_vars[k].memory; return hipSuccess; }
    return hipErrorInvalidSymbol;
}

/* device blocks and pinned ones: how many were allocated, how many of them live, the last one's size, and the
 * largest that there is room for */
static struct { unsigned long allocated, live; size_t largest, last; } g_memory[2] = {{0, 0, (size_t)-1, 0}, {0, 0, (size_t)-1, 0}};
unsigned long fake_allocated(int pinned) { return g_memory[pinned].allocated; }
unsigned long fake_live(int pinned) { return g_memory[pinned].live; }
unsigned long fake_last_size(int pinned) { return g_memory[pinned].last; }
void fake_largest(int pinned, size_t n) { g_memory[pinned].largest = n; }
static hipError_t allocate(int pinned, void** p, size_t n) {
    if (n > g_memory[pinned].largest || posix_memalign(p, 256, n ? n : 1)) return hipErrorOutOfMemory;
    g_memory[pinned].last = n;
    ++g_memory[pinned].allocated;
    ++g_memory[pinned].live;
    return hipSuccess;
}
static hipError_t release(int pinned, void* p) {
    if (p) --g_memory[pinned].live;
    free(p);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return allocate(0, p, n); }
hipError_t hipFree(void* p) { return release(0, p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) { (void)flags; return allocate(1, p, n); }
hipError_t hipHostFree(void* p) { return release(1, p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
static unsigned long g_copied;
unsigned long fake_copied(void) { return g_copied; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t q) { (void)q; g_copied += n; return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
/* memory is on the device where the test says so */
static uintptr_t g_device_lo, g_device_hi;
void fake_device_range(void* p, size_t n) { g_device_lo = (uintptr_t)p; g_device_hi = g_device_lo + n; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof(*a));
    a->type = (uintptr_t)p >= g_device_lo && (uintptr_t)p < g_device_hi ? hipMemoryTypeDevice : hipMemoryTypeHost;
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned flags) { (void)flags; *s = (hipStream_t)malloc(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned flags) { (void)s; (void)e; (void)flags; return hipSuccess; }
/* events recorded while the device is held are not reached until it goes on */
void fake_hold(int on) { g_held = on ? ++g_holds : 0; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) { (void)flags; static int n; *e = (hipEvent_t)calloc(1, sizeof(event)); ((event*)*e)->number = ++n; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)s; op("record", e); ((event*)e)->held = g_held; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { return g_held && ((event*)e)->held == g_held ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { (void)a; (void)b; *ms = 0.0f; return hipSuccess; }
