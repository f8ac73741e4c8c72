/* A HIP runtime that runs nothing, for tests of the library's host side on a
 * machine without a GPU: every call succeeds unless it was told to fail,
 * device memory is address space that nothing reads, and the calls that
 * matter (allocations, launches) are written to a log, one line each.
 * Loaded with RTLD_GLOBAL ahead of libschulze.so, so that its definitions
 * are found before the runtime's. */
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

enum { MAX_KERNELS = 1024, LOG_BYTES = 1 << 20 };
static struct { const void *fn; char name[256]; } kernels[MAX_KERNELS];
static int n_kernels;
static char log_text[LOG_BYTES];
static size_t log_len;
static int fail_malloc_in = -1;  /* device allocations until one fails; -1: never */
static int fail_attribute, refuse_cooperative;
static uintptr_t next_address = (uintptr_t)1 << 44;
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } pushed;

static void note(const char *format, ...) {
    va_list a;
    va_start(a, format);
    if (log_len < LOG_BYTES) {
        const int n = vsnprintf(log_text + log_len, LOG_BYTES - log_len, format, a);
        if (n > 0) log_len += (size_t)n;
    }
    va_end(a);
}

const char *fake_log(void) { return log_text; }
void fake_reset(void) { log_len = 0; log_text[0] = 0; fail_malloc_in = -1; fail_attribute = refuse_cooperative = 0; }
void fake_fail_malloc(int after) { fail_malloc_in = after; }
void fake_fail_attribute(int on) { fail_attribute = on; }
void fake_refuse_cooperative(int on) { refuse_cooperative = on; }

/* ---- registration of the library's kernels */
void **__hipRegisterFatBinary(const void *data) { (void)data; return (void **)&kernels; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned int threads,
                           void *tid, void *bid, void *bdim, void *gdim, int *wsize) {
    (void)modules, (void)device, (void)threads, (void)tid, (void)bid, (void)bdim, (void)gdim, (void)wsize;
    if (n_kernels == MAX_KERNELS) abort();
    kernels[n_kernels].fn = host;
    snprintf(kernels[n_kernels++].name, sizeof kernels[0].name, "%s", name);
}
void __hipRegisterVar(void **modules, void *var, char *host, char *device, int ext, size_t size, int constant,
                      int global) {
    (void)modules, (void)var, (void)host, (void)device, (void)ext, (void)size, (void)constant, (void)global;
}

/* ---- launches */
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    pushed.grid = grid, pushed.block = block, pushed.lds = lds, pushed.stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
    *grid = pushed.grid, *block = pushed.block, *lds = pushed.lds, *stream = pushed.stream;
    return hipSuccess;
}
static hipError_t launch(const char *how, const void *fn, dim3 grid, dim3 block) {
    /* the runtime's limit on threads of a dimension */
    if ((uint64_t)grid.x * block.x >> 32) {
        note("%s refused: %u x %u threads\n", how, grid.x, block.x);
        return hipErrorInvalidConfiguration;
    }
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].fn == fn) note("%s %s %u %u %u\n", how, kernels[i].name, grid.x, grid.y, block.x);
    return hipSuccess;
}
static hipError_t last_error;
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
    (void)args, (void)lds, (void)stream;
    return last_error = launch("launch", fn, grid, block);
}
hipError_t hipLaunchCooperativeKernel(const void *fn, dim3 grid, dim3 block, void **args, unsigned int lds,
                                      hipStream_t stream) {
    (void)args, (void)lds, (void)stream;
    return last_error = refuse_cooperative ? hipErrorCooperativeLaunchTooLarge
                                           : launch("cooperative", fn, grid, block);
}
hipError_t hipGetLastError(void) { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *fn, int threads, size_t lds) {
    (void)fn, (void)threads, (void)lds;
    *blocks = 2;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *fn, hipFuncAttribute attribute, int value) {
    (void)fn, (void)attribute, (void)value;
    return fail_attribute ? hipErrorInvalidValue : hipSuccess;
}

/* ---- memory */
hipError_t hipMalloc(void **p, size_t bytes) {
    if (fail_malloc_in == 0) {
        note("malloc refused: %zu\n", bytes);
        *p = NULL;
        return last_error = hipErrorOutOfMemory;
    }
    if (fail_malloc_in > 0) --fail_malloc_in;
    *p = (void *)next_address;
    next_address += (bytes + 4095) / 4096 * 4096;
    note("malloc %zu\n", bytes);
    return hipSuccess;
}
hipError_t hipFree(void *p) { (void)p; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned int flags) {
    (void)flags;
    return (*p = calloc(1, bytes)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned int flags) { (void)flags; *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *symbol) { *p = (void *)(uintptr_t)symbol; return hipSuccess; }
hipError_t hipMemset(void *p, int value, size_t bytes) { (void)p, (void)value, (void)bytes; return hipSuccess; }
static hipError_t copy(void *dst, size_t bytes, hipMemcpyKind kind) {
    if (kind == hipMemcpyDeviceToHost) memset(dst, 0, bytes);
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t bytes, hipMemcpyKind kind) {
    (void)src;
    return copy(dst, bytes, kind);
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind kind, hipStream_t stream) {
    (void)src, (void)stream;
    return copy(dst, bytes, kind);
}

/* ---- device, streams, events */
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int device) { (void)device; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int device) {
    (void)device;
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t stream) { (void)stream; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t stream, hipStreamCaptureStatus *status) {
    (void)stream;
    *status = hipStreamCaptureStatusNone;
    return hipSuccess;
}
