/* A stand-in for the HIP calls of the library's host code, so that a test can
 * follow on the CPU which calls it makes: nothing runs, launches and copies
 * are counted, and pinned host memory is the one range that
 * fake_set_pinned names.  Loaded with RTLD_GLOBAL ahead of the library. */
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

static char* pin_at;
static size_t pin_len;
static long n_launch, n_memcpy;
static unsigned last_grid;
static void* page;
static size_t page_len;

void fake_set_pinned(void* at, size_t len) { pin_at = at, pin_len = len; }
void fake_fill_page(int byte) { memset(page, byte, page_len); } /* the newest hipHostMalloc */
unsigned fake_last_grid(void) { return last_grid; }
long fake_launches(void) { return n_launch; }
long fake_memcpys(void) { return n_memcpy; }

static int pinned(const void* p) { return pin_at != NULL && (char*)p >= pin_at && (char*)p < pin_at + pin_len; }

hipError_t hipEventCreate(hipEvent_t* e) { return *e = malloc(1), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { return (void)f, *e = malloc(1), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { return (void)a, (void)b, *ms = 0, hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return (void)e, (void)s, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) {
    return (void)f, *p = page = calloc(1, n), page_len = n, hipSuccess;
}
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned f) { return (void)f, *d = h, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return (void)s, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { return (void)s, (void)e, (void)f, hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t s) { return (void)p, (void)v, (void)n, (void)s, hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st) {
    return (void)d, (void)s, (void)n, (void)k, (void)st, n_memcpy++, hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof *a);
    if (!pinned(p)) return hipErrorInvalidValue;
    a->type = hipMemoryTypeHost;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
    if (!pinned(p)) return hipErrorNotFound;
    return *base = pin_at, *size = pin_len, hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t l, hipStream_t s) {
    return (void)f, (void)b, (void)a, (void)l, (void)s, last_grid = g.x, n_launch++, hipSuccess;
}
static dim3 conf_grid, conf_block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) {
    return (void)l, (void)s, conf_grid = g, conf_block = b, hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
    return *g = conf_grid, *b = conf_block, *l = 0, *s = NULL, hipSuccess;
}
