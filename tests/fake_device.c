/* A device that runs nothing, for tests of the host side without a GPU: the
 * runtime calls that the library makes, with memory from the host and launches
 * that are only counted.  fake_* set what fails and read the counts. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };

static long long launches, launch_limit = -1, uploads, upload_limit = -1;
static size_t upload_bytes, held;

/* launches (uploads) after the n-th from now fail; n < 0: none */
void fake_launches(long long n) { launches = 0; launch_limit = n; }
void fake_uploads(long long n) { uploads = 0; upload_bytes = 0; upload_limit = n; }
long long fake_launch_count(void) { return launches; }
long long fake_upload_count(void) { return uploads; }
size_t fake_upload_bytes(void) { return upload_bytes; }
size_t fake_held_bytes(void) { return held; }

/* (memory is touched only where it is written) */
hipError_t hipMalloc(void** p, size_t n)
{
    size_t* m = mmap(0, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    *m = n;
    held += n;
    *p = (char*)m + 4096;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (!p) return hipSuccess;
    size_t* m = (size_t*)((char*)p - 4096);
    held -= *m;
    munmap(m, *m + 4096);
    return hipSuccess;
}
/* kind 1: to the device; 1 MiB and more are counted only */
hipError_t hipMemcpy(void* d, const void* s, size_t n, int kind)
{
    if (kind == 1) {
        if (upload_limit >= 0 && uploads >= upload_limit) return hipErrorUnknown;
        ++uploads;
        upload_bytes += n;
        if (n >= ((size_t)1 << 20)) return hipSuccess;
    }
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { return hipMemcpy(d, s, n, kind); }

static hipError_t last;
static struct { dim3 g, b; size_t lds; void* st; } conf;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* st)
{
    conf.g = g; conf.b = b; conf.lds = lds; conf.st = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** st)
{
    *g = conf.g; *b = conf.b; *lds = conf.lds; *st = conf.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* st)
{
    if (launch_limit >= 0 && launches >= launch_limit) return last = hipErrorUnknown;
    ++launches;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t e) { return e ? "planned failure" : "no error"; }

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(void* s) { return hipSuccess; }
hipError_t hipStreamIsCapturing(void* s, int* c) { *c = 0; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, int a, int v) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l) { *n = 2; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { static char area[8]; *p = area; return hipSuccess; }
hipError_t hipEventCreate(void** e) { static int ev; *e = &ev; return hipSuccess; }
hipError_t hipEventDestroy(void* e) { return hipSuccess; }
hipError_t hipEventRecord(void* e, void* s) { return hipSuccess; }
hipError_t hipEventSynchronize(void* e) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 1.0f; return hipSuccess; }
