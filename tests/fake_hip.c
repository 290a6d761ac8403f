/* The HIP runtime entry points that libdualmap.so uses, on host memory and
 * without a device: kernels do not run, copies are memcpy, and every call is
 * counted.  The host side of the library (what it allocates, waits for and
 * reports) runs against it on a machine without a GPU; test_host_calls.py
 * loads it in front of the runtime. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef int hipError_t;
typedef struct { uint32_t x, y, z; } dim3;

/* counters, and what the test sets */
uint64_t fake_mallocs, fake_frees, fake_syncs, fake_launches, fake_bytes;
int fake_last_error, fake_capturing;
void* fake_host;                   /* the last pinned allocation */
hipError_t (*fake_on_sync)(void);  /* result of a stream's synchronization */

hipError_t hipMalloc(void** p, size_t n)
{
    if (fake_capturing)
        return 900; /* hipErrorStreamCaptureUnsupported */
    fake_mallocs++;
    uint64_t* b = calloc(1, n + 4096);
    if (!b)
        return 2;
    b[0] = n;
    fake_bytes += n;
    *p = (char*)b + 4096;
    return 0;
}
hipError_t hipFree(void* p)
{
    if (p) {
        uint64_t* b = (uint64_t*)((char*)p - 4096);
        fake_frees++;
        fake_bytes -= b[0];
        free(b);
    }
    return 0;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned f)
{
    (void)f;
    *p = fake_host = calloc(1, n);
    return 0;
}
hipError_t hipHostFree(void* p) { free(p); return 0; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; memset(d, v, n); return 0; }
hipError_t hipStreamSynchronize(void* st)
{
    (void)st;
    if (fake_capturing)
        return 900;
    fake_syncs++;
    return fake_on_sync ? fake_on_sync() : 0;
}
hipError_t hipStreamIsCapturing(void* st, int* s) { (void)st; *s = fake_capturing; return 0; }
static char some;
hipError_t hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &some; return 0; }
hipError_t hipExtStreamCreateWithCUMask(void** s, uint32_t n, const uint32_t* m) { (void)n; (void)m; *s = &some; return 0; }
hipError_t hipStreamDestroy(void* s) { (void)s; return 0; }
hipError_t hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
hipError_t hipEventCreate(void** e) { *e = &some; return 0; }
hipError_t hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = &some; return 0; }
hipError_t hipEventDestroy(void* e) { (void)e; return 0; }
hipError_t hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
hipError_t hipEventSynchronize(void* e) { (void)e; return 0; }
hipError_t hipEventElapsedTime(float* t, void* a, void* b) { (void)a; (void)b; *t = 0; return 0; }
hipError_t hipGetDevice(int* d) { *d = 0; return 0; }
hipError_t hipSetDevice(int d) { (void)d; return 0; }
hipError_t hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
hipError_t hipGetLastError(void) { return fake_last_error; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "error of the runtime"; }
hipError_t hipGetSymbolAddress(void** p, const void* s)
{
    (void)s;
    static void* area;
    if (!area)
        area = calloc(1, 64u << 20);
    *p = area;
    return 0;
}

static struct { dim3 g, b; size_t lds; void* st; } cfg;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* st)
{
    cfg.g = g;
    cfg.b = b;
    cfg.lds = lds;
    cfg.st = st;
    return 0;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** st)
{
    *g = cfg.g;
    *b = cfg.b;
    *lds = cfg.lds;
    *st = cfg.st;
    return 0;
}
/* kernels by their host function, with the waves of their latest launch */
static struct { const void* f; const char* name; uint64_t waves; } kernel[1024];
static int kernels;
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* st)
{
    (void)args; (void)lds; (void)st;
    fake_launches++;
    for (int i = 0; i < kernels; i++)
        if (kernel[i].f == f)
            kernel[i].waves = (uint64_t)g.x * g.y * g.z * ((b.x * b.y * b.z + 63) / 64);
    return 0;
}
/* most waves of a launch, since the last question, of kernels so named */
uint64_t fake_waves(const char* part)
{
    uint64_t most = 0;
    for (int i = 0; i < kernels; i++)
        if (strstr(kernel[i].name, part)) {
            most = kernel[i].waves > most ? kernel[i].waves : most;
            kernel[i].waves = 0;
        }
    return most;
}
void** __hipRegisterFatBinary(const void* p) { (void)p; static void* h; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* f, char* d, const char* n, unsigned l, void* a, void* b, void* c, void* e, int* w)
{
    (void)h; (void)d; (void)l; (void)a; (void)b; (void)c; (void)e; (void)w;
    if (kernels < 1024) {
        kernel[kernels].f = f;
        kernel[kernels++].name = n;
    }
}
void __hipRegisterVar(void** h, void* v, char* hv, const char* n, int x, size_t s, int c, int g)
{ (void)h; (void)v; (void)hv; (void)n; (void)x; (void)s; (void)c; (void)g; }
