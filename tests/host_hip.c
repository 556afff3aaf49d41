/* A HIP runtime without a device, for tests of the library's host code: copies are copies in host
 * memory, launches run nothing and are recorded, and a launch that asks for more LDS than a CU has,
 * or every launch after host_hip_fail(1), fails as the real runtime's would.  Loaded before the
 * library with RTLD_GLOBAL, so that its calls resolve here.  Buffers come zeroed, so clearing does
 * nothing. */
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
enum { LDS_CU = 160 * 1024, E_VALUE = 1 };

static dim3_t g_grid, g_block;
static size_t g_shmem, g_max;
static void* g_stream;
static long g_launches;
static int g_fail, g_err;

long host_hip_launches(void) { return g_launches; }
size_t host_hip_max_lds(void) { return g_max; }
void host_hip_reset(void) { g_launches = 0; g_max = 0; g_err = 0; }
void host_hip_fail(int on) { g_fail = on; }

void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* a, const char* b, unsigned t, void* c, void* d, void* e,
                           void* g, int* w) { (void)m; (void)f; (void)a; (void)b; (void)t; (void)c; (void)d; (void)e; (void)g; (void)w; }
void __hipRegisterVar(void** m, void* v, char* a, char* b, int e, size_t n, int c, int g)
{ (void)m; (void)v; (void)a; (void)b; (void)e; (void)n; (void)c; (void)g; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t s, void* st)
{ g_grid = g; g_block = b; g_shmem = s; g_stream = st; return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* s, void** st)
{ *g = g_grid; *b = g_block; *s = g_shmem; *st = g_stream; return 0; }

int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t shmem, void* st)
{
    (void)f; (void)g; (void)b; (void)args; (void)st;
    g_launches++;
    if (shmem > g_max) g_max = shmem;
    if (g_fail || shmem > LDS_CU) return g_err = E_VALUE;
    return 0;
}
int hipGetLastError(void) { const int e = g_err; g_err = 0; return e; }
const char* hipGetErrorString(int e) { return e ? "launch failed" : "no error"; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d)
{ (void)a; (void)d; *v = LDS_CU; return 0; }     /* the library asks for the LDS and for the number of CUs */
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t s)
{ (void)f; (void)b; (void)s; *n = 1; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipMemset(void* p, int v, size_t n) { (void)p; (void)v; (void)n; return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { (void)p; (void)v; (void)n; (void)s; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
int hipEventCreate(void** e) { static char event; *e = &event; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.0f; return 0; }
