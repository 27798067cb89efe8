/* Stands in for the HIP runtime in tests of the host code, without a GPU: loaded ahead of libbrownout_moe.so, it hands
 * every kernel launch to a callback (name, grid and block sizes, dynamic LDS, pointers to the arguments) whose result becomes
 * the launch's status.  Nothing runs; memory is never touched. */
#include <stddef.h>
#include <string.h>

typedef int hipError_t;
typedef struct { unsigned x, y, z; } dim3_t;
typedef int (*launch_fn)(const char* name, dim3_t grid, dim3_t block, size_t lds, void** args);

static launch_fn g_launch;
static hipError_t g_last;
static struct { const void* host; const char* name; } g_kernels[512];
static int g_n;
static struct { dim3_t grid, block; size_t lds; void* stream; } g_call;
static char g_symbol[256];

void fake_on_launch(launch_fn f) { g_launch = f; }
static hipError_t done(hipError_t e) { if (e) g_last = e; return e; }

void** __hipRegisterFatBinary(const void* data) { (void)data; static void* h; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* device, const char* name, unsigned threads, void* tid, void* bid,
                           dim3_t* bd, dim3_t* gd, int* ws)
{
    (void)m; (void)device; (void)threads; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (g_n < 512) { g_kernels[g_n].host = host; g_kernels[g_n].name = name; ++g_n; }
}
void __hipRegisterVar(void** m, void* var, char* h, char* d, int ext, size_t size, int c, int g)
{
    (void)m; (void)var; (void)h; (void)d; (void)ext; (void)size; (void)c; (void)g;
}
hipError_t __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream)
{
    g_call.grid = grid; g_call.block = block; g_call.lds = lds; g_call.stream = stream;
    return 0;
}
hipError_t __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream)
{
    *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *stream = g_call.stream;
    return 0;
}
hipError_t hipLaunchKernel(const void* host, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream)
{
    (void)stream;
    const char* name = "?";
    for (int i = 0; i < g_n; ++i)
        if (g_kernels[i].host == host) name = g_kernels[i].name;
    return done(g_launch ? g_launch(name, grid, block, lds, args) : 0);
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream)
{
    (void)d; (void)s; (void)n; (void)kind; (void)stream;
    return 0;
}
hipError_t hipGetDevice(int* d) { *d = 0; return 0; }
hipError_t hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
hipError_t hipFuncSetAttribute(const void* f, int attr, int v) { (void)f; (void)attr; (void)v; return 0; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = g_symbol; return 0; }
hipError_t hipGetLastError(void) { hipError_t e = g_last; g_last = 0; return e; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "injected"; }
