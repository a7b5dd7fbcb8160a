/* A stand-in for the HIP runtime on a machine without a GPU: loaded with global
 * symbols before one of the package's libraries, it takes the runtime calls of
 * the library's host code, launches nothing, and notes every kernel launch. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_;
typedef struct { const char* name; dim3_ grid, block; const void* arg[2]; } launch_t;

enum { kMost = 65536, kError = 719 };
static struct { const void* host; const char* name; } kernels[4096];
static int nkernels;
static launch_t launches[kMost];
static int nlaunches, fail_at = -1, last_error, capturing, queries, cus = 256;
static dim3_ cfg_grid, cfg_block;

/* for the test: forget the launches; make launch number n fail (-1: none);
 * whether streams are being captured; compute units of the device */
void rec_reset(int fail, int capture, int compute_units)
{
    nlaunches = queries = last_error = 0;
    fail_at = fail;
    capturing = capture;
    cus = compute_units;
}
int rec_count(void) { return nlaunches; }
int rec_queries(void) { return queries; }
const launch_t* rec_get(int i) { return &launches[i]; }

void** __hipRegisterFatBinary(const void* data) { return (void**)&data; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned t, void* a, void* b,
                           void* c, void* d, int* w)
{
    kernels[nkernels].host = host;
    kernels[nkernels++].name = name;
}
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t shared, void* stream)
{
    cfg_grid = grid;
    cfg_block = block;
    return 0;
}
int __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* shared, void** stream)
{
    *grid = cfg_grid;
    *block = cfg_block;
    *shared = 0;
    *stream = NULL;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_ grid, dim3_ block, void** args, size_t shared, void* stream)
{
    if (nlaunches == fail_at || nlaunches == kMost) return last_error = kError;
    launch_t* l = &launches[nlaunches++];
    l->name = "";
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].host == f) l->name = kernels[i].name;
    l->grid = grid;
    l->block = block;
    memcpy(&l->arg[0], args[0], sizeof(void*));
    memcpy(&l->arg[1], args[1], sizeof(void*));
    return 0;
}
int hipGetLastError(void)
{
    int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int e) { return e ? "planted failure" : "no error"; }
int hipGetDevice(int* d) { return *d = 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev)
{
    *v = cus;
    return 0;
}
int hipStreamIsCapturing(void* stream, int* status)
{
    ++queries;
    *status = capturing;
    return 0;
}
int hipStreamSynchronize(void* stream) { return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { return 1; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t shared) { return !(*n = 1); }
