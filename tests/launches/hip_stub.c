/* The HIP runtime's entry points that the library's host code calls, for tests
 * that look at the launches of a call without a GPU: a launch is recorded (the
 * kernel's name, grid and block) and nothing runs.  Loaded before the library,
 * with global symbols, it takes the runtime's place. */
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;

#define MAX_KERNELS 4096
static struct { const void* host; char name[192]; } kernels[MAX_KERNELS];
static int kernel_count;

#define MAX_LAUNCHES 65536
static struct { const void* host; unsigned grid, block; const void* stream; } launches[MAX_LAUNCHES];
static int launch_count;

void stub_reset(void) { launch_count = 0; }
int stub_launches(void) { return launch_count; }
unsigned stub_grid(int q) { return launches[q].grid; }
unsigned stub_block(int q) { return launches[q].block; }
const char* stub_name(int q) {
    for (int i = 0; i < kernel_count; ++i)
        if (kernels[i].host == launches[q].host) return kernels[i].name;
    return "";
}

void** __hipRegisterFatBinary(const void* data) {
    static void* module;
    (void)data;
    return &module;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned lim,
                           void* tid, void* bid, void* bd, void* gd, int* ws) {
    (void)m; (void)dev; (void)lim; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (kernel_count >= MAX_KERNELS) return;
    kernels[kernel_count].host = host;
    strncpy(kernels[kernel_count].name, name, sizeof(kernels[0].name) - 1);
    ++kernel_count;
}
void __hipRegisterVar(void** m, void* var, char* host, char* dev, int ext, size_t size, int c, int g) {
    (void)m; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)c; (void)g;
}

static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
    cfg_grid = grid;
    cfg_block = block;
    cfg_lds = lds;
    cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
    *grid = cfg_grid;
    *block = cfg_block;
    *lds = cfg_lds;
    *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
    (void)args; (void)lds;
    if (launch_count >= MAX_LAUNCHES) return 1;
    launches[launch_count].host = f;
    launches[launch_count].grid = grid.x;
    launches[launch_count].block = block.x;
    launches[launch_count].stream = stream;
    ++launch_count;
    return 0;
}

int hipGetLastError(void) { return 0; }
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds) {
    (void)f; (void)block; (void)lds;
    *n = 2;
    return 0;
}
int hipFuncSetAttribute(const void* f, int attr, int v) { (void)f; (void)attr; (void)v; return 0; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = 0; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned flags) { static int x; (void)flags; *s = &x; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) { (void)s; (void)e; (void)flags; return 0; }
int hipEventCreateWithFlags(void** e, unsigned flags) { static int x; (void)flags; *e = &x; return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
