/* The HIP calls of libleb.so's host code, recorded instead of run: loaded before the
 * library (RTLD_GLOBAL), these definitions take the place of the runtime's, so that the
 * host side of an entry point runs without a GPU.  Memory is handed out as addresses that
 * nothing reads; a launch is recorded with its size, and one that asks for more dynamic LDS
 * than its kernel may use on the current device is counted as refused. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_;

enum { MAX_LAUNCHES = 1 << 16, MAX_KERNELS = 256, MAX_DEVICES = 8, DEFAULT_LDS = 65536 };
static struct { const void* f; uint64_t groups, lanes; uint32_t gx, gy, gz; size_t lds; } launches[MAX_LAUNCHES];
static struct { const void* f; size_t lds[MAX_DEVICES]; } limits[MAX_KERNELS];
static int n_launches, n_limits, device, refused;
static uintptr_t next_address = 0x100000000;
static char host_memory[1 << 16];

void recorder_device(int d) { device = d; }
void recorder_clear(void) { n_launches = refused = 0; }
int recorder_refused(void) { return refused; }
int recorder_launches(void) { return n_launches; }
const char* recorder_kernel(int i) {
    Dl_info d;
    return dladdr(launches[i].f, &d) && d.dli_sname ? d.dli_sname : "";
}
uint64_t recorder_lanes(int i) { return launches[i].lanes; }
uint64_t recorder_groups(int i) { return launches[i].groups; }
uint64_t recorder_lds(int i) { return launches[i].lds; }

static size_t* limit(const void* f) {
    for (int i = 0; i < n_limits; ++i)
        if (limits[i].f == f) return limits[i].lds;
    limits[n_limits].f = f;
    for (int d = 0; d < MAX_DEVICES; ++d) limits[n_limits].lds[d] = DEFAULT_LDS;
    return limits[n_limits++].lds;
}

static int launch(const void* f, dim3_ g, dim3_ b, size_t lds) {
    if (n_launches == MAX_LAUNCHES) abort();
    launches[n_launches].f = f;
    launches[n_launches].groups = (uint64_t)g.x * g.y * g.z;
    launches[n_launches].lanes = launches[n_launches].groups * b.x * b.y * b.z;
    launches[n_launches].lds = lds;
    ++n_launches;
    if (lds > limit(f)[device]) ++refused;
    return 0;
}

/* a launch's shape on its way to the kernel's stub */
static struct { dim3_ g, b; size_t lds; void* stream; } shape;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void* stream) {
    shape.g = g;
    shape.b = b;
    shape.lds = lds;
    shape.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* lds, void** stream) {
    *g = shape.g;
    *b = shape.b;
    *lds = shape.lds;
    *stream = shape.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, size_t lds, void* stream) {
    (void)args; (void)stream;
    return launch(f, g, b, lds);
}
int hipExtLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, size_t lds, void* stream, void* e0, void* e1,
                       int flags) {
    (void)args; (void)stream; (void)e0; (void)e1; (void)flags;
    return launch(f, g, b, lds);
}
int hipFuncSetAttribute(const void* f, int attr, int value) {
    (void)attr;                                   /* the library sets this one only */
    limit(f)[device] = (size_t)value;
    return 0;
}
int hipFuncGetAttributes(void* attr, const void* f) {
    (void)f;
    memset(attr, 0, 56);                          /* hipFuncAttributes */
    return 0;
}
int hipGetDevice(int* d) { *d = device; return 0; }
int hipMalloc(void** p, size_t bytes) {
    *p = (void*)next_address;
    next_address += (bytes + 4095) & ~(size_t)4095;
    return 0;
}
int hipFree(void* p) { (void)p; return 0; }
int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
    (void)flags;
    *p = host_memory;
    return bytes <= sizeof(host_memory) ? 0 : 2;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned flags) { (void)flags; *d = h; return 0; }
int hipHostFree(void* p) { (void)p; return 0; }
int hipMemcpy(void* d, const void* s, size_t bytes, int kind) { (void)d; (void)s; (void)bytes; (void)kind; return 0; }
int hipMemset(void* d, int v, size_t bytes) { (void)d; (void)v; (void)bytes; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; return hipMalloc(p, 1); }
int hipGetLastError(void) { return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipEventCreate(void** e) { *e = (void*)8; return 0; }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; *e = (void*)8; return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) { (void)s; (void)e; (void)flags; return 0; }
