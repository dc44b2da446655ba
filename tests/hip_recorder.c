/* The HIP runtime calls that libbgpo makes, without a device: every kernel
 * launch is checked against the runtime's launch limits and recorded, nothing
 * runs.  Loaded into the global scope before the library, its symbols take the
 * place of the runtime's (test_launches.py). */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { const void* fn; const char* name; } kernel_t;
typedef struct { const char* name; uint32_t grid[3], block[3]; } launch_t;

enum { kSuccess = 0, kInvalidConfiguration = 9, kMaxKernels = 512, kMaxLaunches = 65536 };

static kernel_t kernels[kMaxKernels];
static int n_kernels;
launch_t rec_launches[kMaxLaunches];
int rec_n_launches;
static int last_error;

void rec_reset(void) { rec_n_launches = 0; last_error = kSuccess; }

void* __hipRegisterFatBinary(const void* data) { static void* h; (void)data; return &h; }
void __hipUnregisterFatBinary(void* h) { (void)h; }
void __hipRegisterVar(void* h, void* var, char* host, char* dev, int ext, size_t size, int c, int g) {
  (void)h; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)c; (void)g;
}
void __hipRegisterFunction(void* h, const void* fn, char* dev, const char* name, unsigned threads,
                           void* tid, void* bid, dim3_t* bd, dim3_t* gd, int* ws) {
  (void)h; (void)dev; (void)threads; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
  if (n_kernels < kMaxKernels) kernels[n_kernels++] = (kernel_t){fn, name};
}

static struct { dim3_t grid, block; size_t shmem; void* stream; } cfg;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void* stream) {
  cfg.grid = grid; cfg.block = block; cfg.shmem = shmem; cfg.stream = stream;
  return kSuccess;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shmem, void** stream) {
  *grid = cfg.grid; *block = cfg.block; *shmem = cfg.shmem; *stream = cfg.stream;
  return kSuccess;
}

/* The runtime's limits: workgroups of at most 1024 work-items, at least one
 * workgroup, at most 65535 in y and z, and fewer than 2^32 work-items in each
 * dimension. */
int hipLaunchKernel(const void* fn, dim3_t grid, dim3_t block, void** args, size_t shmem, void* stream) {
  (void)args; (void)shmem; (void)stream;
  const uint32_t g[3] = {grid.x, grid.y, grid.z}, b[3] = {block.x, block.y, block.z};
  int bad = (uint64_t)b[0] * b[1] * b[2] > 1024 || g[1] > 65535 || g[2] > 65535;
  for (int i = 0; i < 3; ++i) bad |= g[i] == 0 || b[i] == 0 || (uint64_t)g[i] * b[i] >= UINT64_C(1) << 32;
  if (bad) return last_error = kInvalidConfiguration;
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].fn == fn) name = kernels[i].name;
  if (rec_n_launches < kMaxLaunches) {
    launch_t* l = &rec_launches[rec_n_launches++];
    l->name = name;
    memcpy(l->grid, g, sizeof g);
    memcpy(l->block, b, sizeof b);
  }
  return kSuccess;
}
int hipGetLastError(void) { const int e = last_error; last_error = kSuccess; return e; }

int hipGetDevice(int* dev) { *dev = 0; return kSuccess; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return kSuccess; }
int hipGetSymbolAddress(void** p, const void* sym) { (void)sym; *p = (void*)(uintptr_t)0x100000; return kSuccess; }
/* an interval's "time" is the number of launches inside it */
int hipEventCreate(void** e) { static int n; *e = (void*)(uintptr_t)(++n); return kSuccess; }
int hipEventDestroy(void* e) { (void)e; return kSuccess; }
static int event_at[1 << 20];
int hipEventRecord(void* e, void* s) { (void)s; event_at[(uintptr_t)e & 0xFFFFF] = rec_n_launches; return kSuccess; }
int hipEventSynchronize(void* e) { (void)e; return kSuccess; }
int hipEventElapsedTime(float* ms, void* a, void* b) {
  *ms = (float)(event_at[(uintptr_t)b & 0xFFFFF] - event_at[(uintptr_t)a & 0xFFFFF]);
  return kSuccess;
}
