/* The HIP calls that libbbo_mlp.so makes, as a record of what was asked: lets a test without a GPU follow a call's
 * planning and launches.  Loaded with RTLD_GLOBAL ahead of the library.  Nothing runs, and no pointer is followed but
 * those the host owns.  hr_fail_launch: the launch (counted from 1) that fails, 0 for none; hr_fail_record: likewise for
 * event records. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
  uint32_t x, y, z;
} dim3;
enum { OK = 0, INVALID = 1 };

static char text[1 << 20];
static size_t used;
static intptr_t handles;
static int launches, records;
int hr_fail_launch, hr_fail_record, hr_capturing;

const char* hr_log(void) { return text; }
void hr_reset(void) {
  used = 0;
  text[0] = 0;
  launches = records = 0;
}
#define LOG(...) (used += (size_t)snprintf(text + used, sizeof(text) - used, __VA_ARGS__))

int hipGetDevice(int* dev) { return *dev = 0, OK; }
int hipDeviceGetAttribute(int* v, int what, int dev) { return (void)what, (void)dev, *v = 256, OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int threads, size_t lds) {
  return (void)f, (void)threads, (void)lds, *n = 2, OK;
}
int hipFuncSetAttribute(const void* f, int what, int v) { return (void)f, (void)what, (void)v, OK; }
int hipGetLastError(void) { return OK; }
int hipGetSymbolAddress(void** p, const void* sym) { return (void)sym, *p = (void*)(intptr_t)0x10000, OK; }
int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
  (void)flags;
  LOG("host_malloc\n");
  return (*p = malloc(bytes)) ? OK : INVALID;
}
int hipHostFree(void* p) { return free(p), OK; }
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int kind, intptr_t s) {
  return (void)dst, (void)src, (void)bytes, (void)kind, LOG("copy %ld\n", (long)s), OK;
}
int hipStreamIsCapturing(intptr_t s, int* status) { return (void)s, *status = hr_capturing, OK; }
int hipStreamCreateWithFlags(intptr_t* s, unsigned flags) {
  (void)flags;
  *s = ++handles;
  return LOG("new_stream %ld\n", (long)*s), OK;
}
int hipStreamDestroy(intptr_t s) { return (void)s, OK; }
int hipStreamSynchronize(intptr_t s) { return LOG("sync %ld\n", (long)s), OK; }
int hipEventCreateWithFlags(intptr_t* e, unsigned flags) {
  (void)flags;
  *e = ++handles;
  return LOG("new_event %ld\n", (long)*e), OK;
}
int hipEventDestroy(intptr_t e) { return (void)e, OK; }
int hipEventSynchronize(intptr_t e) { return (void)e, OK; }
int hipEventRecord(intptr_t e, intptr_t s) {
  if (++records == hr_fail_record) return LOG("record_failed %ld %ld\n", (long)e, (long)s), INVALID;
  return LOG("record %ld %ld\n", (long)e, (long)s), OK;
}
int hipStreamWaitEvent(intptr_t s, intptr_t e, unsigned flags) {
  return (void)flags, LOG("wait %ld %ld\n", (long)s, (long)e), OK;
}

/* kernel<<<...>>> keeps its configuration here between the call and the stub that launches */
static dim3 grid_, block_;
static size_t lds_;
static intptr_t stream_;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, intptr_t s) {
  return grid_ = grid, block_ = block, lds_ = lds, stream_ = s, OK;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, intptr_t* s) {
  return *grid = grid_, *block = block_, *lds = lds_, *s = stream_, OK;
}
/* the library's kernels, as its constructor registers them */
static struct {
  const void* f;
  const char* name;
} kernels[1024];
static int n_kernels;
void __hipRegisterFunction(void** modules, const void* f, char* device_function, const char* name, unsigned threads, void* tid,
                           void* bid, void* block, void* grid, int* wave_size) {
  (void)modules, (void)device_function, (void)threads, (void)tid, (void)bid, (void)block, (void)grid, (void)wave_size;
  if (n_kernels < 1024) kernels[n_kernels].f = f, kernels[n_kernels++].name = name;
}
const char* hr_kernel(int i) { return i < n_kernels ? kernels[i].name : 0; }
static const char* name_of(const void* f) {
  for (int i = 0; i < n_kernels; i++)
    if (kernels[i].f == f) return kernels[i].name;
  return "?";
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, intptr_t s) {
  (void)args;
  if (++launches == hr_fail_launch) return LOG("launch_failed %ld\n", (long)s), INVALID;
  return LOG("launch %ld %u %u %zu %s\n", (long)s, grid.x, block.x, lds, name_of(f)), OK;
}
