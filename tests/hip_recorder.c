/* A stand-in for the HIP runtime calls that libscmoe makes: it runs nothing and writes down, one
 * line per call, what would have been enqueued on which stream.  Loaded ahead of libscmoe in a
 * process without a GPU, it shows the launches of a library call, their grids and their order. */
#include <stdint.h>
#include <stdio.h>

typedef struct { uint32_t x, y, z; } dim3_t;

static char text[1 << 20];
static size_t used;
#define LOG(...)                                                                    \
  do {                                                                              \
    int n_ = snprintf(text + used, sizeof text - used, __VA_ARGS__);                \
    if (n_ > 0 && used + (size_t)n_ < sizeof text) used += (size_t)n_;              \
  } while (0)

const char* recorder_text(void) { return text; }
void recorder_reset(void) { used = 0; text[0] = 0; }

static struct { const void* stub; const char* name; } kernels[1024];
static int nkernels;
static struct { dim3_t grid, block; size_t lds; void* stream; } pushed;

void** __hipRegisterFatBinary(const void* data) { static void* h; (void)data; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* stub, char* dev, const char* name, unsigned lim, void* a, void* b, void* c,
                           void* d, int* e) {
  (void)h; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)e;
  if (nkernels < 1024) { kernels[nkernels].stub = stub; kernels[nkernels++].name = name; }
}
void __hipRegisterVar(void** h, void* var, char* dev, char* name, int ext, size_t size, int cst, int glob) {
  (void)h; (void)var; (void)dev; (void)name; (void)ext; (void)size; (void)cst; (void)glob;
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* stream) {
  const char* name = "?";
  (void)args;
  for (int i = 0; i < nkernels; ++i)
    if (kernels[i].stub == f) name = kernels[i].name;
  LOG("kernel %p %s %u %u %u %u %u %u %zu\n", stream, name, g.x, g.y, g.z, b.x, b.y, b.z, lds);
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int kind, void* stream) {
  (void)kind;
  LOG("copy %p %p %p %zu\n", stream, dst, src, bytes);
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned flags) {
  static uintptr_t next = 0x100;
  (void)flags;
  *e = (void*)next++;
  return 0;
}
int hipEventRecord(void* e, void* stream) { LOG("record %p %p\n", stream, e); return 0; }
int hipStreamWaitEvent(void* stream, void* e, unsigned flags) { (void)flags; LOG("wait %p %p\n", stream, e); return 0; }
int hipStreamSynchronize(void* stream) { LOG("sync %p\n", stream); return 0; }
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int attr, int v) { (void)f; (void)attr; (void)v; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* sym) { (void)sym; *p = (void*)0x7000000; return 0; }
