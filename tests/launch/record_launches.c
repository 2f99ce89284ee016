// Stands in for the HIP runtime's launch calls in a process without a GPU: a launch is written down and not carried out.  Loaded
// ahead of the library with global symbols, so that the library's calls bind to these.
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { dim3_t grid, block; size_t lds; void* stream; } config_t;

static _Thread_local config_t g_config;
enum { kMax = 256 };
static uint32_t g_launches[kMax][6];
static int g_count;
static const char* g_launched[kMax];  // names of the kernels launched
static struct { const void* host; const char* name; } g_kernels[kMax];  // the library's own, as it registers them
static int g_registered;

void __hipRegisterFunction(void** module, const void* host, char* device, const char* name, unsigned threads, void* tid, void* bid,
                           dim3_t* block, dim3_t* grid, int* warp) {
  (void)module; (void)device; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
  if (strncmp(name, "_ZN2sb", 6) == 0 && g_registered < kMax) {
    g_kernels[g_registered].host = host;
    g_kernels[g_registered++].name = name;
  }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  g_config.grid = grid; g_config.block = block; g_config.lds = lds; g_config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
  return 0;
}
int hipLaunchKernel(const void* kernel, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)args; (void)lds; (void)stream;
  if (g_count < kMax) {
    uint32_t* l = g_launches[g_count];
    l[0] = grid.x; l[1] = grid.y; l[2] = grid.z; l[3] = block.x; l[4] = block.y; l[5] = block.z;
    g_launched[g_count] = "";
    for (int i = 0; i < g_registered; ++i)
      if (g_kernels[i].host == kernel) g_launched[g_count] = g_kernels[i].name;
  }
  ++g_count;
  return 0;
}
int hipGetLastError(void) { return 0; }

// number of launches so far; `out` takes the first kMax of them, grid and block sizes
int recorded_launches(uint32_t* out) {
  for (int i = 0; i < g_count && i < kMax; ++i)
    for (int a = 0; a < 6; ++a) out[6 * i + a] = g_launches[i][a];
  return g_count;
}
// name of the kernel of launch i < kMax, as the compiler mangled it
const char* recorded_kernel(int i) { return g_launched[i]; }
