// A stand-in for the HIP runtime that runs no kernel: device memory is host memory, launches are counted by kernel and a
// virtual clock advances by a cost of each launch. An executable's own symbols come before those of the
// libraries it loads, so the solver's library, opened below, calls these. The program then makes one scenario's calls
// (argv[2]) of the solver's C interface and prints what the runtime saw.
//   tuned NX NY COUNT ROWS: an autotuned batch of COUNT instances on a device where a launch of more than ROWS rows per march
//       is the slower the more, and one of fewer the slower the fewer; then a second batch of the class; prints the rows
//       returned, the wavefronts of a run's stage and those of the rows returned, for both
//   batch STEPS ...: runs of these lengths of one batch; prints for each the stages launched directly, graph launches and the
//       stages that those replayed
#include <dlfcn.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "swe_hweno.h"

struct Dim3 { uint32_t x, y, z; };
struct Graph { long stages; };

static std::map<const void*, std::string> names;
static Dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
static bool capturing = false;
static long captured = 0, direct = 0, graph_launches = 0, replayed = 0;
static unsigned last_waves = 0;
static double now_ms = 0.0;
static std::map<void*, double> event_ms;
static double (*cost)(unsigned waves) = nullptr;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char* device, const char*, unsigned, void*, void*, void*, void*, int*) {
  names[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s) {
  cfg_grid = g; cfg_block = b; cfg_lds = lds; cfg_stream = s;
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s) {
  *g = cfg_grid; *b = cfg_block; *lds = cfg_lds; *s = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3, void**, size_t, void*) {
  if (names[f].find("k_batch_stage") == std::string::npos) return 0;
  if (capturing) { ++captured; return 0; }
  ++direct;
  last_waves = g.x;
  if (cost) now_ms += cost(g.x);
  return 0;
}
int hipMalloc(void** p, size_t n) { return (*p = std::calloc(1, n)) ? 0 : 2; }
int hipFree(void* p) { std::free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { std::memcpy(d, s, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { std::memset(d, v, n); return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetDevicePropertiesR0600(void* p, int) { std::memset(p, 0, 1024); return 0; }  // the architecture's name is empty
int hipStreamCreateWithFlags(void** s, unsigned) { *s = std::malloc(1); return 0; }
int hipStreamDestroy(void* s) { std::free(s); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamBeginCapture(void*, int) { capturing = true; captured = 0; return 0; }
int hipStreamEndCapture(void*, void** g) { capturing = false; *g = new Graph{captured}; return 0; }
int hipGraphInstantiate(void** e, void* g, void*, char*, size_t) { *e = new Graph(*(Graph*)g); return 0; }
int hipGraphDestroy(void* g) { delete (Graph*)g; return 0; }
int hipGraphExecDestroy(void* g) { delete (Graph*)g; return 0; }
int hipGraphLaunch(void* g, void*) { ++graph_launches; replayed += ((Graph*)g)->stages; return 0; }
int hipEventCreate(void** e) { *e = std::malloc(1); return 0; }
int hipEventDestroy(void* e) { std::free(e); return 0; }
int hipEventRecord(void* e, void*) { event_ms[e] = now_ms; return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = (float)(event_ms[b] - event_ms[a]); return 0; }
}

static std::vector<double> plane(64 * 64 * 9, 1.0);

static swe_hweno_instance instance(int nx, int ny) {
  swe_hweno_instance i{};
  i.nx = nx; i.ny = ny; i.x1 = i.y1 = 1.0;
  i.b = i.bx = i.by = plane.data();
  i.state = plane.data();
  return i;
}

static int nx, ny, count;
static double fast_rows;
static unsigned waves_of(int rows) { return (unsigned)(count * ((nx + 59) / 60) * ((ny + rows - 1) / rows)); }
static double away(unsigned waves) {  // how far the launch's marches are from the fast ones
  const double rows = (double)count * ((nx + 59) / 60) * ny / waves;
  return rows > fast_rows ? rows / fast_rows : fast_rows / rows;
}

int main(int argc, char** argv) {
  void* lib = argc > 2 ? dlopen(argv[1], RTLD_NOW | RTLD_LOCAL) : nullptr;
  if (!lib) { std::fprintf(stderr, "%s\n", argc > 2 ? dlerror() : "usage"); return 2; }
  const auto init = (decltype(&swe_hweno_batch_init))dlsym(lib, "swe_hweno_batch_init");
  const auto run = (decltype(&swe_hweno_batch_run))dlsym(lib, "swe_hweno_batch_run");
  const auto tune = (decltype(&swe_hweno_batch_autotune))dlsym(lib, "swe_hweno_batch_autotune");
  const auto destroy = (decltype(&swe_hweno_batch_destroy))dlsym(lib, "swe_hweno_batch_destroy");
  swe_hweno_params p{};
  p.dim = 2; p.nx = p.ny = 4; p.x1 = p.y1 = 1.0; p.g = 9.812; p.cfl = 0.6; p.eps = 1e-6;
  const std::string what = argv[2];
  if (what == "tuned") {
    nx = std::atoi(argv[3]); ny = std::atoi(argv[4]); count = std::atoi(argv[5]); fast_rows = std::atof(argv[6]);
    std::vector<swe_hweno_instance> v(count, instance(nx, ny));
    for (int k = 0; k < 2; ++k) {
      swe_hweno_batch* bt = nullptr;
      int rows = 0;
      if (init(&p, v.data(), count, nullptr, &bt)) return 3;
      cost = away;
      if (tune(bt, &rows)) return 4;
      cost = nullptr;
      if (run(bt, 1, nullptr)) return 5;
      std::printf("%d %u %u\n", rows, last_waves, waves_of(rows));
      destroy(bt);
    }
  } else {
    const swe_hweno_instance one = instance(32, 32);
    swe_hweno_batch* bt = nullptr;
    if (init(&p, &one, 1, nullptr, &bt)) return 3;
    for (int k = 3; k < argc; ++k) {
      direct = graph_launches = replayed = 0;
      if (run(bt, std::atoi(argv[k]), nullptr)) return 5;
      std::printf("%ld %ld %ld\n", direct, graph_launches, replayed);
    }
    destroy(bt);
  }
  return 0;
}
