// MI355X (gfx950) implementation of the C ABI in include/swe_hweno.h: the right-hand side of the
// well-balanced fifth-order finite-difference HWENO scheme for the shallow water equations, its
// derivative limiter and SSP-RK3 stages (Zhao & Zhang, arXiv 2208.01260), in FP64 or FP32 (the
// same kernels instantiated for both types).
//
// Kernel design (the kernels of the scheme are in hweno_stage.inc, included once per arithmetic type):
//   * k_stage, one wavefront per workgroup, is the whole stage of eq. (2.11) in one pass: each lane owns one grid
//     column and marches up a strip of rows. The y-sweep keeps a four-row window of raw node records in
//     registers and carries the interface flux of the previous row, so each y-interface is
//     computed once. The x-sweep exchanges the current row between lanes through LDS: lane l
//     computes the interface left of its column and reads the right one from lane l+1. A wave
//     covers 64 columns (2 halo columns each side) and writes the 60 interior ones.
//   * k_small is the same stage for 2D grids too small to fill the GPU with marches: a workgroup shares out the interfaces
//     and limiters of a few rows. k_line is a whole 1D run in one launch where the grid fits a workgroup.
//   * The stage kernels write the bare right-hand side (MODE_RHS), or fuse the time step, the limiter of
//     Sec. 2.2 at the node, the Runge-Kutta combination and the max-reduction of the next
//     stage's Lax-Friedrichs speeds (MODE_STAGE0/1/2).
//   * Boundary nodes are read through an index fold: periodic wrap, or the mirror about the wall
//     face with each field's parity.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>
#include <algorithm>
#include <cstdio>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "swe_hweno.h"

namespace swe {

constexpr int WAVE = 64;
constexpr int OUT_COLS = WAVE - 4;  // interior columns written per wave
constexpr int ROWS_DEFAULT = 32;    // rows marched per wave unless tuned

enum { MODE_RHS = 0, MODE_STAGE0 = 1, MODE_STAGE1 = 2, MODE_STAGE2 = 3 };
enum { ERR_DRY = 1, ERR_NONFINITE = 2 };

// Device scalars of a context.
struct DevScal {
  double dt, t, t_end, pad0;
  int active, steps, err;
  int err0;  // batch: what the first stage of the running step met (see step_start)
};

// A set of Lax-Friedrichs speeds: (alpha_x, alpha_y) (bits of positive doubles) in each of
// a power-of-two number of slots, one 128-byte line per slot; the set's value is the maximum over
// its slots. Atomics on one address are served one after another, 8.6 ns apart on this device when they come
// from all XCDs: with a single slot the wavefronts that end together queue there (k_alpha
// over 1021 x 777 nodes took 284 us for 25 MB). Spread over 64 lines the same reduction is bound by its
// reads again. A reader loads one slot per lane and takes the maximum over the wavefront.
constexpr int ASTRIDE = 16;  // 64-bit words per slot
constexpr int ASLOTS = 64;   // slots of a context's sets
constexpr int ASET = ASLOTS * ASTRIDE;
// alpha of U^n, U^(1), U^(2), fixed, and of a bare right-hand side. A stage reads one of the first three,
// fills the next and clears the one before: nothing else touches that one while it runs.
enum { SP_N = 0, SP_1, SP_2, SP_FIX, SP_RHS, SP_SETS };

// Largest finite value of the arithmetic type.
template <class T> __device__ __forceinline__ constexpr T big_value();
template <> __device__ __forceinline__ constexpr double big_value<double>() { return DBL_MAX; }
template <> __device__ __forceinline__ constexpr float big_value<float>() { return FLT_MAX; }

__device__ __forceinline__ double bits2d(unsigned long long u) { return __longlong_as_double((long long)u); }

// CFL time step from the Lax-Friedrichs speeds, rounded operation by operation (no contraction)
// so that every wavefront and kernel that computes it gets the same bits.
__device__ __forceinline__ double cfl_step(int dim, double cfl, double ax, double ay, double dx, double dy) {
#pragma clang fp contract(off)
  return dim == 2 ? cfl / (ax / dx + ay / dy) : cfl / (ax / dx);
}

// Fold an index into [0, n): periodic wrap or mirror about the wall face (one fold suffices for
// the stencil halos; indices of halo lanes farther out are clamped, their results are unused).
__device__ __forceinline__ int fold(int i, int n, int bc, bool& refl) {
  refl = false;
  if (i < 0) {
    if (bc == SWE_BC_PERIODIC) i += n; else { i = -1 - i; refl = true; }
  } else if (i >= n) {
    if (bc == SWE_BC_PERIODIC) i -= n; else { i = 2 * n - 1 - i; refl = true; }
  }
  return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// A global pointer the compiler cannot see through. Fields are reached by bumping such a pointer
// by the field stride, so that the only loop-invariant scalar is the stride itself: without it the
// compiler keeps one hoisted 64-bit base per (array, field), about thirty scalar pairs, and spills
// them to vector-register lanes that are read back on every row.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* opq(T* p) {
  auto g = (__attribute__((address_space(1))) T*)p;
  asm("" : "+v"(g));
  return g;
}

// The largest value of a wavefront (all 64 lanes active), the same in every lane. Through the data-parallel
// primitives: shifts by 1, 2, 4, 8 within rows of 16, the rows' last lanes broadcast to the next rows, then lane 63. A
// lane without a source keeps its own value. (Six exchanges through LDS took about 0.4 us at the end and start of
// every wavefront.)
template <int CTRL>
__device__ __forceinline__ double dpp_max(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const int lo = (int)(unsigned)u, hi = (int)(unsigned)(u >> 32);
  const unsigned l2 = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
  const unsigned h2 = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
  return fmax(v, bits2d(((unsigned long long)h2 << 32) | l2));
}
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0x111>(v);
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  v = dpp_max<0x118>(v);
  v = dpp_max<0x142>(v);
  v = dpp_max<0x143>(v);
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, WAVE - 1);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), WAVE - 1);
  return bits2d(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ float wave_max(float v) { return (float)wave_max((double)v); }

// Error flags of a wavefront's lanes together.
__device__ __forceinline__ int wave_err(int e) {
  return (__ballot(e & ERR_DRY) ? ERR_DRY : 0) | (__ballot(e & ERR_NONFINITE) ? ERR_NONFINITE : 0);
}

// The two speeds of a set (all 64 lanes of a wavefront take part), in scalar registers. A grid of few
// wavefronts keeps one slot, which needs no reduction.
__device__ __forceinline__ double uniform(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return bits2d(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ void read_speeds(const unsigned long long* __restrict__ p, int amask, double& ax, double& ay) {
  if (amask == 0) {
    ax = bits2d(p[0]);
    ay = bits2d(p[1]);
    return;
  }
  const unsigned long long* q = p + (size_t)((int)(threadIdx.x & (WAVE - 1)) & amask) * ASTRIDE;
  ax = uniform(wave_max(bits2d(q[0])));
  ay = uniform(wave_max(bits2d(q[1])));
}

// Workgroups are handed to the 8 XCDs of the device round-robin by linear id. band_tile maps
// the linear id i < n of a workgroup to a tile index so that each XCD receives a contiguous
// band of tiles: neighbouring tiles, which read each other's halo columns and rows, then meet
// in the same L2 (at 4096^2 this takes the stage kernels' fetched bytes down by a fifth). It is
// a permutation of [0, n).
constexpr unsigned NXCD = 8;
__host__ __device__ __forceinline__ unsigned band_tile(unsigned i, unsigned n) {
  const unsigned x = i % NXCD, k = i / NXCD, q = n / NXCD, rm = n % NXCD;
  return x * q + (x < rm ? x : rm) + k;
}

// Set a set of ASLOTS speeds to given values (one wavefront).
__global__ void k_set_speeds(unsigned long long* p, unsigned long long v0, unsigned long long v1) {
  unsigned long long* q = p + (size_t)threadIdx.x * ASTRIDE;
  q[0] = threadIdx.x == 0 ? v0 : 0ull;
  q[1] = threadIdx.x == 0 ? v1 : 0ull;
}

// Reset the clock of a run or a single step (the error flag is left alone) and clear the sets of speeds
// of its stages. One wavefront.
__device__ __forceinline__ void reset_run(DevScal* s, unsigned long long* sp, double t_end, int l) {
  if (l == 0) { s->t = 0.0; s->t_end = t_end; s->dt = 0.0; s->active = 1; s->steps = 0; }
  unsigned long long* q = sp + (size_t)l * ASTRIDE;
  q[SP_1 * ASET] = q[SP_1 * ASET + 1] = q[SP_2 * ASET] = q[SP_2 * ASET + 1] = 0ull;
}
__global__ void k_reset(DevScal* s, unsigned long long* sp, double t_end) {
  reset_run(s, sp, t_end, (int)threadIdx.x);
  unsigned long long* q = sp + SP_N * ASET + (size_t)threadIdx.x * ASTRIDE;
  q[0] = q[1] = 0ull;
}


// Threads of a workgroup of k_start.
constexpr int START_THREADS = 1024;
// LDS of k_small at R rows per workgroup: the quantities and the task counter.
constexpr int NNODE = 18;  // slots of a node's fluxes
constexpr int SMALL_ROWS = 8;  // rows per workgroup at most
constexpr size_t small_lds_bytes(int R, size_t esz) { return WAVE * (R * NNODE + (R + 1) * 14 + R * 6) * esz + 16; }
static_assert(small_lds_bytes(SMALL_ROWS, sizeof(double)) <= 163840, "160 KB of LDS");

}  // namespace swe

// The scheme's routines and kernels, once per arithmetic type: the two differ in how products and sums become FMAs.
// Single precision contracts across statements (the compiler's choice per inlined copy); its results near
// a lake at rest are rounding amplified by 1/dx, so its arithmetic is kept as it is. Double precision contracts within an
// expression only (0.3% more FP64 instructions), so that every inlined copy of a routine rounds alike and all
// tilings give the same bits.
namespace swe32 { using namespace swe; }
#define SWE_NS swe32
#include "hweno_device.hpp"
#include "hweno_stage.inc"
#undef SWE_NS
#pragma clang fp contract(on)
#define SWE_NS swe
#include "hweno_device.hpp"
#include "hweno_stage.inc"
#undef SWE_NS
#pragma clang fp contract(fast)

#include "hweno_adjoint.hpp"

namespace swe {

__global__ void k_clear_err(DevScal* s) {
  if (threadIdx.x == 0) s->err = 0;
}

// Elementwise check of the arithmetic building blocks (rcp, sqrt_pos, div3).
__global__ __launch_bounds__(256) void k_math_check(int which, const double* __restrict__ x, double* __restrict__ y,
                                                    size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double v = x[i];
    y[i] = which == 0 ? rcp(v) : (which == 1 ? sqrt_pos(v) : div3(v));
  }
}

// Allocation-free step (swe_hweno_step_noalloc): its stage buffers and device scalars live in
// this array, one copy per GPU, held until the process ends. Host code takes its address with
// hipGetSymbolAddress (per device) and never uses the array's name as a device address.
constexpr size_t NOALLOC_BYTES = size_t(32) << 20;
constexpr size_t NOALLOC_SCAL = 256;  // DevScal at the start, stage planes after it
static_assert(sizeof(DevScal) <= NOALLOC_SCAL, "device scalars must fit their slot");
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];
static __device__ __align__(256) unsigned long long scratch_speeds[SP_SETS * ASET];

// The device scalars of a new context (or of an allocation-free step, whose array keeps whatever the
// previous call on this GPU left): the fixed speeds, everything else zero. One wavefront.
__global__ void k_setup(DevScal* s, unsigned long long* sp, unsigned long long afx, unsigned long long afy) {
  const int l = (int)threadIdx.x;
#pragma unroll
  for (int k = 0; k < SP_SETS; ++k) {
    unsigned long long* q = sp + (size_t)k * ASET + (size_t)l * ASTRIDE;
    q[0] = k == SP_FIX && l == 0 ? afx : 0ull;
    q[1] = k == SP_FIX && l == 0 ? afy : 0ull;
  }
  if (l == 0) {
    s->dt = s->t = s->t_end = s->pad0 = 0.0;
    s->active = s->steps = s->err = s->err0 = 0;
  }
}

}  // namespace swe

// =========================================================================== host runtime
using namespace swe;

struct swe_hweno_ctx {
  swe_hweno_params p{};
  int f32 = 0;                // arithmetic and storage type: 0 = double, 1 = float
  size_t esz = sizeof(double);
  hipStream_t stream = nullptr;
  hipStream_t cap = nullptr;  // capture stream for the per-step graphs
  int nf = 0, nd = 0;
  size_t n = 0;
  void* mem = nullptr;        // the one block of device memory that the pointers below point into
  bool own_mem = false;       // allocated here (else the caller's)
  void *b = nullptr, *bx = nullptr, *by = nullptr;  // planes of the context's type
  void *S1 = nullptr, *S2 = nullptr, *Dn = nullptr;
  DevScal* sc = nullptr;
  unsigned long long* sp = nullptr;  // SP_SETS sets of speeds
  hipGraphExec_t g1 = nullptr, g8 = nullptr;
  const void* g_state = nullptr;
  int g_tend = 0;
  long g_steps = 0;  // steps launched on g_state before its graphs were captured
  unsigned cus = 256;       // compute units of the device
  int rows = ROWS_DEFAULT;  // rows marched per wave (2D), chosen at init
  int small = 0;            // 2D: rows per workgroup of k_small, or 0 for marching wavefronts
  int line = 0;             // 1D: wavefronts of k_line's workgroup, or 0 for a launch per stage
  // kernel timing: event pairs around stage kernels (slot 0 = bare right-hand side, 1..3 = stages)
  bool timing = false;
  struct Pending { hipEvent_t a, b; int slot; };
  std::vector<Pending> pending;
  std::vector<hipEvent_t> pool;
  double ms[4] = {0, 0, 0, 0};
  long long launches[4] = {0, 0, 0, 0};
  void* adj = nullptr;  // work buffers of the adjoint, allocated on first use
};

void swe_adj_release(swe_hweno_ctx* c);

namespace {

bool params_ok(const swe_hweno_params* p) {
  if (!p) return false;
  if (p->dim != 1 && p->dim != 2) return false;
  if (p->nx < 4 || p->nx > (1 << 20)) return false;
  if (p->dim == 2 && (p->ny < 4 || p->ny > (1 << 20))) return false;
  if (p->dim == 1 && p->ny != 1) return false;
  if ((size_t)p->nx * (size_t)p->ny > ((size_t)1 << 31)) return false;
  if (!(p->x1 > p->x0) || (p->dim == 2 && !(p->y1 > p->y0))) return false;
  // finite domain whose node spacing and its reciprocal are finite and positive
  const auto spacing_ok = [](double a, double b, int n) {
    const double d = (b - a) / n;
    return std::isfinite(a) && std::isfinite(b) && d > 0 && std::isfinite(d) && std::isfinite(1.0 / d);
  };
  if (!spacing_ok(p->x0, p->x1, p->nx) || (p->dim == 2 && !spacing_ok(p->y0, p->y1, p->ny))) return false;
  // eps >= 1e-20: the kernels form products of two or three weight sums, each at least of
  // order eps^4, and these stay normal doubles down to that floor
  if (!(p->g > 0) || !(p->cfl > 0) || !(p->eps >= 1e-20)) return false;
  if (!std::isfinite(p->g) || !std::isfinite(p->cfl) || !std::isfinite(p->eps)) return false;
  if (p->bc_x < 0 || p->bc_x > 1 || p->bc_y < 0 || p->bc_y > 1) return false;
  if (p->flags & ~(SWE_FIXED_DT | SWE_FIXED_ALPHA | SWE_NO_LIMITER | SWE_CHECK_DRY)) return false;
  if ((p->flags & SWE_FIXED_DT) && !(p->fixed_dt > 0 && p->fixed_dt <= DBL_MAX)) return false;
  if ((p->flags & SWE_FIXED_ALPHA) &&
      (!(p->alpha_x > 0 && p->alpha_x <= DBL_MAX) || (p->dim == 2 && !(p->alpha_y > 0 && p->alpha_y <= DBL_MAX))))
    return false;
  return true;
}

unsigned long long dbits(double v) {
  unsigned long long u;
  std::memcpy(&u, &v, sizeof u);
  return u;
}

template <class T> using KArgsOf = std::conditional_t<sizeof(T) == 8, swe::KArgs<T>, swe32::KArgs<T>>;
// The kernels of an arithmetic type's namespace.
template <class T> struct Kern;
template <> struct Kern<double> {
  template <int DIM, int MODE> static constexpr auto stage = swe::k_stage<double, DIM, MODE>;
  template <int DIM> static constexpr auto start = swe::k_start<double, DIM>;
  template <int DIM> static constexpr auto alpha = swe::k_alpha<double, DIM>;
  template <int DIM> static constexpr auto limit = swe::k_limit<double, DIM>;
};
template <> struct Kern<float> {
  template <int DIM, int MODE> static constexpr auto stage = swe32::k_stage<float, DIM, MODE>;
  template <int DIM> static constexpr auto start = swe32::k_start<float, DIM>;
  template <int DIM> static constexpr auto alpha = swe32::k_alpha<float, DIM>;
  template <int DIM> static constexpr auto limit = swe32::k_limit<float, DIM>;
};

template <class T> bool is_type(const swe_hweno_ctx* c) { return c->f32 == (sizeof(T) == sizeof(float) ? 1 : 0); }

dim3 stage_grid(const swe_hweno_ctx* c) {
  const unsigned gx = (unsigned)((c->p.nx + OUT_COLS - 1) / OUT_COLS);
  const int rows = c->small ? c->small : c->rows;
  const unsigned gy = c->p.dim == 2 ? (unsigned)((c->p.ny + rows - 1) / rows) : 1u;
  return dim3(gx, gy, 1);
}

unsigned long long* speeds_set(const swe_hweno_ctx* c, int set) { return c->sp + (size_t)set * ASET; }

// Slots in use, less one: one slot up to 48 wavefronts in a stage (their atomics queue for under 1 us, about
// what reading and reducing 64 slots costs each of a step's kernels), else all.
int speeds_mask(const swe_hweno_ctx* c) {
  const dim3 g = stage_grid(c);
  return g.x * g.y <= 48 ? 0 : ASLOTS - 1;
}

template <class T> KArgsOf<T> base_args(const swe_hweno_ctx* c) {
  KArgsOf<T> a;
  std::memset(&a, 0, sizeof a);
  a.b = (const T*)c->b; a.bx = (const T*)c->bx; a.by = (const T*)c->by;
  a.sc = c->sc;
  a.amask = speeds_mask(c);
  a.nx = c->p.nx; a.ny = c->p.dim == 2 ? c->p.ny : 1;
  a.bcx = c->p.bc_x; a.bcy = c->p.bc_y;
  a.limiter = (c->p.flags & SWE_NO_LIMITER) ? 0 : 1;
  const double dx = (c->p.x1 - c->p.x0) / c->p.nx;
  const double dy = c->p.dim == 2 ? (c->p.y1 - c->p.y0) / c->p.ny : 1.0;
  a.dx = T(dx); a.dy = T(dy);
  a.idx = T(1.0 / dx); a.idy = T(1.0 / dy);
  a.g = T(c->p.g); a.eps = T(c->p.eps);
  a.rows = c->small ? c->small : c->rows;
  a.cfl = c->p.cfl; a.fdt = c->p.fixed_dt; a.cdx = dx; a.cdy = dy;
  a.fixed_dt = (c->p.flags & SWE_FIXED_DT) ? 1 : 0;
  return a;
}

// Speeds read, filled and cleared by the stages of a step (the first stage also forms the step from those of U^n).
template <class A> void stage_speeds(const swe_hweno_ctx* c, A& a, int stage) {
  const bool fa = (c->p.flags & SWE_FIXED_ALPHA) != 0;
  a.a_in = speeds_set(c, fa ? SP_FIX : stage);
  a.a_out = speeds_set(c, (stage + 1) % 3);
  a.a_clear = speeds_set(c, (stage + 2) % 3);
  a.a_n = speeds_set(c, SP_N);
}

template <class T, int MODE> void launch_stage_mode(const swe_hweno_ctx* c, const KArgsOf<T>& a, hipStream_t s) {
  if constexpr (sizeof(T) == 8) if (c->small) {
    const size_t lds = small_lds_bytes(c->small, sizeof(T));
    if (c->small == 1) hipLaunchKernelGGL((swe::k_small<T, MODE, 4, true>), stage_grid(c), dim3(4 * WAVE), lds, s, a);
    else if (c->small == 2) hipLaunchKernelGGL((swe::k_small<T, MODE, 8, true>), stage_grid(c), dim3(8 * WAVE), lds, s, a);
    else hipLaunchKernelGGL((swe::k_small<T, MODE, 8, false>), stage_grid(c), dim3(8 * WAVE), lds, s, a);
    return;
  }
  if (c->p.dim == 2) hipLaunchKernelGGL((Kern<T>::template stage<2, MODE>), stage_grid(c), dim3(WAVE), 0, s, a);
  else hipLaunchKernelGGL((Kern<T>::template stage<1, MODE>), stage_grid(c), dim3(WAVE), 0, s, a);
}

// Speeds of a state into a set; with begin (set SP_N), at the start of a run or step whose clock it resets.
template <class T> void launch_alpha(const swe_hweno_ctx* c, const T* S, int set, bool begin, double t_end, hipStream_t s) {
  const T* b = (const T*)c->b;
  const int amask = speeds_mask(c);
  // one launch while a workgroup has at most four nodes per thread (in one slot at most 16): at 400^2 4.9 us
  // against 4.5 + 5.4 us of the two launches
  const size_t most = amask ? (size_t)4 * ASLOTS * START_THREADS : (size_t)16 * START_THREADS;
  if (c->n <= most) {
    const size_t blocks = amask ? std::min<size_t>((c->n + START_THREADS - 1) / START_THREADS, ASLOTS) : 1;
    if (c->p.dim == 2)
      hipLaunchKernelGGL((Kern<T>::template start<2>), dim3((unsigned)blocks), dim3(START_THREADS), 0, s, S, b, c->n, T(c->p.g), c->sp,
                         set, c->sc, begin ? 1 : 0, t_end);
    else
      hipLaunchKernelGGL((Kern<T>::template start<1>), dim3((unsigned)blocks), dim3(START_THREADS), 0, s, S, b, c->n, T(c->p.g), c->sp,
                         set, c->sc, begin ? 1 : 0, t_end);
    return;
  }
  unsigned long long* out = speeds_set(c, set);
  if (begin) hipLaunchKernelGGL(k_reset, dim3(1), dim3(ASLOTS), 0, s, c->sc, c->sp, t_end);
  else hipLaunchKernelGGL(k_set_speeds, dim3(1), dim3(ASLOTS), 0, s, out, 0ull, 0ull);
  // a node per thread up to eight workgroups per CU, which fill the memory system; each ends in one pair of atomics
  const size_t blocks = (c->n + 255) / 256;
  const unsigned grid = (unsigned)(blocks < 2048 ? blocks : 2048);
  if (c->p.dim == 2)
    hipLaunchKernelGGL((Kern<T>::template alpha<2>), dim3(grid), dim3(256), 0, s, S, b, c->n, T(c->p.g), out, amask, &c->sc->err);
  else
    hipLaunchKernelGGL((Kern<T>::template alpha<1>), dim3(grid), dim3(256), 0, s, S, b, c->n, T(c->p.g), out, amask, &c->sc->err);
}

hipEvent_t take_event(swe_hweno_ctx* c) {
  if (!c->pool.empty()) {
    hipEvent_t e = c->pool.back();
    c->pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Start / end an event-timed region on the context stream (no-op unless timing is on).
int time_begin(swe_hweno_ctx* c, hipStream_t s) {
  if (!c || !c->timing || s != c->stream) return -1;
  hipEvent_t a = take_event(c), b = take_event(c);
  if (!a || !b) return -1;
  (void)hipEventRecord(a, s);
  c->pending.push_back({a, b, -1});
  return (int)c->pending.size() - 1;
}
void time_end(swe_hweno_ctx* c, int id, int slot, hipStream_t s) {
  if (id < 0) return;
  (void)hipEventRecord(c->pending[id].b, s);
  c->pending[id].slot = slot;
}

// Accumulate finished event pairs (the stream must have been synchronised).
void collect_timing(swe_hweno_ctx* c) {
  for (const auto& pe : c->pending) {
    float ms = 0.f;
    if (pe.slot >= 0 && hipEventElapsedTime(&ms, pe.a, pe.b) == hipSuccess) {
      c->ms[pe.slot] += ms;
      c->launches[pe.slot] += 1;
    }
    c->pool.push_back(pe.a);
    c->pool.push_back(pe.b);
  }
  c->pending.clear();
}

// nsteps steps of a 1D grid in one launch (rhs null), or its right-hand side with given speeds (alpha > 0) or the state's.
void launch_line(const swe_hweno_ctx* c, double* state, double* rhs, int nsteps, bool begin, int use_tend, double t_end,
                 double alpha, hipStream_t s) {
  swe::LineArgs<double> a;
  std::memset(&a, 0, sizeof a);
  a.state = state; a.rhs = rhs;
  a.b = (const double*)c->b; a.bx = (const double*)c->bx;
  a.sc = c->sc;
  a.nx = c->p.nx; a.bc = c->p.bc_x;
  a.limiter = (c->p.flags & SWE_NO_LIMITER) ? 0 : 1;
  a.nsteps = nsteps; a.begin = begin ? 1 : 0; a.use_tend = use_tend;
  a.fixed_dt = (c->p.flags & SWE_FIXED_DT) ? 1 : 0;
  a.fixed_alpha = rhs ? alpha > 0 : (c->p.flags & SWE_FIXED_ALPHA) != 0;
  a.alpha = rhs ? alpha : c->p.alpha_x;
  a.t_end = t_end; a.cfl = c->p.cfl; a.fdt = c->p.fixed_dt;
  a.cdx = (c->p.x1 - c->p.x0) / c->p.nx;
  a.dx = a.cdx; a.idx = 1.0 / a.cdx; a.g = c->p.g; a.eps = c->p.eps;
  if (rhs) hipLaunchKernelGGL((swe::k_line<double, true>), dim3(1), dim3(c->line * WAVE), 0, s, a);
  else hipLaunchKernelGGL((swe::k_line<double, false>), dim3(1), dim3(c->line * WAVE), 0, s, a);
}

// One step on stream s: three fused stages; U^n is `state`, updated in place.
// With timing on (direct launches only) every stage kernel is bracketed by an event pair.
template <class T> void enqueue_step(swe_hweno_ctx* c, T* state, int use_tend, hipStream_t s) {
  KArgsOf<T> base = base_args<T>(c);
  base.use_tend = use_tend;
  T* S1 = (T*)c->S1;
  T* S2 = (T*)c->S2;
  T* Dn = (T*)c->Dn;
  KArgsOf<T> a = base;
  stage_speeds(c, a, 0);
  a.S = state; a.out = S1; a.Dn_out = Dn;
  int id = time_begin(c, s);
  launch_stage_mode<T, MODE_STAGE0>(c, a, s);
  time_end(c, id, 1, s);
  a = base;
  stage_speeds(c, a, 1);
  a.S = S1; a.Sn = state; a.Dn = Dn; a.out = S2;
  id = time_begin(c, s);
  launch_stage_mode<T, MODE_STAGE1>(c, a, s);
  time_end(c, id, 2, s);
  a = base;
  stage_speeds(c, a, 2);
  a.S = S2; a.Sn = state; a.Dn = Dn; a.out = state;
  id = time_begin(c, s);
  launch_stage_mode<T, MODE_STAGE2>(c, a, s);
  time_end(c, id, 3, s);
}

int hip_status(hipError_t e) { return e == hipSuccess ? SWE_OK : SWE_EHIP; }

// Rows marched per wave in 2D: the wave count gx * ceil(ny / rows) should fill whole rounds of
// the SIMDs, while each march repays its start-up (four window rows and one extra y-interface,
// about two rows of work). Cost model: rounds * (rows + 2) over 3 .. 128 rows; ties go to fewer
// rows. Small grids, which cannot fill the GPU, get short marches and so more wavefronts; below 3
// rows the start-up of each wavefront costs more than the extra wavefronts gain. In double precision a SIMD holds one
// wavefront. In single precision it holds two, whose rows take 6.1 us together against 3.9 us of one alone
// (2048^2): a round is 2 wavefronts per SIMD at 1.54, its rest counts 1 or 1.54. (At 2048^2 36 rows, 1995 wavefronts, in
// place of 71 rows, 1015: 275 -> 220 us a stage; the rows change no bit.) SWE_HWENO_ROWS overrides the choice.
int choose_rows(int nx, int ny, int simds, bool two) {
  if (const char* e = std::getenv("SWE_HWENO_ROWS")) {
    const int r = std::atoi(e);
    if (r >= 1 && r <= 4096) return r;
  }
  const long gx = (nx + OUT_COLS - 1) / OUT_COLS;
  int best = ROWS_DEFAULT;
  double best_cost = 1e300;
  for (int r = 3; r <= 128; ++r) {
    const long waves = gx * ((ny + r - 1) / r);
    double rounds;
    if (two) {
      const long full = waves / (2L * simds), rest = waves % (2L * simds);
      rounds = 1.54 * (double)full + (rest == 0 ? 0.0 : (rest <= simds ? 1.0 : 1.54));
    } else {
      rounds = (double)((waves + simds - 1) / simds);
    }
    const double cost = rounds * (double)(std::min(r, ny) + 2);
    if (cost < best_cost * (1 - 1e-12)) { best_cost = cost; best = r; }
  }
  return best;
}

// Rows per workgroup of k_small, or 0 for marching wavefronts: the fewest for which every workgroup is resident at
// once, one per CU, up to 8 (their LDS). With one row a workgroup has 4 wavefronts, one per SIMD, else 8. A further
// row costs about 1.5 us, from 6.8 us at one row to 17.6 at 8; marching wavefronts take 18.8 us at their shortest marches, 20.6
// where this rule ends (about 340^2), and 21.9 at 400^2, where two rounds of 6 rows would take 28. Double
// precision only: in single precision (6.9 to 13.3 us against 16.9) the two tilings would round differently. A choice of
// rows by the environment keeps the marching wavefronts.
int choose_small(int nx, int ny, int cus) {
  if (std::getenv("SWE_HWENO_ROWS")) return 0;
  const long gx = (nx + OUT_COLS - 1) / OUT_COLS;
  for (int r = 1; r <= SMALL_ROWS; ++r)
    if (gx * ((ny + r - 1) / r) <= cus) return r;
  return 0;
}

// The tile of a context on the current device.
void choose_tile(swe_hweno_ctx* c) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
      hipSuccess || cus <= 0)
    cus = 256;
  c->cus = (unsigned)cus;
  c->rows = choose_rows(c->p.nx, c->p.dim == 2 ? c->p.ny : 1, 4 * cus, c->f32 != 0);
  c->small = c->p.dim == 2 && !c->f32 ? choose_small(c->p.nx, c->p.ny, cus) : 0;
  // a 1D grid that fits one workgroup runs in one launch (double precision: see the namespaces' contraction)
  const int waves = (c->p.nx + OUT_COLS - 1) / OUT_COLS;
  c->line = c->p.dim == 1 && !c->f32 && waves <= LINE_WAVES && !std::getenv("SWE_HWENO_ROWS") ? waves : 0;
}

// The device scalars in one copy (every copy to pageable memory costs a round trip), and the error they report,
// which is cleared.
int take_device_error(swe_hweno_ctx* c, DevScal* out = nullptr) {
  DevScal s;
  if (hipMemcpyAsync(&s, c->sc, sizeof s, hipMemcpyDeviceToHost, c->stream) != hipSuccess) return SWE_EHIP;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return SWE_EHIP;
  if (out) *out = s;
  if (s.err) {
    hipLaunchKernelGGL(k_clear_err, dim3(1), dim3(64), 0, c->stream, c->sc);
    if (hipStreamSynchronize(c->stream) != hipSuccess) return SWE_EHIP;
    return (s.err & ERR_NONFINITE) ? SWE_ENONFINITE : SWE_EDRY;
  }
  return SWE_OK;
}

void destroy_graphs(swe_hweno_ctx* c) {
  if (c->g1) hipGraphExecDestroy(c->g1);
  if (c->g8) hipGraphExecDestroy(c->g8);
  c->g1 = c->g8 = nullptr;
  c->g_state = nullptr;
}

template <class T> int capture(swe_hweno_ctx* c, T* state, int steps, int use_tend, hipGraphExec_t* out) {
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal) != hipSuccess) return SWE_EHIP;
  for (int k = 0; k < steps; ++k) enqueue_step<T>(c, state, use_tend, c->cap);
  if (hipStreamEndCapture(c->cap, &g) != hipSuccess || !g) return SWE_EHIP;
  const hipError_t e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  hipGraphDestroy(g);
  return hip_status(e);
}

// ------------------------------------------------------------------ typed bodies of the entry points
// Places in a context's block: the scalars, the sets of speeds and the planes, each on a boundary of 256 bytes.
struct CtxLayout { size_t sp, b, s1, s2, dn, bytes; };
CtxLayout ctx_layout(const swe_hweno_params* p, size_t esz) {
  const auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  const size_t plane = (size_t)p->nx * (size_t)(p->dim == 2 ? p->ny : 1) * esz, nf = p->dim == 2 ? 9 : 4;
  CtxLayout l;
  l.sp = up(sizeof(DevScal));
  l.b = up(l.sp + sizeof(unsigned long long) * SP_SETS * ASET);
  l.s1 = up(l.b + 3 * plane);
  l.s2 = up(l.s1 + nf * plane);
  l.dn = up(l.s2 + nf * plane);
  l.bytes = up(l.dn + (p->dim == 2 ? 6 : 2) * plane);
  return l;
}

// A context in `mem` (bytes of it), or in memory allocated here if mem is null.
template <class T>
int init_impl(const swe_hweno_params* p, const T* b, const T* bx, const T* by, void* stream, void* mem, size_t bytes,
              swe_hweno_ctx** out) {
  if (!out) return SWE_EINVAL;
  *out = nullptr;
  if (!params_ok(p) || !b || !bx || (p->dim == 2 && !by)) return SWE_EINVAL;
  // single precision: the weights, of order eps^4 where the data are flat, stay normal floats
  if (sizeof(T) == 4 && !(p->eps >= 1e-9)) return SWE_EINVAL;
  const CtxLayout at = ctx_layout(p, sizeof(T));
  if (mem && (bytes < at.bytes || (uintptr_t)mem % 256)) return SWE_EINVAL;
  swe_hweno_ctx* c = new (std::nothrow) swe_hweno_ctx();
  if (!c) return SWE_ENOMEM;
  c->p = *p;
  c->f32 = sizeof(T) == sizeof(float) ? 1 : 0;
  c->esz = sizeof(T);
  c->stream = (hipStream_t)stream;
  c->nf = p->dim == 2 ? 9 : 4;
  c->nd = p->dim == 2 ? 6 : 2;
  c->n = (size_t)p->nx * (size_t)(p->dim == 2 ? p->ny : 1);
  const size_t plane = c->n * sizeof(T);
  c->mem = mem;
  c->own_mem = mem == nullptr;
  if (!mem && hipMalloc(&c->mem, at.bytes) != hipSuccess) {
    c->mem = nullptr;
    swe_hweno_destroy(c);
    return SWE_ENOMEM;
  }
  char* base = (char*)c->mem;
  c->sc = (DevScal*)base;
  c->sp = (unsigned long long*)(base + at.sp);
  c->b = base + at.b;
  c->S1 = base + at.s1;
  c->S2 = base + at.s2;
  c->Dn = base + at.dn;
  c->bx = (T*)c->b + c->n;
  c->by = (T*)c->b + 2 * c->n;
  choose_tile(c);
  bool ok = hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking) == hipSuccess;
  ok = ok && hipMemcpyAsync(c->b, b, plane, hipMemcpyDeviceToDevice, c->stream) == hipSuccess;
  ok = ok && hipMemcpyAsync(c->bx, bx, plane, hipMemcpyDeviceToDevice, c->stream) == hipSuccess;
  if (p->dim == 2) ok = ok && hipMemcpyAsync(c->by, by, plane, hipMemcpyDeviceToDevice, c->stream) == hipSuccess;
  else ok = ok && hipMemsetAsync(c->by, 0, plane, c->stream) == hipSuccess;
  hipLaunchKernelGGL(k_setup, dim3(1), dim3(ASLOTS), 0, c->stream, c->sc, c->sp, dbits(p->alpha_x),
                     dbits(p->dim == 2 ? p->alpha_y : 0.0));
  ok = ok && hipGetLastError() == hipSuccess;
  ok = ok && hipStreamSynchronize(c->stream) == hipSuccess;
  if (!ok) { swe_hweno_destroy(c); return SWE_EHIP; }
  *out = c;
  return SWE_OK;
}

template <class T> int rhs_impl(swe_hweno_ctx* c, const T* state, T* rhs, double alpha_x, double alpha_y) {
  if (!c || !state || !rhs || state == rhs || !is_type<T>(c)) return SWE_EINVAL;
  // alpha_x < 0 asks for the state's speeds; otherwise alpha_x (and alpha_y in 2D) must be
  // finite and positive (NaN fails every comparison and is refused here)
  if (!(alpha_x < 0) && !(alpha_x > 0 && std::isfinite(alpha_x))) return SWE_EINVAL;
  if (alpha_x > 0 && c->p.dim == 2 && !(alpha_y > 0 && std::isfinite(alpha_y))) return SWE_EINVAL;
  const size_t bytes = c->n * c->nf * sizeof(T);
  if ((const char*)rhs < (const char*)state + bytes && (const char*)state < (const char*)rhs + bytes) return SWE_EINVAL;
  if constexpr (sizeof(T) == 8) if (c->line && !c->timing) {
    launch_line(c, const_cast<double*>(state), rhs, 0, false, 0, 0.0, alpha_x, c->stream);
    if (hipGetLastError() != hipSuccess) return SWE_EHIP;
    return (c->p.flags & SWE_CHECK_DRY) ? take_device_error(c) : SWE_OK;
  }
  if (alpha_x < 0) launch_alpha<T>(c, state, SP_RHS, false, 0.0, c->stream);
  else
    hipLaunchKernelGGL(k_set_speeds, dim3(1), dim3(ASLOTS), 0, c->stream, speeds_set(c, SP_RHS), dbits(alpha_x),
                       dbits(c->p.dim == 2 ? alpha_y : 0.0));
  KArgsOf<T> a = base_args<T>(c);
  a.S = state; a.out = rhs; a.a_in = speeds_set(c, SP_RHS);
  const int id = time_begin(c, c->stream);
  launch_stage_mode<T, MODE_RHS>(c, a, c->stream);
  time_end(c, id, 0, c->stream);
  if (hipGetLastError() != hipSuccess) return SWE_EHIP;
  return (c->p.flags & SWE_CHECK_DRY) ? take_device_error(c) : SWE_OK;
}

template <class T> int limit_impl(swe_hweno_ctx* c, const T* state, T* dmod) {
  if (!c || !state || !dmod || !is_type<T>(c)) return SWE_EINVAL;
  if constexpr (sizeof(T) == 8) if (c->p.dim == 2) {
    const KArgs<double> k = base_args<double>(c);
    swe::LimitArgs<double> a{state, k.b, dmod, k.nx, k.ny, k.bcx, k.bcy, 6, k.dx, k.dy, k.idx, k.idy, k.g, k.eps};
    while (a.lw > 2 && (1 << (a.lw - 1)) >= a.nx) --a.lw;  // 64 nodes wide, narrower where the grid is
    const size_t w = (size_t)1 << a.lw, h = 256 >> a.lw;
    const size_t tiles = ((size_t)a.nx + w - 1) / w * (((size_t)a.ny + h - 1) / h);
    hipLaunchKernelGGL(swe::k_limit_tile<double>, dim3((unsigned)tiles), dim3(256), 0, c->stream, a);
    return hip_status(hipGetLastError());
  }
  KArgsOf<T> a = base_args<T>(c);
  a.S = state; a.out = dmod;
  const size_t blocks = (c->n + 255) / 256;
  const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
  if constexpr (sizeof(T) == 4) if (c->p.dim == 2) {
    hipLaunchKernelGGL((Kern<T>::template limit<2>), dim3(grid), dim3(256), 0, c->stream, a);
    return hip_status(hipGetLastError());
  }
  hipLaunchKernelGGL((Kern<T>::template limit<1>), dim3(grid), dim3(256), 0, c->stream, a);
  return hip_status(hipGetLastError());
}

template <class T> int alpha_impl(swe_hweno_ctx* c, const T* state, double* alpha_host) {
  if (!c || !state || !alpha_host || !is_type<T>(c)) return SWE_EINVAL;
  launch_alpha<T>(c, state, SP_RHS, false, 0.0, c->stream);
  unsigned long long u[ASET];
  if (hipMemcpyAsync(u, speeds_set(c, SP_RHS), sizeof u, hipMemcpyDeviceToHost, c->stream) != hipSuccess)
    return SWE_EHIP;
  const int e = take_device_error(c);
  for (int k = 0; k < 2; ++k) {  // bits of non-negative doubles order as the doubles do
    unsigned long long m = 0;
    for (int l = 0; l < ASLOTS; ++l) m = std::max(m, u[l * ASTRIDE + k]);
    std::memcpy(&alpha_host[k], &m, 8);
  }
  return e;
}

// A single step and the start of its clock.
template <class T> void launch_step(swe_hweno_ctx* c, T* state, hipStream_t s) {
  if constexpr (sizeof(T) == 8) if (c->line && !c->timing) {
    launch_line(c, state, nullptr, 1, true, 0, 0.0, 0.0, s);
    return;
  }
  launch_alpha<T>(c, state, SP_N, true, 0.0, s);
  enqueue_step<T>(c, state, 0, s);
}

template <class T> int step_impl(swe_hweno_ctx* c, T* state, double dt, double* dt_used) {
  if (!c || !state || !is_type<T>(c)) return SWE_EINVAL;
  if (!(dt <= DBL_MAX)) return SWE_EINVAL;
  const swe_hweno_params saved = c->p;
  if (dt > 0) { c->p.flags |= SWE_FIXED_DT; c->p.fixed_dt = dt; }
  launch_step<T>(c, state, c->stream);
  c->p = saved;
  if (hipGetLastError() != hipSuccess) return SWE_EHIP;
  if (dt_used) {
    DevScal s;
    const int e = take_device_error(c, &s);
    if (e != SWE_EHIP) *dt_used = s.dt;
    return e;
  }
  return (c->p.flags & SWE_CHECK_DRY) ? take_device_error(c) : SWE_OK;
}

// Steps launched directly on a state before its graphs are captured. A capture takes 250 to 420 us of host time, and a
// replayed step is at most 1 us shorter than three launches (61 x 47 20.5 us against 20.9, 256^2 41.9 against 42 to 44) but leaves
// the host idle: short runs go without.
constexpr long GRAPH_AFTER = 256;
constexpr int LINE_STEPS = 1024;  // steps of a launch of k_line, about 6 ms

template <class T> int run_impl(swe_hweno_ctx* c, T* state, int nsteps, double t_end, double* t_out, int* steps_out) {
  if (!c || !state || !is_type<T>(c)) return SWE_EINVAL;
  if (!(t_end <= DBL_MAX) || (nsteps <= 0 && !(t_end > 0))) return SWE_EINVAL;
  const int use_tend = t_end > 0 ? 1 : 0;
  bool line = false;
  if constexpr (sizeof(T) == 8) line = c->line && !c->timing;
  if (!line && (c->g_state != state || c->g_tend != use_tend)) {
    destroy_graphs(c);
    c->g_state = state;
    c->g_tend = use_tend;
    c->g_steps = 0;
  }
  // t = 0, t_end, steps = 0 and alpha of the initial state
  if (!line) launch_alpha<T>(c, state, SP_N, true, t_end, c->stream);
  if (hipGetLastError() != hipSuccess) return SWE_EHIP;
  int done = 0;
  const int chunk = line ? LINE_STEPS : 64;
  for (;;) {
    int todo = nsteps > 0 ? nsteps - done : chunk;
    if (todo <= 0) break;
    if ((use_tend || line) && todo > chunk) todo = chunk;
    int k = 0;
    if constexpr (sizeof(T) == 8) if (line) {
      launch_line(c, state, nullptr, todo, done == 0, use_tend, t_end, 0.0, c->stream);
      if (hipGetLastError() != hipSuccess) return SWE_EHIP;
      k = todo;
    }
    if (!line && (c->timing || (!c->g8 && c->g_steps < GRAPH_AFTER))) {
      for (; k < todo && (c->timing || c->g_steps < GRAPH_AFTER); ++k) {
        enqueue_step<T>(c, state, use_tend, c->stream);
        if (!c->timing) c->g_steps += 1;
      }
      if (hipGetLastError() != hipSuccess) return SWE_EHIP;
    }
    if (k < todo && !c->g8) {
      int e = capture<T>(c, state, 1, use_tend, &c->g1);
      if (!e) e = capture<T>(c, state, 8, use_tend, &c->g8);
      if (e) { destroy_graphs(c); return e; }
    }
    for (; k + 8 <= todo; k += 8)
      if (hipGraphLaunch(c->g8, c->stream) != hipSuccess) return SWE_EHIP;
    for (; k < todo; ++k)
      if (hipGraphLaunch(c->g1, c->stream) != hipSuccess) return SWE_EHIP;
    done += todo;
    if (use_tend) {
      int active = 0;
      if (hipMemcpyAsync(&active, &c->sc->active, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess)
        return SWE_EHIP;
      if (hipStreamSynchronize(c->stream) != hipSuccess) return SWE_EHIP;
      if (!active) break;
    }
  }
  DevScal s;
  const int e = take_device_error(c, &s);
  if (e == SWE_EHIP) return e;
  if (c->timing) collect_timing(c);
  if (t_out) *t_out = s.t;
  if (steps_out) *steps_out = s.steps;
  return e;
}

// Device addresses of `scratch` and `scratch_speeds` on the current device, looked up once per device.
std::mutex g_scratch_mu;
struct ScratchAddr { void* planes; void* speeds; };
std::map<int, ScratchAddr> g_scratch_addr;

int scratch_address(ScratchAddr* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SWE_EHIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  auto it = g_scratch_addr.find(dev);
  if (it == g_scratch_addr.end()) {
    ScratchAddr a{nullptr, nullptr};
    if (hipGetSymbolAddress(&a.planes, HIP_SYMBOL(scratch)) != hipSuccess || !a.planes) return SWE_EHIP;
    if (hipGetSymbolAddress(&a.speeds, HIP_SYMBOL(scratch_speeds)) != hipSuccess || !a.speeds) return SWE_EHIP;
    it = g_scratch_addr.emplace(dev, a).first;
  }
  *out = it->second;
  return SWE_OK;
}

// Bytes of scratch an allocation-free step needs: device scalars, then S1, S2 (nf planes each)
// and D^{n,mod} (nd planes).
size_t noalloc_bytes(const swe_hweno_params* p) {
  const size_t n = (size_t)p->nx * (size_t)(p->dim == 2 ? p->ny : 1);
  const size_t planes = p->dim == 2 ? 2 * 9 + 6 : 2 * 4 + 2;
  return NOALLOC_SCAL + planes * n * sizeof(double);
}

int step_noalloc_impl(const swe_hweno_params* p, double* state, const double* b, const double* bx,
                      const double* by, double dt, void* stream, double* dt_used) {
  if (!params_ok(p) || !state || !b || !bx || (p->dim == 2 && !by)) return SWE_EINVAL;
  if (!(dt <= DBL_MAX)) return SWE_EINVAL;
  if (noalloc_bytes(p) > NOALLOC_BYTES) return SWE_EINVAL;
  ScratchAddr at{nullptr, nullptr};
  if (const int e = scratch_address(&at)) return e;
  // a context on the host stack that points into the scratch array and at the caller's bottom
  swe_hweno_ctx c;
  c.p = *p;
  c.stream = (hipStream_t)stream;
  c.nf = p->dim == 2 ? 9 : 4;
  c.nd = p->dim == 2 ? 6 : 2;
  c.n = (size_t)p->nx * (size_t)(p->dim == 2 ? p->ny : 1);
  c.b = (void*)b;
  c.bx = (void*)bx;
  c.by = (void*)by;
  c.sc = (DevScal*)at.planes;
  c.sp = (unsigned long long*)at.speeds;
  double* planes = (double*)((char*)at.planes + NOALLOC_SCAL);
  c.S1 = planes;
  c.S2 = planes + (size_t)c.nf * c.n;
  c.Dn = planes + (size_t)2 * c.nf * c.n;
  choose_tile(&c);
  if (dt > 0) { c.p.flags |= SWE_FIXED_DT; c.p.fixed_dt = dt; }
  hipLaunchKernelGGL(k_setup, dim3(1), dim3(ASLOTS), 0, c.stream, c.sc, c.sp, dbits(p->alpha_x),
                     dbits(p->dim == 2 ? p->alpha_y : 0.0));
  launch_step<double>(&c, state, c.stream);
  if (hipGetLastError() != hipSuccess) return SWE_EHIP;
  if (dt_used) {
    DevScal s;
    const int e = take_device_error(&c, &s);
    if (e != SWE_EHIP) *dt_used = s.dt;
    return e;
  }
  return SWE_OK;
}

}  // namespace

extern "C" {

int swe_hweno_abi_version(void) { return SWE_HWENO_ABI_VERSION; }

int swe_hweno_tile(int* cols_per_wave, int* rows_per_wave) {
  if (!cols_per_wave || !rows_per_wave) return SWE_EINVAL;
  *cols_per_wave = OUT_COLS;
  *rows_per_wave = ROWS_DEFAULT;
  return SWE_OK;
}

int swe_hweno_ctx_tile(const swe_hweno_ctx* c, int* cols_per_wave, int* rows_per_wave) {
  if (!c || !cols_per_wave || !rows_per_wave) return SWE_EINVAL;
  *cols_per_wave = OUT_COLS;
  *rows_per_wave = c->small ? c->small : c->rows;
  return SWE_OK;
}

const char* swe_hweno_strerror(int code) {
  switch (code) {
    case SWE_OK: return "ok";
    case SWE_EINVAL: return "invalid argument";
    case SWE_ENOMEM: return "device allocation failed";
    case SWE_EHIP: return "HIP runtime error";
    case SWE_EDRY: return "dry node (h <= 0)";
    case SWE_ENONFINITE: return "non-finite value";
    default: return "unknown error";
  }
}

int swe_hweno_init(const swe_hweno_params* p, const double* b, const double* bx, const double* by, void* stream,
                   swe_hweno_ctx** out) {
  return init_impl<double>(p, b, bx, by, stream, nullptr, 0, out);
}
int swe_hweno_init_f32(const swe_hweno_params* p, const float* b, const float* bx, const float* by, void* stream,
                       swe_hweno_ctx** out) {
  return init_impl<float>(p, b, bx, by, stream, nullptr, 0, out);
}
unsigned long swe_hweno_context_bytes(const swe_hweno_params* p, int single) {
  return params_ok(p) ? (unsigned long)ctx_layout(p, single ? sizeof(float) : sizeof(double)).bytes : 0;
}
int swe_hweno_init_in(const swe_hweno_params* p, int single, const void* b, const void* bx, const void* by, void* stream,
                      void* mem, unsigned long bytes, swe_hweno_ctx** out) {
  if (out) *out = nullptr;
  if (!mem) return SWE_EINVAL;
  if (single) return init_impl<float>(p, (const float*)b, (const float*)bx, (const float*)by, stream, mem, bytes, out);
  return init_impl<double>(p, (const double*)b, (const double*)bx, (const double*)by, stream, mem, bytes, out);
}

void swe_hweno_destroy(swe_hweno_ctx* c) {
  if (!c) return;
  if (c->stream || c->mem) (void)hipStreamSynchronize(c->stream);
  destroy_graphs(c);
  collect_timing(c);
  for (hipEvent_t e : c->pool) (void)hipEventDestroy(e);
  if (c->cap) (void)hipStreamDestroy(c->cap);
  if (c->mem && c->own_mem) (void)hipFree(c->mem);
  swe_adj_release(c);
  delete c;
}

int swe_hweno_rhs(swe_hweno_ctx* c, const double* state, double* rhs, double alpha_x, double alpha_y) {
  return rhs_impl<double>(c, state, rhs, alpha_x, alpha_y);
}
int swe_hweno_rhs_f32(swe_hweno_ctx* c, const float* state, float* rhs, double alpha_x, double alpha_y) {
  return rhs_impl<float>(c, state, rhs, alpha_x, alpha_y);
}

int swe_hweno_limit(swe_hweno_ctx* c, const double* state, double* dmod) { return limit_impl<double>(c, state, dmod); }
int swe_hweno_limit_f32(swe_hweno_ctx* c, const float* state, float* dmod) { return limit_impl<float>(c, state, dmod); }

int swe_hweno_alpha(swe_hweno_ctx* c, const double* state, double* alpha_host) {
  return alpha_impl<double>(c, state, alpha_host);
}
int swe_hweno_alpha_f32(swe_hweno_ctx* c, const float* state, double* alpha_host) {
  return alpha_impl<float>(c, state, alpha_host);
}

int swe_hweno_step(swe_hweno_ctx* c, double* state, double dt, double* dt_used) {
  return step_impl<double>(c, state, dt, dt_used);
}
int swe_hweno_step_f32(swe_hweno_ctx* c, float* state, double dt, double* dt_used) {
  return step_impl<float>(c, state, dt, dt_used);
}

int swe_hweno_run(swe_hweno_ctx* c, double* state, int nsteps, double t_end, double* t_out, int* steps_out) {
  return run_impl<double>(c, state, nsteps, t_end, t_out, steps_out);
}
int swe_hweno_run_f32(swe_hweno_ctx* c, float* state, int nsteps, double t_end, double* t_out, int* steps_out) {
  return run_impl<float>(c, state, nsteps, t_end, t_out, steps_out);
}

int swe_hweno_set_timing(swe_hweno_ctx* c, int on) {
  if (!c) return SWE_EINVAL;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return SWE_EHIP;
  collect_timing(c);
  c->timing = on != 0;
  for (int k = 0; k < 4; ++k) { c->ms[k] = 0; c->launches[k] = 0; }
  return SWE_OK;
}

int swe_hweno_get_timing(swe_hweno_ctx* c, double* ms, long long* launches) {
  if (!c || !ms || !launches) return SWE_EINVAL;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return SWE_EHIP;
  collect_timing(c);
  for (int k = 0; k < 4; ++k) { ms[k] = c->ms[k]; launches[k] = c->launches[k]; }
  return SWE_OK;
}

int swe_hweno_step_noalloc(const swe_hweno_params* params, double* state, const double* b, const double* bx,
                           const double* by, double dt, void* stream, double* dt_used) {
  return step_noalloc_impl(params, state, b, bx, by, dt, stream, dt_used);
}

unsigned long swe_hweno_noalloc_capacity(void) { return (unsigned long)NOALLOC_BYTES; }

int swe_hweno_math_check(int which, const double* x, double* y, unsigned long n, void* stream) {
  if (which < 0 || which > 2 || !x || !y || n == 0) return SWE_EINVAL;
  const size_t blocks = (n + 255) / 256;
  const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
  hipLaunchKernelGGL(k_math_check, dim3(grid), dim3(256), 0, (hipStream_t)stream, which, x, y, (size_t)n);
  if (hipGetLastError() != hipSuccess) return SWE_EHIP;
  return hip_status(hipStreamSynchronize((hipStream_t)stream));
}

#ifndef SWE_HWENO_SOURCE_HASH
#define SWE_HWENO_SOURCE_HASH "unstamped"
#endif
const char* swe_hweno_source_hash(void) { return SWE_HWENO_SOURCE_HASH; }

int swe_hweno_sync(swe_hweno_ctx* c) {
  if (!c) return SWE_EINVAL;
  return take_device_error(c);
}

}  // extern "C"

#include "swe_hweno_batch.inc"
#include "swe_hweno_adjoint.inc"
