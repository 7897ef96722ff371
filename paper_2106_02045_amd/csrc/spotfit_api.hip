// spotfit_api.hip -- host side of the C ABI declared in include/spotfit.h:
// option defaults and validation, the device context and the launch of the fit
// kernels.  Every check runs on the host before any HIP call; the fit itself
// runs entirely on the GPU.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>

#include "spotfit.h"
#include "spotfit_internal.h"
#include "spotfit_lm.h"

struct spotfit_ctx {
  int device;
  int n_cu;
  // resident 64-lane workgroups per CU, per (ppl class, per-pixel precision:
  // FP32, MIXED, COMP)
  int occupancy[5][3];
  // separable kernel: plan used for each size class (max side <= 8, <= 16, <= 32)
  // and resident 64-lane workgroups per CU of every plan
  int plan_for_class[3];
  bool plan_forced[3];  // set by the SPOTFIT_GROUP_PLAN override: no switch by batch size
  int occ_plan[16];
  // mixed-size batches: plan and residency of the persistent kernel, workspace
  int mixed_plan;
  bool mixed_forced;  // set by the SPOTFIT_MIXED_PLAN override
  int occ_mixed[8];
  int occ_matrix[4][2][2];  // matrix-core kernel: by spots per wavefront, width and pixel type
  int matrix_slots;      // SPOTFIT_MATRIX_SLOTS override: one of kMatrixSlots; else 0
  int32_t* ws;      // counters[8] then 3 lists of ws_cap spot indices
  int64_t ws_cap;
  void* stats;  // host memory that the blocks of spotfit_get_stats write, from its first call on
  int32_t* queue;             // the launches' spot counters
  int32_t* scratch;           // device address of this device's copy of `scratch` (below)
};

// Scratch memory of spotfit_fit_spots_noalloc: first the spot counters (one
// cache line each), then the mixed schedule's workspace: 8 counters, the classify pass's 128 words, then its 3 size-class lists of
// SPOTFIT_NOALLOC_MAX_SPOTS spot indices.  Every GPU
// holds its own copy at its own address.  In host code this name only stands
// for the array: kernels get the address that hipGetSymbolAddress returns for
// the current device (kept per device in g_scratch_addr and in each context).
constexpr int64_t kScratchMixedAt = sf::kMatrixCounters * sf::kMatrixCounterWords;
constexpr int64_t kScratchWords = kScratchMixedAt + sf::kMixedHeadWords + 3 * (int64_t)SPOTFIT_NOALLOC_MAX_SPOTS;
static __device__ __align__(256) int32_t scratch[kScratchWords];

namespace {

thread_local std::string g_last_error;

int fail(int code, const char* what) {
  g_last_error = what;
  return code;
}

int fail_hip(hipError_t e, const char* where) {
  g_last_error = std::string(where) + ": " + hipGetErrorString(e);
  return SPOTFIT_E_HIP;
}

int fail(int code, const std::string& what) { return fail(code, what.c_str()); }
int fail_hip(hipError_t e, const std::string& where) { return fail_hip(e, where.c_str()); }

// Device address of `scratch` on each device, looked up once per device (with
// that device current) by the first context created there.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch_addr[kMaxDevices] = {};

// Address of `scratch` on `device`, which must be current.
hipError_t scratch_address(int device, int32_t** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_addr[device]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_addr[device] = static_cast<int32_t*>(ptr);
  }
  *out = g_scratch_addr[device];
  return hipSuccess;
}

// Plan numbers of the matrix-core kernel, after the other plans'.
int matrix_plan() { return sf::group_plan_count(); }
int matrix_mixed_plan() { return sf::mixed_plan_count(); }
constexpr int kMatrixBuilds = 4;
constexpr int kMatrixSlots[kMatrixBuilds] = {4, 16, 32, 64};  // its builds: spots per wavefront

int ppl_index(int ppl) {
  switch (ppl) {
    case 1: return 0;
    case 2: return 1;
    case 4: return 2;
    case 8: return 3;
    default: return 4;
  }
}

// One block's share of spotfit_get_stats.
struct StatsBlock {
  uint32_t status[6], iters[65], pad;
  unsigned long long evals[2];
};
constexpr int kStatsBlocks = 128, kStatsThreads = 1024;
constexpr int64_t kStatsSpots = 4096;  // spots per block, up to kStatsBlocks

// Every block leaves its counts in host memory and the host adds them up once the
// stream is done: no buffer to clear, no copy, and no atomics on the same 74
// words from every block, which pass one by one (about 50 ns each: of 100,000 spots
// the counting took 12.3 us and the clearing 4.7, and start values, fit and
// statistics together went from 161.7 us to 145.2).  The counts of a block are in
// kCopies histograms by lane, so that the lanes of a wavefront, mostly with the
// same few values, collide less.
__global__ __launch_bounds__(kStatsThreads) void stats_kernel(const int32_t* status, const int32_t* iters,
                                                              const int32_t* evals, int64_t n,
                                                              StatsBlock* out) {
  constexpr int kCopies = 16, kBins = 6 + 65, kPitch = kBins + 2;
  __shared__ uint32_t hist[kCopies * kPitch];
  __shared__ unsigned long long ev[2];
  for (int i = threadIdx.x; i < kCopies * kPitch; i += kStatsThreads) hist[i] = 0u;
  if (threadIdx.x < 2) ev[threadIdx.x] = 0ull;
  __syncthreads();
  uint32_t* mine = hist + (threadIdx.x % kCopies) * kPitch;
  unsigned long long gsum = 0, tsum = 0;
  for (int64_t s = (int64_t)blockIdx.x * kStatsThreads + threadIdx.x; s < n;
       s += (int64_t)gridDim.x * kStatsThreads) {
    const int st = status[s], it = iters[s];
    int32_t ng = 0, nt = 0;
    if (evals) {
      ng = evals[2 * s];
      nt = evals[2 * s + 1];
    }
    if (st >= 0 && st < 6) atomicAdd(&mine[st], 1u);
    atomicAdd(&mine[6 + (it < 0 ? 0 : it > 64 ? 64 : it)], 1u);
    gsum += (unsigned long long)(ng > 0 ? ng : 0);
    tsum += (unsigned long long)(nt > 0 ? nt : 0);
  }
  if (evals) {
    for (int d = 32; d > 0; d >>= 1) {
      gsum += __shfl_down(gsum, d);
      tsum += __shfl_down(tsum, d);
    }
    if (threadIdx.x % 64 == 0) {
      atomicAdd(&ev[0], gsum);
      atomicAdd(&ev[1], tsum);
    }
  }
  __syncthreads();
  StatsBlock& b = out[blockIdx.x];
  if (threadIdx.x < kBins) {
    uint32_t v = 0;
    for (int c = 0; c < kCopies; ++c) v += hist[c * kPitch + threadIdx.x];
    if (threadIdx.x < 6)
      b.status[threadIdx.x] = v;
    else
      b.iters[threadIdx.x - 6] = v;
  }
  if (threadIdx.x < 2) b.evals[threadIdx.x] = ev[threadIdx.x];
}

// y = e^x with the fit kernels' own exponential (grid-stride over n values)
__global__ __launch_bounds__(256) void exp_neg_kernel(const double* x, double* y, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] = sf::lm::exp_neg(x[i]);
}

}  // namespace

extern "C" {

void spotfit_default_options(spotfit_options_t* o) {
  if (!o) return;
  std::memset(o, 0, sizeof *o);
  o->max_iter = 20;               // Results section: at most 20 iterations
  o->lambda0_exp10 = -2;          // LM section: initial damping 0.01
  o->lambda_max_exp10 = 4;        // LM section: stop once damping would exceed 1e4
  o->precision = SPOTFIT_PREC_FP64;
  o->max_error_per_px = 1.0 / 3.0;  // Results section: chi^2 < A/3, A = pixel count
  o->min_delta = 1e-6;            // Results section: decrease below 1e-6 chi^2
  o->min_step_rel = 1e-4;         // Results section: |dp_j| < 1e-4 |p_j|
  o->tie_tau = 0.0;
  o->sigma_min = 0.3;
  o->sigma_max_frac = 1.0;
  o->max_pixels = 1024;           // Implementation section: at most 1024 pixels per fit
  o->max_side = 32;
  o->schedule = SPOTFIT_SCHEDULE_UNIFORM;
  o->plan_hint = SPOTFIT_PLAN_THROUGHPUT;
}

int spotfit_validate_options(const spotfit_options_t* o) {
  if (!o) return fail(SPOTFIT_E_NULL, "options: NULL");
  if (o->max_iter < 0 || o->max_iter > 1000) return fail(SPOTFIT_E_OPTIONS, "max_iter not in [0, 1000]");
  if (o->lambda0_exp10 < -300 || o->lambda0_exp10 > 300 || o->lambda_max_exp10 < -300 ||
      o->lambda_max_exp10 > 300)
    return fail(SPOTFIT_E_OPTIONS, "lambda exponents not in [-300, 300]");
  if (o->precision != SPOTFIT_PREC_FP32 && o->precision != SPOTFIT_PREC_MIXED &&
      o->precision != SPOTFIT_PREC_FP64 && o->precision != SPOTFIT_PREC_FP32_PLAIN &&
      o->precision != SPOTFIT_PREC_COMP)
    return fail(SPOTFIT_E_OPTIONS, "unknown precision");
  if (!std::isfinite(o->max_error_per_px) || o->max_error_per_px < 0)
    return fail(SPOTFIT_E_OPTIONS, "max_error_per_px must be finite and >= 0");
  if (!std::isfinite(o->min_delta) || o->min_delta < 0 || o->min_delta >= 1)
    return fail(SPOTFIT_E_OPTIONS, "min_delta not in [0, 1)");
  if (!std::isfinite(o->min_step_rel) || o->min_step_rel < 0)
    return fail(SPOTFIT_E_OPTIONS, "min_step_rel must be finite and >= 0");
  if (!std::isfinite(o->tie_tau) || o->tie_tau < 0 || o->tie_tau >= 1)
    return fail(SPOTFIT_E_OPTIONS, "tie_tau not in [0, 1)");
  if (!std::isfinite(o->sigma_min) || o->sigma_min <= 0)
    return fail(SPOTFIT_E_OPTIONS, "sigma_min must be > 0");
  if (!std::isfinite(o->sigma_max_frac) || o->sigma_max_frac * 3.0 <= o->sigma_min)
    return fail(SPOTFIT_E_OPTIONS, "sigma_max_frac * 3 must exceed sigma_min");
  if (o->max_pixels < 9 || o->max_pixels > 1024)
    return fail(SPOTFIT_E_OPTIONS, "max_pixels not in [9, 1024]");
  if (o->max_side < 3 || o->max_side > 32)
    return fail(SPOTFIT_E_OPTIONS, "max_side not in [3, 32]");
  if (o->schedule != SPOTFIT_SCHEDULE_UNIFORM && o->schedule != SPOTFIT_SCHEDULE_MIXED)
    return fail(SPOTFIT_E_OPTIONS, "unknown schedule");
  if (o->plan_hint != SPOTFIT_PLAN_THROUGHPUT && o->plan_hint != SPOTFIT_PLAN_LATENCY)
    return fail(SPOTFIT_E_OPTIONS, "unknown plan hint");
  return SPOTFIT_OK;
}

int spotfit_ctx_create(spotfit_ctx_t** out, int device) {
  if (!out) return fail(SPOTFIT_E_NULL, "ctx_create: NULL out pointer");
  *out = nullptr;
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDeviceCount");
  if (device < 0 || device >= ndev) return fail(SPOTFIT_E_DEVICE, "ctx_create: no such device");
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) return fail_hip(e, "hipGetDeviceProperties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(SPOTFIT_E_DEVICE, "ctx_create: device is not gfx950");
  e = hipSetDevice(device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  spotfit_ctx* c = new (std::nothrow) spotfit_ctx();
  if (!c) return fail(SPOTFIT_E_DEVICE, "ctx_create: out of host memory");
  c->device = device;
  c->n_cu = prop.multiProcessorCount;
  const int ppls[5] = {1, 2, 4, 8, 16};
  for (int i = 0; i < 5; ++i) {
    for (int pr = 0; pr < 3; ++pr) {
      const int prec = pr == 0 ? SPOTFIT_PREC_FP32 : pr == 1 ? SPOTFIT_PREC_MIXED : SPOTFIT_PREC_COMP;
      int nb = 0;
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sf::wave_kernel_symbol(ppls[i], prec), 64, 0);
      if (e != hipSuccess) {
        delete c;
        return fail_hip(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
      }
      c->occupancy[i][pr] = nb > 0 ? nb : 1;
    }
  }
  for (int pl = 0; pl < sf::group_plan_count(); ++pl) {
    int nb = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sf::group_kernel_symbol(pl), 64, 0);
    if (e != hipSuccess) {
      delete c;
      return fail_hip(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    }
    c->occ_plan[pl] = nb > 0 ? nb : 1;
  }
  for (int pl = 0; pl < sf::mixed_plan_count(); ++pl) {
    int nb = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sf::mixed_kernel_symbol(pl), 64, 0);
    if (e != hipSuccess) {
      delete c;
      return fail_hip(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    }
    c->occ_mixed[pl] = nb > 0 ? nb : 1;
  }
  for (int i = 0; i < 4 * kMatrixBuilds; ++i) {
    const int slots = i >> 2, wide = (i >> 1) & 1, f32 = i & 1;
    int nb = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &nb, sf::matrix_kernel_symbol(kMatrixSlots[slots], wide != 0, f32 ? SPOTFIT_F32 : SPOTFIT_U16),
        64, 0);
    if (e != hipSuccess) {
      delete c;
      return fail_hip(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    }
    c->occ_matrix[slots][wide][f32] = nb > 0 ? nb : 1;
  }
  if (const char* env = std::getenv("SPOTFIT_MATRIX_SLOTS")) {
    const int v = std::atoi(env);
    for (int i = 0; i < kMatrixBuilds; ++i)
      if (v == kMatrixSlots[i]) c->matrix_slots = v;
  }
  // default mixed-size plan: the matrix-core kernel
  c->mixed_plan = matrix_mixed_plan();
  if (const char* env = std::getenv("SPOTFIT_MIXED_PLAN")) {
    const int v = std::atoi(env);
    if (v >= 0 && v <= matrix_mixed_plan()) {
      c->mixed_plan = v;
      c->mixed_forced = true;
    }
  }
  c->ws = nullptr;
  c->ws_cap = 0;
  c->stats = nullptr;
  c->queue = nullptr;
  c->scratch = nullptr;
  e = scratch_address(device, &c->scratch);
  if (e != hipSuccess) {
    delete c;
    return fail_hip(e, "hipGetSymbolAddress (no-allocation scratch)");
  }
  e = hipMalloc((void**)&c->queue, sizeof(int32_t) * sf::kMatrixCounters * sf::kMatrixCounterWords);
  if (e != hipSuccess) {
    delete c;
    return fail_hip(e, "hipMalloc (context buffers)");
  }
  // default plan of every size class: the matrix-core kernel
  for (int i = 0; i < 3; ++i) c->plan_for_class[i] = matrix_plan();
  if (const char* env = std::getenv("SPOTFIT_GROUP_PLAN")) {
    // tuning override "a,b,c": plan for each size class
    int a = -1, b = -1, d = -1;
    if (std::sscanf(env, "%d,%d,%d", &a, &b, &d) == 3) {
      const int want[3] = {a, b, d};
      const int side[3] = {8, 16, 32};
      for (int i = 0; i < 3; ++i) {
        int L = 0, C = 0;
        if (want[i] != matrix_plan()) sf::group_plan_shape(want[i], &L, &C);
        if (want[i] == matrix_plan() || L * C >= side[i]) {
          c->plan_for_class[i] = want[i];
          c->plan_forced[i] = true;
        }
      }
    }
  }
  if (const char* env = std::getenv("SPOTFIT_WAVES_PER_CU")) {
    const int v = std::atoi(env);
    if (v > 0 && v <= 64) {
      for (int i = 0; i < 5; ++i) c->occupancy[i][0] = c->occupancy[i][1] = c->occupancy[i][2] = v;
      for (int i = 0; i < 16; ++i) c->occ_plan[i] = v;
    }
  }
  *out = c;
  return SPOTFIT_OK;
}

void spotfit_ctx_destroy(spotfit_ctx_t* ctx) {
  if (!ctx) return;
  if (ctx->ws || ctx->stats || ctx->queue) {
    int cur = -1;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(ctx->device);
    if (ctx->ws) (void)hipFree(ctx->ws);
    if (ctx->stats) (void)hipHostFree(ctx->stats);
    if (ctx->queue) (void)hipFree(ctx->queue);
    if (cur >= 0) (void)hipSetDevice(cur);
  }
  delete ctx;
}

int spotfit_ctx_reserve(spotfit_ctx_t* ctx, int64_t n) {
  if (!ctx) return fail(SPOTFIT_E_NULL, "ctx_reserve: NULL context");
  if (n < 0 || n > ((int64_t)1 << 31) - 1) return fail(SPOTFIT_E_ARG, "ctx_reserve: n not in [0, 2^31)");
  if (n <= ctx->ws_cap) return SPOTFIT_OK;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  if (cur != ctx->device && (e = hipSetDevice(ctx->device)) != hipSuccess)
    return fail_hip(e, "hipSetDevice");
  if (ctx->ws) {
    e = hipDeviceSynchronize();  // a previous call may still use the old workspace
    if (e == hipSuccess) e = hipFree(ctx->ws);
    ctx->ws = nullptr;
    ctx->ws_cap = 0;
  }
  int32_t* p = nullptr;
  if (e == hipSuccess) e = hipMalloc((void**)&p, sizeof(int32_t) * (size_t)(sf::kMixedHeadWords + 3 * n));
  if (cur != ctx->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return fail_hip(e, "hipMalloc (mixed workspace)");
  ctx->ws = p;
  ctx->ws_cap = n;
  return SPOTFIT_OK;
}

}  // extern "C"

namespace {

// Checks of a fit call that need no HIP call; fills the validated options.
int check_call(spotfit_ctx_t* ctx, const void* data, int32_t dtype, const spotfit_shape_t* sizes,
               const int64_t* offsets, const float* init, int64_t n, const spotfit_options_t* opt,
               float* params_out, float* chi2_out, int32_t* iters_out, int32_t* status_out,
               spotfit_options_t* o, const char* who, bool init_optional = false) {
  if (!ctx) return fail(SPOTFIT_E_NULL, (std::string(who) + ": NULL context").c_str());
  if (n < 0) return fail(SPOTFIT_E_ARG, (std::string(who) + ": n_spots < 0").c_str());
  if (dtype != SPOTFIT_U16 && dtype != SPOTFIT_F32)
    return fail(SPOTFIT_E_ARG, (std::string(who) + ": unknown dtype").c_str());
  if (opt) {
    *o = *opt;
  } else {
    spotfit_default_options(o);
  }
  int rc = spotfit_validate_options(o);
  if (rc != SPOTFIT_OK) return rc;
  if (n == 0) return SPOTFIT_OK;
  if (!data || !sizes || !offsets || (!init && !init_optional) || !params_out || !chi2_out ||
      !iters_out || !status_out)
    return fail(SPOTFIT_E_NULL, (std::string(who) + ": NULL array").c_str());
  return SPOTFIT_OK;
}

// The mixed schedule's spot indices are 32-bit: a larger batch is refused as
// spotfit_ctx_reserve refuses its workspace, whether or not this batch would go
// through it.
int check_mixed_count(const spotfit_options_t& o, int64_t n, const char* who) {
  if (o.precision == SPOTFIT_PREC_FP64 && o.schedule == SPOTFIT_SCHEDULE_MIXED &&
      n > ((int64_t)1 << 31) - 1)
    return fail(SPOTFIT_E_ARG, std::string(who) + ": a mixed-schedule call takes fewer than 2^31 spots");
  return SPOTFIT_OK;
}

// The lane-owned plans hold 16-64 spots per wavefront and make a pass per
// spot of a group each step: they pay off when every resident spot slot fits
// several spots in turn; a smaller batch takes the narrow plan of the same
// bits.  Spots per resident slot from which a uniform launch takes the
// lane-owned plan, in halves: the crossovers measured against the narrow
// plans (15x15: between 262k and 393k spots, 2.0-3.0 per slot; 7x7: between
// 131k and 197k, 1.0-1.5; 32x32: between 66k and 131k, 2.0-4.0); plans that
// are not defaults keep 4.
int64_t owned_min_halves(int plan) {
  if (plan == sf::owned_plan_id(4, 4, 4) || plan == sf::owned_plan_id(16, 2, 4)) return 5;
  if (plan == sf::owned_plan_id(4, 2, 4)) return 3;
  return 8;
}
// The same rule for a mixed-size launch with lane-owned classes (over the
// whole batch; measured at 2M spots only).
constexpr int64_t kOwnedMinSpotsPerLane = 4;

// Batches of uneven sizes up to this many spots are fitted in the order given:
// a wavefront goes over its own slots by size, and the sort of the whole batch
// costs more than it saves (7..32 px, in order / sorted: 130,000 spots 320 us /
// 395, 200,000 486 / 503; 400,000 970 / 959, 2M 3723 / 3185).
constexpr int64_t kMatrixUnsorted = 262144;

// Whether a fit with these options runs the matrix-core kernel: always with the
// latency hint, and otherwise unless an override or the autotuner chose another
// plan.
bool takes_matrix(const spotfit_ctx_t* ctx, const spotfit_options_t& o) {
  if (o.precision != SPOTFIT_PREC_FP64) return false;
  if (o.plan_hint == SPOTFIT_PLAN_LATENCY) return true;
  if (o.schedule == SPOTFIT_SCHEDULE_MIXED) return ctx->mixed_plan == matrix_mixed_plan();
  return ctx->plan_for_class[o.max_side <= 8 ? 0 : o.max_side <= 16 ? 1 : 2] == matrix_plan();
}

// Wavefronts of the matrix-core kernel that the device holds at once.
int64_t matrix_resident(const spotfit_ctx_t* ctx, int slots_index, int32_t dtype, int32_t max_side) {
  return (int64_t)ctx->n_cu * ctx->occ_matrix[slots_index][max_side > 16][dtype == SPOTFIT_F32];
}

// Spots per wavefront (index into kMatrixSlots) for a batch of n spots.  With few
// spots a launch takes as long as a spot's steps, and a step is the shorter the
// fewer spots share it; with many it is the work per spot that counts, which
// falls with the spots that share the scalar part of a step.  In between, the
// fewest with which every spot is in flight at once are the fastest, within a
// few percent.  Measured, 16-bit pixels, us with 4 / 16 / 32 / 64 spots:
//   9 px     12,000: 34 / 35 / 43 / 64    48,000: 115 / 58 / 60 / 66    100,000: 222 / 124 / 108 / 94
//   15 px    12,000: 43 / 47 / 58 / 86    65,000: 176 / 99 / 88 / 98    100,000: 245 / 161 / 136 / 131
//   21 px     8,000: 54 / 67 / 94 / 145   32,000: 149 / 98 / 97 / 149    65,000: 274 / 198 / 147 / 153
//   32 px     8,000: 71 / 94 / 134 / 217  65,000: 367 / 267 / 202 / 224 100,000: 534 / 379 / 343 / 351
//   7..32 px  8,000: 54 / 80 / 115 / 190  65,000: 321 / 249 / 188 / 211 130,000: 600 / 414 / 387 / 320
// Wide floats, whose products wait longer for their pixels, keep 4 spots for half
// as many more (4 / 16 spots, 10,000 and 12,288: 17 px 54 / 63, 70 / 64; 24 px 59 /
// 74, 77 / 79; 32 px 77 / 99, 94 / 100; 7..32 px 78 / 95, 96 / 97; 16,384 of 28 px 97
// / 87).
//
// Large batches of floats in order are what the lane-owned mapping still fits sooner
// at some sizes, for the second pass of a step here over the pixels, for the
// residuals.  Lane-owned / here: of 29..32 px from 100,000 spots on (32x32 538 us /
// 565, 1M 3.97 ms / 4.95, but 400,000 of 17x17 1.55 / 1.02), of up to 16 px from about
// 500,000 (1M of 7x7 0.68 / 0.78, 4..8 px 0.79 / 1.00, 9x9 1.00 / 1.02, 15x15 1.13 /
// 1.20, 16x6 1.01 / 1.25; 400,000 of 15x15 0.52 / 0.52).  Nothing on the host tells
// these from the others (32 is max_side's default), and a spot's bits are not to
// depend on its batch; spotfit_autotune finds them.
int matrix_slot_index(const spotfit_ctx_t* ctx, int64_t n, int32_t dtype, const spotfit_options_t& o) {
  int64_t most[kMatrixBuilds - 1];
  for (int i = 0; i < kMatrixBuilds - 1; ++i)
    most[i] = kMatrixSlots[i] * matrix_resident(ctx, i, dtype, o.max_side);
  if (dtype == SPOTFIT_F32 && o.max_side > 16) most[0] = most[0] * 3 / 2;
  for (int i = 0; i < kMatrixBuilds; ++i) {
    if (ctx->matrix_slots ? ctx->matrix_slots == kMatrixSlots[i] : i == kMatrixBuilds - 1 || n <= most[i])
      return i;
  }
  return kMatrixBuilds - 1;
}

// Enqueue one fit with validated options o and n > 0.  init_out not NULL (with
// init NULL, double precision): start values are computed, in a launch before the
// fit's or by the narrow and wide plans in theirs, and written there.  Mixed schedule: `classified` is a
// workspace whose class lists are already built (no classify pass); otherwise
// `own_ws` (not NULL: a workspace of at least n spots that the caller owns) or
// the context's workspace, grown to n spots if needed, takes the classify pass.
int launch_fit(spotfit_ctx_t* ctx, const void* data, int32_t dtype, const spotfit_shape_t* sizes,
               const int64_t* offsets, const float* init, int64_t n, const spotfit_options_t& o,
               float* params_out, float* chi2_out, int32_t* iters_out, int32_t* status_out,
               int32_t* evals_out, void* stream, float* init_out = nullptr,
               const sf::MixedWs* classified = nullptr, const sf::MixedWs* own_ws = nullptr,
               int32_t* own_queue = nullptr) {
  sf::KArgs ka;
  std::memset(&ka, 0, sizeof ka);
  ka.data = data;
  ka.sizes = sizes;
  ka.offsets = offsets;
  ka.init = init;
  ka.init_out = init_out;
  ka.params_out = params_out;
  ka.chi2_out = chi2_out;
  ka.iters_out = iters_out;
  ka.status_out = status_out;
  ka.evals_out = evals_out;
  ka.queue = own_queue ? own_queue : ctx->queue;
  ka.n = n;
  ka.dtype = dtype;
  ka.opt.max_iter = o.max_iter;
  ka.opt.lambda0_exp10 = o.lambda0_exp10;
  ka.opt.lambda_max_exp10 = o.lambda_max_exp10;
  ka.opt.max_pixels = o.max_pixels;
  ka.opt.max_side = o.max_side;
  ka.opt.max_error_per_px = o.max_error_per_px;
  ka.opt.min_delta = o.min_delta;
  ka.opt.min_step_rel = o.min_step_rel;
  ka.opt.tie_tau = o.tie_tau;
  ka.opt.one_minus_tau = 1.0 - o.tie_tau;
  ka.opt.one_plus_tau = 1.0 + o.tie_tau;
  ka.opt.one_minus_min_delta = 1.0 - o.min_delta;
  ka.opt.sigma_min = o.sigma_min;
  ka.opt.sigma_max_frac = o.sigma_max_frac;

  hipError_t e;
  if (takes_matrix(ctx, o)) {
    const bool mixed = o.schedule == SPOTFIT_SCHEDULE_MIXED;
    if (init_out) {
      e = sf::launch_start_values(sf::kInitMoments, data, dtype, sizes, offsets, n, o.max_side,
                                  o.max_pixels, init_out, (hipStream_t)stream,
                                  o.plan_hint == SPOTFIT_PLAN_LATENCY);
      if (e != hipSuccess) return fail_hip(e, "start-value kernel launch");
      ka.init = init_out;
      ka.init_out = nullptr;
    }
    // a large batch of uneven sizes goes through the sorted class lists, so that
    // the spots of a wavefront are about as large as each other
    const bool lists = mixed && n > kMatrixUnsorted && n <= (int64_t)1 << 30;
    sf::MixedWs ws{};
    if (lists) {
      if (!classified && !own_ws && n > ctx->ws_cap) {
        const int rr = spotfit_ctx_reserve(ctx, n);
        if (rr != SPOTFIT_OK) return rr;
      }
      ws = classified ? *classified
           : own_ws   ? *own_ws
                      : sf::MixedWs{ctx->ws, ctx->ws + sf::kMixedHeadWords, ctx->ws_cap, ctx->ws + 8};
      if (!classified) {
        e = sf::launch_classify(ka, ws, (hipStream_t)stream);
        if (e != hipSuccess) return fail_hip(e, "classify launch");
      }
    }
    const bool wide = o.max_side > 16;
    const int si = matrix_slot_index(ctx, n, dtype, o);
    const int resident = (int)matrix_resident(ctx, si, dtype, o.max_side);
    e = hipSuccess;
    const int64_t chunk = (int64_t)1 << 30;  // the spot counter is 32-bit
    for (int64_t c0 = 0; c0 < n && e == hipSuccess; c0 += chunk) {
      sf::KArgs kc = ka;
      kc.n = n - c0 < chunk ? n - c0 : chunk;
      kc.sizes = sizes + c0;
      kc.offsets = offsets + c0;
      kc.init = ka.init + 4 * c0;
      kc.params_out = params_out + 6 * c0;
      kc.chi2_out = chi2_out + c0;
      kc.iters_out = iters_out + c0;
      kc.status_out = status_out + c0;
      kc.evals_out = evals_out ? evals_out + 2 * c0 : nullptr;
      e = sf::launch_matrix_kernel(kMatrixSlots[si], wide, kc, lists ? &ws : nullptr, resident,
                                   mixed ? ctx->n_cu : 0,
                                   kc.n <= 4 * kMatrixSlots[0] * (int64_t)ctx->n_cu, (hipStream_t)stream);
    }
  } else if (o.precision == SPOTFIT_PREC_FP64 && o.schedule == SPOTFIT_SCHEDULE_MIXED) {
    if (!classified && !own_ws && n > ctx->ws_cap) {
      const int rr = spotfit_ctx_reserve(ctx, n);
      if (rr != SPOTFIT_OK) return rr;
    }
    const sf::MixedWs ws = classified ? *classified
                           : own_ws   ? *own_ws
                                      : sf::MixedWs{ctx->ws, ctx->ws + sf::kMixedHeadWords, ctx->ws_cap,
                                                    ctx->ws + 8};
    int mplan = ctx->mixed_plan;
    if (sf::mixed_plan_narrow(mplan) != mplan && !ctx->mixed_forced &&
        n < kOwnedMinSpotsPerLane * (int64_t)ctx->n_cu * ctx->occ_mixed[mplan] * 64)
      mplan = sf::mixed_plan_narrow(mplan);
    const int64_t resident = (int64_t)ctx->n_cu * ctx->occ_mixed[mplan];
    const int64_t need = (n + 1) / 2;
    const int grid = (int)(need < resident ? need : resident);
    e = classified ? sf::launch_mixed_fit(mplan, ka, ws, grid, (hipStream_t)stream)
                   : sf::launch_mixed(mplan, ka, ws, grid, (hipStream_t)stream);
  } else if (o.precision == SPOTFIT_PREC_FP64) {
    const int cls = o.max_side <= 8 ? 0 : o.max_side <= 16 ? 1 : 2;
    int plan = ctx->plan_for_class[cls];
    if (sf::plan_for_raw(plan) != plan) {  // a lane-owned plan
      int ol = 0, oc = 0;
      sf::group_plan_shape(plan, &ol, &oc);
      const int64_t lanes_resident = (int64_t)ctx->n_cu * ctx->occ_plan[plan] * (64 / ol);
      if (init_out || (!ctx->plan_forced[cls] && 2 * n < owned_min_halves(plan) * lanes_resident))
        plan = sf::plan_for_raw(plan);
    }
    int lanes = 0, cpl = 0;
    sf::group_plan_shape(plan, &lanes, &cpl);
    const int64_t per_wave = 64 / lanes;
    const int64_t need = (n + per_wave - 1) / per_wave;
    // persistent grid: as many one-wave workgroups as can be resident at once
    const int64_t resident = (int64_t)ctx->n_cu * ctx->occ_plan[plan];
    const int grid = (int)(need < resident ? need : resident);
    // the narrow kernel's spot counter is 32-bit: batches of up to 2^30 spots per launch
    const int64_t chunk = (int64_t)1 << 30;
    e = hipSuccess;
    for (int64_t c0 = 0; c0 < n && e == hipSuccess; c0 += chunk) {
      sf::KArgs kc = ka;
      kc.n = n - c0 < chunk ? n - c0 : chunk;
      kc.sizes = sizes + c0;
      kc.offsets = offsets + c0;
      kc.init = init ? init + 4 * c0 : nullptr;
      kc.init_out = init_out ? init_out + 4 * c0 : nullptr;
      kc.params_out = params_out + 6 * c0;
      kc.chi2_out = chi2_out + c0;
      kc.iters_out = iters_out + c0;
      kc.status_out = status_out + c0;
      kc.evals_out = evals_out ? evals_out + 2 * c0 : nullptr;
      e = sf::launch_group_kernel(plan, kc, grid, (hipStream_t)stream);
    }
  } else if (o.precision == SPOTFIT_PREC_FP32_PLAIN) {
    const int threads = ((o.max_pixels + 63) / 64) * 64;
    e = sf::launch_plain_kernel(ka, threads, (hipStream_t)stream);
  } else {
    const int ppl = sf::ppl_for_pixels(o.max_pixels);
    const int pr = o.precision == SPOTFIT_PREC_MIXED ? 1 : o.precision == SPOTFIT_PREC_COMP ? 2 : 0;
    const int64_t resident = (int64_t)ctx->n_cu * ctx->occupancy[ppl_index(ppl)][pr];
    const int grid = (int)(n < resident ? n : resident);
    e = sf::launch_wave_kernel(ppl, o.precision, ka, grid, (hipStream_t)stream);
  }
  if (e != hipSuccess) return fail_hip(e, "fit kernel launch");
  return SPOTFIT_OK;
}

// Whether a fit of n spots with start values in memory (validated options o)
// takes a lane-owned plan: the plan choice of launch_fit.
bool takes_owned(const spotfit_ctx_t* ctx, int64_t n, const spotfit_options_t& o) {
  if (o.precision != SPOTFIT_PREC_FP64) return false;
  if (o.schedule == SPOTFIT_SCHEDULE_MIXED) {
    const int mplan = ctx->mixed_plan;
    return sf::mixed_plan_narrow(mplan) != mplan &&
           (ctx->mixed_forced || n >= kOwnedMinSpotsPerLane * (int64_t)ctx->n_cu * ctx->occ_mixed[mplan] * 64);
  }
  const int cls = o.max_side <= 8 ? 0 : o.max_side <= 16 ? 1 : 2;
  const int plan = ctx->plan_for_class[cls];
  if (sf::plan_for_raw(plan) == plan) return false;
  int ol = 0, oc = 0;
  sf::group_plan_shape(plan, &ol, &oc);
  const int64_t lanes_resident = (int64_t)ctx->n_cu * ctx->occ_plan[plan] * (64 / ol);
  return ctx->plan_forced[cls] || 2 * n >= owned_min_halves(plan) * lanes_resident;
}

// Enqueue start values and fit (validated options o, n > 0).  The separable
// double-precision kernels of the narrow and wide plans compute them in the
// fit's own launch; a batch that takes a lane-owned plan, and the other
// kernels, get a start-value launch first and read them from memory (the
// lane-owned fit with its start values from memory is the faster of the two
// there: 1M 15x15 1.54 against 1.61 ms, 1M 32x32 5.14 against 6.14, 2M mixed
// sizes 6.45 against 7.11; the same bits either way).
int launch_raw(spotfit_ctx_t* ctx, const void* data, int32_t dtype, const spotfit_shape_t* sizes,
               const int64_t* offsets, int64_t n, const spotfit_options_t& o, float* init_out,
               float* params_out, float* chi2_out, int32_t* iters_out, int32_t* status_out,
               int32_t* evals_out, void* stream, const sf::MixedWs* own_ws = nullptr) {
  if (takes_matrix(ctx, o) || (o.precision == SPOTFIT_PREC_FP64 && !takes_owned(ctx, n, o)))
    return launch_fit(ctx, data, dtype, sizes, offsets, nullptr, n, o, params_out, chi2_out,
                      iters_out, status_out, evals_out, stream, init_out, nullptr, own_ws);
  const hipError_t e = sf::launch_start_values(sf::kInitMoments, data, dtype, sizes, offsets, n,
                                               o.max_side, o.max_pixels, init_out,
                                               (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "start-value kernel launch");
  return launch_fit(ctx, data, dtype, sizes, offsets, init_out, n, o, params_out, chi2_out,
                    iters_out, status_out, evals_out, stream, nullptr, nullptr, own_ws);
}

}  // namespace

namespace sf {

bool reads_class_lists(const spotfit_ctx_t* ctx, int64_t n, const spotfit_options_t& o) {
  return o.precision == SPOTFIT_PREC_FP64 && o.schedule == SPOTFIT_SCHEDULE_MIXED &&
         (!takes_matrix(ctx, o) || n > kMatrixUnsorted);
}

int fit_preclassified(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                      const spotfit_shape_t* sizes, const int64_t* offsets, const float* init,
                      float* init_out, int64_t n, const spotfit_options_t& o, const MixedWs* ws,
                      float* params_out, float* chi2_out, int32_t* iters_out, int32_t* status_out,
                      void* stream) {
  if (o.precision != SPOTFIT_PREC_FP64 || o.schedule != SPOTFIT_SCHEDULE_MIXED)
    return fail(SPOTFIT_E_OPTIONS, "fit_preclassified: double precision, mixed schedule only");
  if (n == 0) return SPOTFIT_OK;
  return launch_fit(ctx, data, dtype, sizes, offsets, init_out ? nullptr : init, n, o, params_out,
                    chi2_out, iters_out, status_out, nullptr, stream, init_out, ws);
}

}  // namespace sf

extern "C" {

int spotfit_fit_spots(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                      const spotfit_shape_t* sizes, const int64_t* offsets, const float* init,
                      int64_t n, const spotfit_options_t* opt, float* params_out,
                      float* chi2_out, int32_t* iters_out, int32_t* status_out,
                      int32_t* evals_out, void* stream) {
  spotfit_options_t o;
  int rc = check_call(ctx, data, dtype, sizes, offsets, init, n, opt, params_out, chi2_out,
                      iters_out, status_out, &o, "fit_spots");
  if (rc == SPOTFIT_OK) rc = check_mixed_count(o, n, "fit_spots");
  if (rc != SPOTFIT_OK || n == 0) return rc;
  return launch_fit(ctx, data, dtype, sizes, offsets, init, n, o, params_out, chi2_out, iters_out,
                    status_out, evals_out, stream);
}

int spotfit_fit_spots_noalloc(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                              const spotfit_shape_t* sizes, const int64_t* offsets,
                              const float* init, int64_t n, const spotfit_options_t* opt,
                              float* params_out, float* chi2_out, int32_t* iters_out,
                              int32_t* status_out, int32_t* evals_out, void* stream) {
  spotfit_options_t o;
  int rc = check_call(ctx, data, dtype, sizes, offsets, init, n, opt, params_out, chi2_out,
                      iters_out, status_out, &o, "fit_spots_noalloc");
  if (rc != SPOTFIT_OK || n == 0) return rc;
  if (o.precision == SPOTFIT_PREC_FP64 && o.schedule == SPOTFIT_SCHEDULE_MIXED &&
      n > (int64_t)SPOTFIT_NOALLOC_MAX_SPOTS)
    return fail(SPOTFIT_E_ARG, "fit_spots_noalloc: a mixed-schedule call takes at most "
                               "SPOTFIT_NOALLOC_MAX_SPOTS (1048576) spots");
  if (!ctx->scratch) return fail(SPOTFIT_E_DEVICE, "fit_spots_noalloc: no scratch address");
  // the counters and lists live in this device's copy of `scratch`; the
  // kernels that use them clear the counters first (no memset, no allocation)
  const sf::MixedWs ws{ctx->scratch + kScratchMixedAt,
                       ctx->scratch + kScratchMixedAt + sf::kMixedHeadWords,
                       (int64_t)SPOTFIT_NOALLOC_MAX_SPOTS, ctx->scratch + kScratchMixedAt + 8};
  return launch_fit(ctx, data, dtype, sizes, offsets, init, n, o, params_out, chi2_out, iters_out,
                    status_out, evals_out, stream, nullptr, nullptr, &ws, ctx->scratch);
}

int spotfit_fit_raw(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                    const spotfit_shape_t* sizes, const int64_t* offsets, int64_t n,
                    const spotfit_options_t* opt, float* init_out, float* params_out,
                    float* chi2_out, int32_t* iters_out, int32_t* status_out,
                    int32_t* evals_out, void* stream) {
  spotfit_options_t o;
  int rc = check_call(ctx, data, dtype, sizes, offsets, init_out, n, opt, params_out, chi2_out,
                      iters_out, status_out, &o, "fit_raw");
  if (rc == SPOTFIT_OK) rc = check_mixed_count(o, n, "fit_raw");
  if (rc != SPOTFIT_OK || n == 0) return rc;
  return launch_raw(ctx, data, dtype, sizes, offsets, n, o, init_out, params_out, chi2_out,
                    iters_out, status_out, evals_out, stream);
}

static int start_values(int method, const char* what, const void* data, int32_t dtype,
                        const spotfit_shape_t* sizes, const int64_t* offsets, int64_t n,
                        const spotfit_options_t* opt, float* init_out, void* stream) {
  if (n < 0) return fail(SPOTFIT_E_ARG, std::string(what) + ": n_spots < 0");
  if (dtype != SPOTFIT_U16 && dtype != SPOTFIT_F32)
    return fail(SPOTFIT_E_ARG, std::string(what) + ": unknown dtype");
  spotfit_options_t o;
  if (opt) {
    o = *opt;
  } else {
    spotfit_default_options(&o);
  }
  const int rc = spotfit_validate_options(&o);
  if (rc != SPOTFIT_OK) return rc;
  if (n == 0) return SPOTFIT_OK;
  if (!data || !sizes || !offsets || !init_out)
    return fail(SPOTFIT_E_NULL, std::string(what) + ": NULL array");
  const hipError_t e = sf::launch_start_values(method, data, dtype, sizes, offsets, n, o.max_side,
                                               o.max_pixels, init_out, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, std::string(what) + " kernel launch");
  return SPOTFIT_OK;
}

int spotfit_moment_init(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                        const spotfit_shape_t* sizes, const int64_t* offsets, int64_t n,
                        const spotfit_options_t* opt, float* init_out, void* stream) {
  if (!ctx) return fail(SPOTFIT_E_NULL, "moment_init: NULL context");
  return start_values(sf::kInitMoments, "moment_init", data, dtype, sizes, offsets, n, opt,
                      init_out, stream);
}

int spotfit_peak_init(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                      const spotfit_shape_t* sizes, const int64_t* offsets, int64_t n,
                      const spotfit_options_t* opt, float* init_out, void* stream) {
  if (!ctx) return fail(SPOTFIT_E_NULL, "peak_init: NULL context");
  return start_values(sf::kInitPeak, "peak_init", data, dtype, sizes, offsets, n, opt, init_out,
                      stream);
}

int spotfit_get_stats(spotfit_ctx_t* ctx, const int32_t* status, const int32_t* iters,
                      const int32_t* evals, int64_t n, spotfit_stats_t* out, void* stream) {
  if (!ctx || !out) return fail(SPOTFIT_E_NULL, "get_stats: NULL context or output");
  if (n < 0) return fail(SPOTFIT_E_ARG, "get_stats: n_spots < 0");
  std::memset(out, 0, sizeof *out);
  if (n == 0) return SPOTFIT_OK;
  if (!status || !iters) return fail(SPOTFIT_E_NULL, "get_stats: NULL array");
  hipStream_t st = (hipStream_t)stream;
  const int64_t want = (n + kStatsSpots - 1) / kStatsSpots;
  const int blocks = (int)(want < kStatsBlocks ? want : kStatsBlocks);
  void* dev = nullptr;
  hipError_t e = hipSuccess;
  // at the first call: with it a context took 57 us to create, without it 13
  if (!ctx->stats)
    e = hipHostMalloc(&ctx->stats, sizeof(StatsBlock) * kStatsBlocks, hipHostMallocMapped | hipHostMallocPortable);
  if (e == hipSuccess) e = hipHostGetDevicePointer(&dev, ctx->stats, 0);
  if (e != hipSuccess) return fail_hip(e, "statistics buffer");
  hipLaunchKernelGGL(stats_kernel, dim3((unsigned)blocks), dim3(kStatsThreads), 0, st, status, iters,
                     evals, n, static_cast<StatsBlock*>(dev));
  e = hipGetLastError();
  if (e != hipSuccess) return fail_hip(e, "statistics kernel launch");
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return fail_hip(e, "statistics kernel");
  const StatsBlock* h = static_cast<const StatsBlock*>(ctx->stats);
  out->n_spots = n;
  for (int k = 0; k < blocks; ++k) {
    for (int i = 0; i < 6; ++i) out->status_count[i] += h[k].status[i];
    for (int i = 0; i < 65; ++i) out->iters_hist[i] += h[k].iters[i];
    out->grad_evals += (int64_t)h[k].evals[0];
    out->trial_evals += (int64_t)h[k].evals[1];
  }
  return SPOTFIT_OK;
}

int spotfit_autotune(spotfit_ctx_t* ctx, const void* data, int32_t dtype,
                     const spotfit_shape_t* sizes, const int64_t* offsets, const float* init,
                     int64_t n, const spotfit_options_t* opt, float* params_out, float* chi2_out,
                     int32_t* iters_out, int32_t* status_out, int32_t reps,
                     spotfit_tune_report_t* report, void* stream) {
  spotfit_options_t o;
  int rc = check_call(ctx, data, dtype, sizes, offsets, init, n, opt, params_out, chi2_out,
                      iters_out, status_out, &o, "autotune");
  if (rc == SPOTFIT_OK) rc = check_mixed_count(o, n, "autotune");
  if (rc != SPOTFIT_OK) return rc;
  if (o.precision != SPOTFIT_PREC_FP64)
    return fail(SPOTFIT_E_OPTIONS, "autotune: only the double-precision separable kernel has plans");
  if (reps < 1) return fail(SPOTFIT_E_ARG, "autotune: reps < 1");
  if (n == 0) return fail(SPOTFIT_E_ARG, "autotune: empty batch");
  const bool mixed = o.schedule == SPOTFIT_SCHEDULE_MIXED;
  const int cls = o.max_side <= 8 ? 0 : o.max_side <= 16 ? 1 : 2;
  const int side = cls == 0 ? 8 : cls == 1 ? 16 : 32;
  constexpr int kMaxPlans = 24;  // at least the plans there are
  constexpr int kReported = 16;  // entries of the report
  int cand[kMaxPlans];
  int nc = 0;
  if (o.plan_hint == SPOTFIT_PLAN_LATENCY) {
    // the hint's calls run one kernel whatever the context keeps (takes_matrix):
    // there is nothing to choose, and what throughput calls take stays as it is
    cand[nc++] = mixed ? matrix_mixed_plan() : matrix_plan();
  } else if (mixed) {
    cand[nc++] = matrix_mixed_plan();
    for (int p = 0; p < sf::mixed_plan_count() && nc < kMaxPlans; ++p) cand[nc++] = p;
  } else {
    cand[nc++] = matrix_plan();
    for (int p = 0; p < sf::group_plan_count() && nc < kMaxPlans; ++p) {
      int L = 0, C = 0;
      sf::group_plan_shape(p, &L, &C);
      if (L * C >= side) cand[nc++] = p;
    }
  }
  double ms[kMaxPlans];
  hipStream_t st = (hipStream_t)stream;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) return fail_hip(e, "hipEventCreate");
  const int keep = mixed ? ctx->mixed_plan : ctx->plan_for_class[cls];
  int best = 0;
  for (int i = 0; i < nc && rc == SPOTFIT_OK; ++i) {
    if (mixed)
      ctx->mixed_plan = cand[i];
    else
      ctx->plan_for_class[cls] = cand[i];
    rc = launch_fit(ctx, data, dtype, sizes, offsets, init, n, o, params_out, chi2_out, iters_out,
                    status_out, nullptr, stream);
    if (rc == SPOTFIT_OK && (e = hipEventRecord(e0, st)) != hipSuccess) rc = fail_hip(e, "hipEventRecord");
    for (int r = 0; r < reps && rc == SPOTFIT_OK; ++r)
      rc = launch_fit(ctx, data, dtype, sizes, offsets, init, n, o, params_out, chi2_out,
                      iters_out, status_out, nullptr, stream);
    if (rc == SPOTFIT_OK && (e = hipEventRecord(e1, st)) != hipSuccess) rc = fail_hip(e, "hipEventRecord");
    if (rc == SPOTFIT_OK && (e = hipEventSynchronize(e1)) != hipSuccess) rc = fail_hip(e, "hipEventSynchronize");
    float t = 0.f;
    if (rc == SPOTFIT_OK && (e = hipEventElapsedTime(&t, e0, e1)) != hipSuccess)
      rc = fail_hip(e, "hipEventElapsedTime");
    ms[i] = double(t) / reps;
    if (rc == SPOTFIT_OK && ms[i] < ms[best]) best = i;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  const int chosen = rc == SPOTFIT_OK && o.plan_hint != SPOTFIT_PLAN_LATENCY ? cand[best] : keep;
  if (mixed)
    ctx->mixed_plan = chosen;
  else
    ctx->plan_for_class[cls] = chosen;
  if (rc != SPOTFIT_OK) return rc;
  // the outputs: the kept plan's results
  rc = launch_fit(ctx, data, dtype, sizes, offsets, init, n, o, params_out, chi2_out, iters_out,
                  status_out, nullptr, stream);
  if (rc != SPOTFIT_OK) return rc;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  while (nc > kReported) {  // the slowest stay out of the report
    int worst = 0;
    for (int i = 1; i < nc; ++i)
      if (ms[i] > ms[worst]) worst = i;
    --nc;
    if (best > worst) --best;
    for (int i = worst; i < nc; ++i) {
      cand[i] = cand[i + 1];
      ms[i] = ms[i + 1];
    }
  }
  if (report) {
    std::memset(report, 0, sizeof *report);
    static_assert(sizeof report->plan_id / sizeof report->plan_id[0] == kReported, "entries of the report");
    report->schedule = o.schedule;
    report->size_class = mixed ? -1 : cls;
    report->n_candidates = nc;
    report->chosen = best;
    for (int i = 0; i < nc; ++i) {
      report->plan_id[i] = cand[i];
      report->plan_ms[i] = ms[i];
    }
  }
  return SPOTFIT_OK;
}

const char* spotfit_last_error(void) { return g_last_error.c_str(); }

int spotfit_version(void) { return 100; }

int spotfit_exp_neg(const double* x, double* y, int64_t n, void* stream) {
  if (n < 0) return fail(SPOTFIT_E_ARG, "exp_neg: n < 0");
  if (n == 0) return SPOTFIT_OK;
  if (!x || !y) return fail(SPOTFIT_E_NULL, "exp_neg: NULL array");
  const int64_t blocks = (n + 255) / 256;
  const int grid = (int)(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(exp_neg_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, x, y, n);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? SPOTFIT_OK : fail_hip(e, "exp_neg launch");
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Captured fits of fixed-shape batches: the copies and kernels of one call,
// recorded once into a HIP graph on a private stream and replayed with one
// launch.
// ---------------------------------------------------------------------------
struct spotfit_graph {
  int device = 0;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  float* init_buf = nullptr;  // start values of a graph that computes them (init NULL)
  int32_t* ws = nullptr;      // the mixed schedule's workspace, owned by the graph (its
                              // kernels keep this address for every replay)
};

extern "C" {

int spotfit_graph_create(spotfit_graph_t** out, spotfit_ctx_t* ctx, const void* data,
                         int32_t dtype, const spotfit_shape_t* sizes, const int64_t* offsets,
                         const float* init, int64_t n, const spotfit_options_t* opt,
                         float* params_out, float* chi2_out, int32_t* iters_out,
                         int32_t* status_out, const spotfit_graph_io_t* io) {
  if (!out) return fail(SPOTFIT_E_NULL, "graph_create: NULL out pointer");
  *out = nullptr;
  spotfit_options_t o;
  int rc = check_call(ctx, data, dtype, sizes, offsets, init, n, opt, params_out, chi2_out,
                      iters_out, status_out, &o, "graph_create", true);
  if (rc != SPOTFIT_OK) return rc;
  if (n == 0) return fail(SPOTFIT_E_ARG, "graph_create: n_spots = 0");
  const bool raw = init == nullptr;  // start values computed on the device
  if (raw && io && io->init)
    return fail(SPOTFIT_E_ARG, "graph_create: io->init needs a device init array");
  if (io && io->data && io->data_bytes <= 0)
    return fail(SPOTFIT_E_ARG, "graph_create: io->data_bytes must be > 0 with io->data");
  // the caller's current device is restored on return
  struct DeviceGuard {
    int prev = -1;
    ~DeviceGuard() {
      if (prev >= 0) (void)hipSetDevice(prev);
    }
  } guard;
  hipError_t e = hipGetDevice(&guard.prev);
  if (e == hipSuccess) e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  spotfit_graph* g = new (std::nothrow) spotfit_graph();
  if (!g) return fail(SPOTFIT_E_ARG, "graph_create: out of host memory");
  g->device = ctx->device;
  // the mixed schedule's workspace belongs to the graph and is allocated before the
  // capture: nothing allocates inside it, and a later call that grows the
  // context's workspace cannot free memory the replays use
  const bool mixed = o.precision == SPOTFIT_PREC_FP64 && o.schedule == SPOTFIT_SCHEDULE_MIXED;
  sf::MixedWs gws{nullptr, nullptr, 0};
  if (mixed) {
    e = hipMalloc((void**)&g->ws, sizeof(int32_t) * (size_t)(sf::kMixedHeadWords + 3 * n));
    if (e != hipSuccess) {
      g->ws = nullptr;
      spotfit_graph_destroy(g);
      return fail_hip(e, "hipMalloc (graph workspace)");
    }
    gws = sf::MixedWs{g->ws, g->ws + sf::kMixedHeadWords, n, g->ws + 8};
  }
  if (raw) {
    e = hipMalloc((void**)&g->init_buf, sizeof(float) * 4 * (size_t)n);
    if (e != hipSuccess) {
      g->init_buf = nullptr;
      spotfit_graph_destroy(g);
      return fail_hip(e, "hipMalloc (graph start values)");
    }
  }
  hipStream_t st = nullptr;
  e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
  if (e != hipSuccess) {
    spotfit_graph_destroy(g);
    return fail_hip(e, "hipStreamCreateWithFlags");
  }
  // the host's arrays as `io` names them: the copies of small ones are one kernel
  // before the fit and one after it
  struct Copy {
    void* dst;
    const void* src;
    int64_t bytes;
  };
  const Copy in[2] = {{const_cast<void*>(data), io ? io->data : nullptr, io ? io->data_bytes : 0},
                      {const_cast<float*>(init), io ? io->init : nullptr, 16 * n}};
  const Copy back[4] = {{io ? io->params : nullptr, params_out, 24 * n},
                        {io ? io->chi2 : nullptr, chi2_out, 4 * n},
                        {io ? io->iters : nullptr, iters_out, 4 * n},
                        {io ? io->status : nullptr, status_out, 4 * n}};
  sf::CopyList in_list{}, back_list{};
  bool in_kernel = true, back_kernel = true;
  for (const Copy& c : in) {
    if (!c.src) continue;
    const void* p = sf::pinned_address(c.src, c.bytes);
    in_kernel = in_kernel && p && in_list.add(c.dst, p, c.bytes);
  }
  for (const Copy& c : back) {
    if (!c.dst) continue;
    void* p = sf::pinned_address(c.dst, c.bytes);
    back_kernel = back_kernel && p && back_list.add(p, c.src, c.bytes);
  }
  e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess && in_kernel) {
    e = sf::launch_copy(in_list, st);
  } else {
    for (const Copy& c : in)
      if (e == hipSuccess && c.src)
        e = hipMemcpyAsync(c.dst, c.src, (size_t)c.bytes, hipMemcpyHostToDevice, st);
  }
  rc = SPOTFIT_OK;
  if (e == hipSuccess && raw)
    rc = launch_raw(ctx, data, dtype, sizes, offsets, n, o, g->init_buf, params_out, chi2_out,
                    iters_out, status_out, nullptr, st, mixed ? &gws : nullptr);
  else if (e == hipSuccess)
    rc = launch_fit(ctx, data, dtype, sizes, offsets, init, n, o, params_out, chi2_out, iters_out,
                    status_out, nullptr, st, nullptr, nullptr, mixed ? &gws : nullptr);
  if (e == hipSuccess && rc == SPOTFIT_OK && back_kernel) {
    e = sf::launch_copy(back_list, st);
  } else {
    for (const Copy& c : back)
      if (e == hipSuccess && rc == SPOTFIT_OK && c.dst)
        e = hipMemcpyAsync(c.dst, c.src, (size_t)c.bytes, hipMemcpyDeviceToHost, st);
  }
  // always end the capture, so the stream leaves capture mode whatever failed
  const hipError_t e_end = hipStreamEndCapture(st, &g->graph);
  if (e == hipSuccess) e = e_end;
  if (e == hipSuccess && rc == SPOTFIT_OK) e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
  (void)hipStreamDestroy(st);
  if (e != hipSuccess || rc != SPOTFIT_OK) {
    const std::string why = rc != SPOTFIT_OK ? std::string(spotfit_last_error()) : hipGetErrorString(e);
    spotfit_graph_destroy(g);
    return rc != SPOTFIT_OK ? fail(rc, "graph_create: " + why) : fail_hip(e, "graph_create");
  }
  *out = g;
  return SPOTFIT_OK;
}

int spotfit_graph_launch(spotfit_graph_t* g, void* stream) {
  if (!g || !g->exec) return fail(SPOTFIT_E_NULL, "graph_launch: NULL graph");
  const hipError_t e = hipGraphLaunch(g->exec, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "hipGraphLaunch");
  return SPOTFIT_OK;
}

void spotfit_graph_destroy(spotfit_graph_t* g) {
  if (!g) return;
  (void)hipSetDevice(g->device);
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  if (g->init_buf) (void)hipFree(g->init_buf);
  if (g->ws) (void)hipFree(g->ws);
  delete g;
}

}  // extern "C"
