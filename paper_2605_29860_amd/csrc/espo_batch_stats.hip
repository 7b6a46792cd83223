// espo_batch_stats: the update at the boundary of a rollout batch (Section 4.2: exponential
// moving averages of the batch mean and variance of the regret; Eq. beta_update: proportional
// controller of the threshold multiplier).
//
// Two small kernels.  The first reduces the valid tokens regret[b, t < L_b] to per-workgroup
// partial sums of d = g - mu_g and d^2 in double (shifting by the current mean estimate keeps
// the one-pass variance free of cancellation), plus token and stop counts; workgroup w takes
// rows w, w + G, ...  Rows of any length are read 16 bytes at a time: where T is no multiple of 4,
// from the 16-byte boundary before them, four loads per lane in flight; many short rows take a wave each.  The second adds the at most 1024 partials in a fixed
// order and forms the outputs.  A batch of at most 16 pieces of 1024 positions is one launch of one
// workgroup, whose waves take four pieces each.  Every reduction tree is fixed, so the result does
// not depend on scheduling.
//
// Bound by latency: launch, lengths, tokens, reduction, and the same once more for the partials.
// us per call on the GPU, before -> now (before: element-wise loads for odd T, two launches always): B = 512, T = 8191:
// 10.2 -> 8.2; B = 1024, T = 16383: 27.7 -> 17.2; B = 8, T = 16383: 12.8 -> 8.5; B = 100000, T = 5: 44.6 -> 24.9; B = 20000, T = 100:
// 15.2 -> 11.1; B = 4, T = 128: 5.7 -> 3.4; B = 1, T = 16384: 6.7 -> 4.4; one launch for 32 pieces instead: 9.1 against 5.8 for B = 32, T = 900, so the line is at 16.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "../../include/espo.h"
#include "espo_device.h"
#include "espo_host.h"

// Scratch of espo_batch_stats_static: room for the partial sums of the largest launch (1024
// workgroups, 32 bytes each).  One copy per GPU, held from the moment the library is loaded.
// In host code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[32768];

namespace espo {
namespace {

constexpr int kStatThreads = 256;
constexpr int kStatWaves = kStatThreads / kWave;
constexpr int kStatQuads = 4;                        // groups of four positions per lane and item
constexpr int kStatItem = kWave * 4 * kStatQuads;    // positions per item: 1024
constexpr int kStatUnroll = 4;                       // items of a wave, their loads in flight together
constexpr int kRowLoads = 4;                         // 16-byte loads of a lane in flight when a workgroup takes whole rows
constexpr uint32_t kDeepLoads = 8;                   // the same in rows of more than kLongRow tokens
constexpr int64_t kLongRow = 4096;
constexpr int kShortUnroll = 2;                      // rows of a wave in flight when every row is one item
constexpr int kMaxStatGroups = 1024;                 // partials the workspace has room for
constexpr int kFinalThreads = 256, kFinalEach = kMaxStatGroups / kFinalThreads;  // partials per thread
constexpr int kOneLaunchItems = kStatWaves * kStatUnroll;  // batches of at most this many items are one launch of one workgroup

struct Partial {
  double s1, s2;
  long long n, nstop;
};

// Sums over the workgroup of W waves in a fixed tree, the same in every thread; lds holds N * W entries.
template <int N, int W>
__device__ __forceinline__ void block_sums(double v[N], double* lds) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_sum_f64(v[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) lds[i * W + wave] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_sum_f64(lane < W ? lds[i * W + lane] : 0.0);
}

struct PartialArgs {
  const float* regret;
  const int32_t* lengths;
  const uint8_t* stopped;
  int64_t B, T;
  float mu_g;
  Partial* part;
};

struct FinalArgs {
  int64_t B;
  float mu_g, var_g, beta, alpha_ema, eta_beta, target_rate, beta_min, beta_max;
  espo_batch_result* out;
};

// The outputs from the four sums (counts are below 2^53: exact in double).
__device__ __forceinline__ void write_result(const FinalArgs& a, double s1, double s2, double n, double ns) {
  espo_batch_result r;
  const double md = n > 0.0 ? s1 / n : 0.0;                        // mean of g - mu_g
  const double mean = n > 0.0 ? (double)a.mu_g + md : 0.0;
  double var = n > 0.0 ? s2 / n - md * md : 0.0;
  if (var < 0.0) var = 0.0;
  const double rate = a.B > 0 ? ns / (double)a.B : 0.0;
  const double al = (double)a.alpha_ema;
  r.mean_g = mean;
  r.var_g_batch = var;
  r.stop_rate = rate;
  r.tokens = (int64_t)n;
  r.stopped = (int32_t)ns;
  r.mu_g = a.mu_g;
  r.var_g = a.var_g;
  r.beta = a.beta;
  if (n > 0.0) {
    r.mu_g = (float)(al * (double)a.mu_g + (1.0 - al) * mean);
    r.var_g = (float)(al * (double)a.var_g + (1.0 - al) * var);
  }
  if (a.B > 0) {
    double bt = (double)a.beta + (double)a.eta_beta * (rate - (double)a.target_rate);  // Eq. beta_update
    bt = bt < (double)a.beta_min ? (double)a.beta_min : bt;
    bt = bt > (double)a.beta_max ? (double)a.beta_max : bt;
    r.beta = (float)bt;
  }
  *a.out = r;
}

// Whether the 256 positions from `at` hold any of [lo, hi) (uniform in the wave: short rows cost what they hold).
__device__ __forceinline__ bool any_in(uint32_t at, uint32_t lo, uint32_t hi) { return lo < hi && at < hi && at + 4 * kWave > lo; }

// This lane's four tokens of those 256 (which hold some of [lo, hi)); positions outside read as the shift, so that they add
// nothing.  At a row's ends every lane loads four tokens by themselves, from the nearest positions inside: with one load for the
// lanes inside and others for the rest, a wave waits for memory twice (B = 100000, T = 5, a workgroup per row: 95 us, and 89 this way).
__device__ __forceinline__ f32x4 load_tokens(const float* __restrict__ src, uint32_t at, uint32_t lo, uint32_t hi, float shift) {
  const uint32_t t = at + (threadIdx.x & (kWave - 1)) * 4;
  if (at >= lo && at + 4 * kWave <= hi) return __builtin_nontemporal_load((const f32x4*)(src + t));
  f32x4 g;
#pragma unroll
  for (int j = 0; j < 4; ++j) g[j] = src[t + j < lo ? lo : (t + j < hi ? t + j : hi - 1)];
#pragma unroll
  for (int j = 0; j < 4; ++j) g[j] = t + j >= lo && t + j < hi ? g[j] : shift;
  return g;
}

__device__ __forceinline__ void add_tokens(const f32x4& g, double shift, double& s1, double& s2) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double d = (double)g[j] - shift;
    s1 += d;
    s2 = fma(d, d, s2);
  }
}

// Where a row's tokens lie: [lo, hi) from `src`, a multiple of 16 bytes (hi is below 2^31 + 3).
struct RowSpan {
  const float* src;
  uint32_t lo, hi;
};

__device__ __forceinline__ RowSpan row_span(const PartialArgs& a, int64_t row, int64_t& L) {
  L = __builtin_amdgcn_readfirstlane(a.lengths[row]);
  L = L < 0 ? 0 : (L > a.T ? a.T : L);
  const int64_t first = row * a.T, head = first & 3;
  return RowSpan{a.regret + (first - head), (uint32_t)head, (uint32_t)(head + L)};
}

// Counts of tokens and of stopped rows of the rows blockIdx.x, blockIdx.x + gridDim.x, ...: a thread each, apart from the
// tokens, whose loads would otherwise queue behind them row by row.  The first ones are loaded by the constructor and
// added, with the rest, by finish().
struct RowCounts {
  int32_t length = 0;
  uint32_t stop = 0;
  __device__ __forceinline__ explicit RowCounts(const PartialArgs& a) {
    const int64_t row = blockIdx.x + (int64_t)threadIdx.x * gridDim.x;
    if (row < a.B) {
      length = a.lengths[row];
      stop = a.stopped[row];
    }
  }
  __device__ __forceinline__ void finish(const PartialArgs& a, double& n, double& nstop) {
    for (int64_t row = blockIdx.x + (int64_t)threadIdx.x * gridDim.x; row < a.B;) {
      n += (double)(length < 0 ? 0 : (length > a.T ? a.T : (int64_t)length));
      nstop += stop != 0 ? 1.0 : 0.0;
      row += (int64_t)kStatThreads * gridDim.x;
      if (row < a.B) {
        length = a.lengths[row];
        stop = a.stopped[row];
      }
    }
  }
};

__device__ __forceinline__ void write_partial(const PartialArgs& a, RowCounts& counts, double s1, double s2, double* lds) {
  double v[4] = {s1, s2, 0.0, 0.0};
  counts.finish(a, v[2], v[3]);
  block_sums<4, kStatWaves>(v, lds);
  if (threadIdx.x == 0) a.part[blockIdx.x] = Partial{v[0], v[1], (long long)v[2], (long long)v[3]};
}

// Rows that start at 16-byte boundaries (T % 4 == 0), long ones of them, and rows that start anywhere.
enum RowKind { kAlignedRows, kLongRows, kAnyRows };

template <RowKind Kind>
__global__ __launch_bounds__(kStatThreads) void batch_partial_kernel(PartialArgs a) {
  __shared__ double lds[4 * kStatWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double shift = (double)a.mu_g;
  double s1 = 0.0, s2 = 0.0;
  RowCounts counts(a);
  for (int64_t row = blockIdx.x; row < a.B; row += gridDim.x) {
    int64_t L;
    const RowSpan r = row_span(a, row, L);
    if (Kind == kLongRows && __builtin_expect(L > kLongRow, 0)) {  // (wave-uniform; the shorter way stays in a straight line)
      // Rounds of eight loads per lane, all on their way before the first is added: one at a time, as below, a row's loads
      // wait for each other (us per call: B = 512, T = 8192: 9.6 -> 9.0; 1024, 16384: 16.5 -> 15.0; 8, 16384: 9.1 -> 8.4; but 300, 2000: 6.5 -> 6.6).
      // Trajectories that end early in such rows are short ones (T = 4100, B = 4000, 256 tokens each: 8.5, in rounds 9.6; B = 1500, 3072: 8.6,
      // 8.9; from 4096 tokens on both take the same).
      constexpr uint32_t kStride = kStatThreads * 4;
      const uint32_t full = (uint32_t)L & ~3u;  // (T is below 2^31)
      for (uint32_t base = 0; base < full; base += kDeepLoads * kStride) {
        f32x4 g[kDeepLoads];
#pragma unroll
        for (uint32_t u = 0; u < kDeepLoads; ++u) {
          const uint32_t t = base + u * kStride + threadIdx.x * 4;
          if (t < full) g[u] = __builtin_nontemporal_load((const f32x4*)(r.src + t));
        }
#pragma unroll
        for (uint32_t u = 0; u < kDeepLoads; ++u)
          if (base + u * kStride + threadIdx.x * 4 < full) add_tokens(g[u], shift, s1, s2);
      }
    } else if constexpr (Kind != kAnyRows) {
      const int64_t full = L & ~(int64_t)3;
      for (int64_t t = (int64_t)threadIdx.x * 4; t < full; t += kStatThreads * 4)
        add_tokens(__builtin_nontemporal_load((const f32x4*)(r.src + t)), shift, s1, s2);
    }
    if constexpr (Kind != kAnyRows) {
      const int64_t full = L & ~(int64_t)3;
      if (threadIdx.x < (unsigned)(L - full)) {  // the last one to three tokens
        const double d = (double)r.src[full + threadIdx.x] - shift;
        s1 += d;
        s2 = fma(d, d, s2);
      }
    } else for (uint32_t at = (uint32_t)wave * 4 * kWave; at < r.hi; at += kRowLoads * kStatThreads * 4) {
      f32x4 g[kRowLoads];
#pragma unroll
      for (int u = 0; u < kRowLoads; ++u)
        if (any_in(at + u * kStatThreads * 4, r.lo, r.hi)) g[u] = load_tokens(r.src, at + u * kStatThreads * 4, r.lo, r.hi, a.mu_g);
#pragma unroll
      for (int u = 0; u < kRowLoads; ++u)
        if (any_in(at + u * kStatThreads * 4, r.lo, r.hi)) add_tokens(g[u], shift, s1, s2);
    }
  }
  write_partial(a, counts, s1, s2, lds);
}

// Rows of one item each: a wave takes a row, and the rows of kShortUnroll
// rounds are on their way together.
__global__ __launch_bounds__(kStatThreads) void batch_short_kernel(PartialArgs a) {
  __shared__ double lds[4 * kStatWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double shift = (double)a.mu_g;
  double s1 = 0.0, s2 = 0.0;
  RowCounts counts(a);
  const int64_t step = (int64_t)gridDim.x * kStatWaves;
  for (int64_t row0 = (int64_t)wave * gridDim.x + blockIdx.x; row0 < a.B; row0 += kShortUnroll * step) {
    int64_t L;
    RowSpan r[kShortUnroll];
    f32x4 g[kShortUnroll][kStatQuads];
#pragma unroll
    for (int u = 0; u < kShortUnroll; ++u) {
      r[u] = RowSpan{nullptr, 0, 0};
      if (row0 + u * step < a.B) r[u] = row_span(a, row0 + u * step, L);
    }
#pragma unroll
    for (int u = 0; u < kShortUnroll; ++u)
#pragma unroll
      for (int q = 0; q < kStatQuads; ++q)
        if (any_in(q * 4 * kWave, r[u].lo, r[u].hi)) g[u][q] = load_tokens(r[u].src, q * 4 * kWave, r[u].lo, r[u].hi, a.mu_g);
#pragma unroll
    for (int u = 0; u < kShortUnroll; ++u)
#pragma unroll
      for (int q = 0; q < kStatQuads; ++q)
        if (any_in(q * 4 * kWave, r[u].lo, r[u].hi)) add_tokens(g[u][q], shift, s1, s2);
  }
  write_partial(a, counts, s1, s2, lds);
}

// One workgroup for a whole batch of at most kOneLaunchItems items (`per_row` of them in a row).
__global__ __launch_bounds__(kStatThreads) void batch_small_kernel(PartialArgs a, FinalArgs f, int items, int per_row) {
  __shared__ double lds[4 * kStatWaves];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double shift = (double)a.mu_g;
  double s1 = 0.0, s2 = 0.0, n = 0.0, nstop = 0.0;
  f32x4 g[kStatUnroll][kStatQuads];
  RowSpan r[kStatUnroll];
#pragma unroll
  for (int u = 0; u < kStatUnroll; ++u) {
    const int it = u * kStatWaves + wave;
    r[u] = RowSpan{nullptr, 0, 0};
    if (it < items) {  // (wave-uniform)
      const int row = it / per_row, off = (it - row * per_row) * kStatItem;
      int64_t L;
      r[u] = row_span(a, row, L);
      r[u].src += off;
      r[u].lo = off == 0 ? r[u].lo : 0;
      r[u].hi = r[u].hi <= (uint32_t)off ? 0u : min(r[u].hi - (uint32_t)off, (uint32_t)kStatItem);
#pragma unroll
      for (int q = 0; q < kStatQuads; ++q)
        if (any_in(q * 4 * kWave, r[u].lo, r[u].hi)) g[u][q] = load_tokens(r[u].src, q * 4 * kWave, r[u].lo, r[u].hi, a.mu_g);
    }
  }
  if (wave == 0 && lane < a.B) {  // at most kOneLaunchItems rows: a lane each
    const int64_t L = a.lengths[lane];
    n = (double)(L < 0 ? 0 : (L > a.T ? a.T : L));
    nstop = a.stopped[lane] != 0 ? 1.0 : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kStatUnroll; ++u)
#pragma unroll
    for (int q = 0; q < kStatQuads; ++q)
      if (any_in(q * 4 * kWave, r[u].lo, r[u].hi)) add_tokens(g[u][q], shift, s1, s2);
  double v[4] = {s1, s2, n, nstop};
  block_sums<4, kStatWaves>(v, lds);
  if (threadIdx.x == 0) write_result(f, v[0], v[1], v[2], v[3]);
}

__global__ __launch_bounds__(kFinalThreads) void batch_final_kernel(const Partial* __restrict__ part, int groups, FinalArgs f) {
  __shared__ double lds[4 * (kFinalThreads / kWave)];
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  Partial p[kFinalEach];
#pragma unroll
  for (int i = 0; i < kFinalEach; ++i) {
    const int at = i * kFinalThreads + (int)threadIdx.x;
    p[i] = at < groups ? part[at] : Partial{0.0, 0.0, 0, 0};
  }
#pragma unroll
  for (int i = 0; i < kFinalEach; ++i) {
    v[0] += p[i].s1;
    v[1] += p[i].s2;
    v[2] += (double)p[i].n;
    v[3] += (double)p[i].nstop;
  }
  block_sums<4, kFinalThreads / kWave>(v, lds);
  if (threadIdx.x == 0) write_result(f, v[0], v[1], v[2], v[3]);
}

// Partials the workspace of B rows has room for.
int stat_groups(int64_t B) { return (int)(B < 1 ? 1 : (B > kMaxStatGroups ? kMaxStatGroups : B)); }

// Device address of `scratch` on the current GPU: looked up once per device, with that device
// current, and kept.  Returns nullptr if the runtime cannot name the device or the symbol.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices];

void* static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

size_t batch_stats_static_capacity() { return sizeof(scratch); }
void* batch_stats_static_scratch() { return static_scratch(); }

size_t batch_stats_workspace(int64_t B) { return (size_t)stat_groups(B) * sizeof(Partial); }

int launch_batch_stats(const float* regret, const int32_t* lengths, const uint8_t* stopped, int64_t B, int64_t T,
                       float mu_g, float var_g, float beta, const espo_batch_ctrl& c, espo_batch_result* out,
                       void* workspace, hipStream_t stream) {
  FinalArgs f;
  f.B = B;
  f.mu_g = mu_g; f.var_g = var_g; f.beta = beta;
  f.alpha_ema = c.alpha_ema; f.eta_beta = c.eta_beta; f.target_rate = c.target_rate;
  f.beta_min = c.beta_min; f.beta_max = c.beta_max;
  f.out = out;
  PartialArgs p;
  p.regret = regret; p.lengths = lengths; p.stopped = stopped;
  p.B = B; p.T = T;
  p.mu_g = mu_g;
  p.part = (Partial*)workspace;
  // a row that starts between boundaries spans up to 3 positions more; a row of no positions is still counted
  const int64_t per_row = T > 0 ? (T + (T % 4 != 0 ? 3 : 0) + kStatItem - 1) / kStatItem : 1;
  if (B * per_row <= kOneLaunchItems) {
    static_assert(kOneLaunchItems <= kWave, "a lane per row");
    hipLaunchKernelGGL(batch_small_kernel, dim3(1), dim3(kStatThreads), 0, stream, p, f, (int)(B * per_row), (int)per_row);
    return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
  }
  // Rows of one item each take a wave each where there are more of them than workgroups (us, a workgroup per row -> a wave
  // per row: B = 100000, T = 8: 47.2 -> 24.8, T = 5: 89 -> 24.9; B = 4000, T = 1001: 11.8 -> 10.0), or where they start between
  // boundaries and a wave has a row in one load per lane (B = 512, T = 127: 7.0 -> 6.4; but B = 64, T = 1001: 6.3 -> 6.8).
  const bool one_item = per_row == 1 && (B > kMaxStatGroups || (T % 4 != 0 && T + 3 <= 4 * kWave));
  const int groups = stat_groups(one_item ? (B + kStatWaves - 1) / kStatWaves : B);
  if (one_item)
    hipLaunchKernelGGL(batch_short_kernel, dim3(groups), dim3(kStatThreads), 0, stream, p);
  else if (T % 4 == 0)
    hipLaunchKernelGGL(T > kLongRow ? batch_partial_kernel<kLongRows> : batch_partial_kernel<kAlignedRows>, dim3(groups), dim3(kStatThreads), 0, stream, p);
  else
    hipLaunchKernelGGL(batch_partial_kernel<kAnyRows>, dim3(groups), dim3(kStatThreads), 0, stream, p);
  if (hipGetLastError() != hipSuccess) return ESPO_EHIP;
  hipLaunchKernelGGL(batch_final_kernel, dim3(1), dim3(kFinalThreads), 0, stream, p.part, groups, f);
  return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
}

}  // namespace espo
