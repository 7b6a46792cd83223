// espo_whiten: advantage whitening over the valid tokens of a batch, the normalisation that
// PPO applies to the GAE output before the clipped objective (the paper keeps the standard PPO
// update, Section 3):  out = (A - mean) / sqrt(var + eps), mean and var over all A[b, t < L_b].
//
// Two launches over the same decomposition.  The batch is cut into items of 1024 positions of
// one row, which start at 16-byte boundaries whatever the row length is and which a wave moves with
// four 16-byte accesses per lane.  The first launch reduces each workgroup's items to
// (n, sum d, sum d^2) in double, with d = A - shift and shift the first valid token of the batch: a
// shift that is itself a data value keeps the one-pass variance free of cancellation however far
// the mean is from zero.  The second launch adds the at most 512 partials in a fixed tree (every
// workgroup gets the same bits whatever the scheduling) while its first items are on their way from
// memory, then rewrites its items.  Each element is normalised in double and rounded to float once.
// A batch of at most 16384 positions is one launch of one workgroup that keeps it in registers.
// Positions at t >= L_b are neither read nor written.
//
// Bound by memory from some 10 MB on, below that by the two launches' latency (load lengths, load
// tokens, reduce, store).  us per call: B = 1024, T = 16384, lengths U[512, T]: 24.5 (104 MB), from the rows' sums 15.9 (69 MB,
// 4.4 TB/s); B = 512, T = 8192: 11.6, 7.5; B = 4, T = 128: 4.1 (with items of 4096 positions and one workgroup-wide access each, the sums merged
// before the first load, element-wise accesses for odd T: 36.7, 23.9, 18.1, 9.8).  The nontemporal accesses stay:
// plain loads in the first launch take 3 us off the largest batch's second one, but leave the
// next pass over other arrays 1.2 us slower on the B = 512 batch.  One workgroup against two launches:
// 6.2 against 9.9 us for 8000 positions, 8.0 against 8.9 for 16384, so the line is there.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/espo.h"
#include "espo_device.h"
#include "espo_host.h"
#include "espo_quad.h"

namespace espo {
namespace {

// A workgroup has W waves, 16 or 8 (a template parameter of what depends on it).
constexpr int kWhQuads = 4;                         // groups of four positions per lane and item
constexpr int kWhItem = kWave * 4 * kWhQuads;       // positions per item: 1024
constexpr int kWhUnroll = 2;                        // items of a wave whose loads are in flight together
constexpr int kWhMaxGroups = 512;                   // workgroups of a launch: what the chip holds of the larger ones
// Up to these many items the sums are formed by workgroups of 8 waves with an item or two for each, not of 16 of which half had none where T is
// 4096 or more: the waves of a launch start over some microseconds, so waves with little to do cost more than they bring (us, both launches,
// B = 512, T = 8192: 14.4 -> 11.9; packed, 2.1 M tokens: 13.1 -> 11.1; B = 300, T = 2001: 13.0 -> 8.9; 2000, 3000: 16.6 -> 14.4).  Beyond, the larger
// workgroups keep twice as much in flight on a compute unit (B = 1024, T = 16384: 7.2, with 8 waves 7.6).
constexpr int64_t kWhEightWavesTo = 8192;
// The rewrite takes workgroups of 8 waves as long as a wave can hold all its items, at most kWhHold, whose loads are then all on their way before the
// sums are merged; beyond, 16 waves that have one item on its way at a time (us, from the rows' sums, with 16 waves / now:
// B = 512, T = 8192, an item a wave: 9.1 / 7.5; 2000, 3000: 12.1 / 11.4 (one item on its way at a time: 12.4); 1024, 16384: 18.5 / 15.6;
// but 1024, 16383, 17408 items in two rounds: 19.8 / 21.8).
constexpr int kWhHold = 4;
constexpr int kWhSmallThreads = 1024, kWhSmallWaves = kWhSmallThreads / kWave;
constexpr int kWhSmallQuads = 4;                    // groups of four positions per lane of the one-workgroup form
constexpr int64_t kWhSmall = (int64_t)kWhSmallThreads * 4 * kWhSmallQuads;
constexpr uint32_t kWhSkew = 389;                   // rows between a wave's items of neighbouring chunk positions

// Sums of some tokens about a shift of their own: the same fields as AdvRowStats.
using Sums = AdvRowStats;

struct WhArgs {
  const float* adv;
  const int32_t* lengths;
  int64_t B, T, nch;  // nch: items per row
  int64_t items;      // B * nch
  int groups;
  float eps;
  int shift_mean, ddof;
  float* out;
  double* stats;  // optional [3]: mean, var, n
  Sums* part;     // [groups]
};

__device__ __forceinline__ double lane_f64(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// An item (uniform in the wave): where it starts in the flat array, a multiple of 4, and which of its positions
// hold valid tokens of its row.
struct Item {
  int64_t start;
  int32_t lo, hi;
};

// Items are numbered chunk position first, so the waves of a workgroup and their successive items see all chunk
// positions; the rows are turned by kWhSkew from one chunk position to the next, so that the items a compute unit
// gets come from different rows (without that, one that drew two long rows had all their chunks:
// 18.6 against 18.0 us for the rewrite of a B = 1024, T = 16384 batch).
__device__ __forceinline__ Item item_of(const WhArgs& a, uint32_t it) {
  Item im{0, 0, 0};
  if (it < (uint32_t)a.items) {
    const uint32_t ch = it / (uint32_t)a.B, row = (it - ch * (uint32_t)a.B + ch * kWhSkew) % (uint32_t)a.B;
    int64_t L = a.lengths[row];
    L = L < 0 ? 0 : (L > a.T ? a.T : L);
    const int64_t first = (int64_t)row * a.T, head = first & 3, off = (int64_t)ch * kWhItem;
    im.start = first - head + off;
    im.lo = ch == 0 ? (int32_t)head : 0;
    const int64_t left = L + head - off;
    im.hi = (int32_t)(left < 0 ? 0 : (left < kWhItem ? left : kWhItem));
    if (L == 0) im.hi = 0;
  }
  return im;
}

// Item k of this wave: the waves of one workgroup take items a whole grid apart.
template <int W>
__device__ __forceinline__ uint32_t item_index(const WhArgs& a, int k) {
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  return ((uint32_t)k * W + wave) * (uint32_t)a.groups + blockIdx.x;
}

__device__ __forceinline__ int quad_at(int q) { return q * kWave * 4 + (int)(threadIdx.x & (kWave - 1)) * 4; }

// Where this lane's four tokens for position t of an item start, and which of them are its own.  Workgroups of 8 waves load four
// tokens of the row at its ends too, from as far inside as it takes: with single loads there, a wave waits for memory
// twice (B = 1000, T = 300: 13.0 -> 8.9 us, the smaller workgroups included).  The larger ones have no registers for that (whole quads there, B = 1024,
// T = 16384: 25.5 -> 27.4).
template <int W>
__device__ __forceinline__ Quad lane_quad(const Item& im, int t) {
  if constexpr (W == 16) {
    const int lo = im.lo - t, hi = im.hi - t;  // its own: lo <= j < hi
    return Quad{t, (hi >= 4 ? 0xfu : hi > 0 ? (1u << hi) - 1u : 0u) & (lo <= 0 ? 0xfu : lo < 4 ? 0xfu << lo : 0u)};
  } else {
    return quad_of(t, im.lo, im.hi);
  }
}

using f32x4_any = float __attribute__((ext_vector_type(4), aligned(4)));  // at any element

// Loads them; returns which of them are the lane's own.  Positions that are not of the row's valid ones are never read.
template <int W>
__device__ __forceinline__ uint32_t load_quad(const float* __restrict__ src, const Item& im, int t, f32x4& g) {
  g = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (W == 16) {
    if (t >= im.lo && t + 4 <= im.hi) {
      g = __builtin_nontemporal_load((const f32x4*)(src + im.start + t));
      return 0xfu;
    }
  }
  const Quad quad = lane_quad<W>(im, t);
  if (quad.in != 0) {
    const float* const from = src + im.start + quad.at;
    if (W != 16 && im.hi - im.lo >= 4) {  // (wave-uniform)
      g = __builtin_nontemporal_load((const f32x4_any*)from);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((quad.in >> j) & 1u) g[j] = from[j];
    }
  }
  return quad.in;
}

// ---------------------------------------------------------------- sums
// A lane's running sums about a shift that is the same in the whole batch.
struct LaneSums {
  double s1 = 0.0, s2 = 0.0;
  int n = 0;  // tokens of the wave
  __device__ __forceinline__ void add(const f32x4& g, uint32_t in, double shift) {
    if (__builtin_amdgcn_ballot_w64(in != 0xfu) == 0) {
      n += 4 * kWave;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double d = (double)g[j] - shift;
        s1 += d;
        s2 = fma(d, d, s2);
      }
    } else if (__builtin_amdgcn_ballot_w64(in != 0) != 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        n += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64((in >> j) & 1u));
        const double d = (in >> j) & 1u ? (double)g[j] - shift : 0.0;
        s1 += d;
        s2 = fma(d, d, s2);
      }
    }
  }
};

// Sum over the first 16 lanes, returned to the wave.
__device__ __forceinline__ double row_sum_f64(double v) {
  v += dpp_f64<kDppRowShr1, 0xf>(v);
  v += dpp_f64<kDppRowShr2, 0xf>(v);
  v += dpp_f64<kDppRowShr4, 0xf>(v);
  v += dpp_f64<kDppRowShr8, 0xf>(v);
  return lane_f64(v, 15);
}

// Three sums over the workgroup in a fixed tree, the same in every thread; lds holds 3 * W entries.
template <int W>
__device__ __forceinline__ void block_sums(double v[3], double* lds) {
  static_assert(W <= 16, "one row of lanes holds the waves' sums");
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 3; ++i) v[i] = wave_sum_f64(v[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 3; ++i) lds[i * W + wave] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) v[i] = row_sum_f64(lane < W ? lds[i * W + lane] : 0.0);
}

// The first valid token of the batch, as its shift (0 without any).
__device__ __forceinline__ double batch_shift(const WhArgs& a) {
  for (int64_t b = 0; b < a.B; ++b)
    if (a.lengths[b] > 0) return (double)a.adv[b * a.T];
  return 0.0;
}

// What a set of sums amounts to: count, mean, and sum of squared deviations from it.
struct Moments {
  double n, mean, m2;
};

template <int W>
__global__ __launch_bounds__(W * kWave, W == 16 ? 8 : 4) void whiten_partial_kernel(WhArgs a) {
  __shared__ double lds[3 * W];
  LaneSums w;
  double shift = W == 16 ? batch_shift(a) : 0.0;
  for (int k = 0; item_index<W>(a, k) < (uint32_t)a.items; k += kWhUnroll) {  // (wave 0 always has an item)
    f32x4 g[kWhUnroll][kWhQuads];
    uint32_t in[kWhUnroll][kWhQuads];
#pragma unroll
    for (int u = 0; u < kWhUnroll; ++u) {
      const Item im = item_of(a, item_index<W>(a, k + u));
#pragma unroll
      for (int q = 0; q < kWhQuads; ++q) in[u][q] = load_quad<W>(a.adv, im, quad_at(q), g[u][q]);
    }
    if (W != 16 && k == 0) shift = batch_shift(a);  // two loads one after the other, behind those of the first items
#pragma unroll
    for (int u = 0; u < kWhUnroll; ++u)
#pragma unroll
      for (int q = 0; q < kWhQuads; ++q) w.add(g[u][q], in[u][q], shift);
  }
  double v[3] = {w.s1, w.s2, (threadIdx.x & (kWave - 1)) == 0 ? (double)w.n : 0.0};
  block_sums<W>(v, lds);
  if (threadIdx.x == 0) a.part[blockIdx.x] = Sums{v[0], v[1], shift, (long long)v[2]};
}

// ---------------------------------------------------------------- rewrite
struct Scale {
  double sub, rstd;
};

__device__ __forceinline__ Scale scale_of(const WhArgs& a, const Moments& m, bool report) {
  const double denom = m.n - (double)a.ddof;
  const double ss = m.m2 > 0.0 ? m.m2 : 0.0;
  const double var = denom > 0.0 ? ss / denom : 0.0;
  const double sd = sqrt(var + (double)a.eps);
  if (report && a.stats) {
    a.stats[0] = m.n > 0.0 ? m.mean : 0.0;
    a.stats[1] = m.n > 0.0 ? var : 0.0;
    a.stats[2] = m.n;
  }
  return Scale{a.shift_mean ? m.mean : 0.0, sd > 0.0 ? 1.0 / sd : 0.0};  // a constant batch with eps = 0: every output is 0
}

__device__ __forceinline__ float normalised(float x, const Scale& s) {
  return s.rstd > 0.0 ? (float)(((double)x - s.sub) * s.rstd) : 0.0f;
}

__device__ __forceinline__ void store_quad(float* __restrict__ dst, const f32x4& g, uint32_t in, const Scale& s) {
  if (in == 0xfu) {
    __builtin_nontemporal_store(f32x4{normalised(g[0], s), normalised(g[1], s), normalised(g[2], s), normalised(g[3], s)}, (f32x4*)dst);
    return;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if ((in >> j) & 1u) dst[j] = normalised(g[j], s);
}

// The moments of the batch from sums about a shift of each set's own, thread i of n taking sets i, i + n, ...; the
// same bits in every workgroup.  Mean first, then the squared deviations from it (each set's about its own shift, moved to the
// mean), so that nothing cancels however far the sets' levels are apart.  The sums on the way to the mean are about
// one of the sets' shifts: a constant batch has its exact mean.
template <int W>
__device__ __forceinline__ Moments moments_of_rows(const Sums* __restrict__ sets, int64_t count, Sums* lds, double* lds_m2) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  Sums mine{0.0, 0.0, 0.0, 0};
  double n = 0.0, s1 = 0.0, to = 0.0;
  for (int64_t i = threadIdx.x; i < count; i += W * kWave) {
    mine = sets[i];
    if (mine.n > 0) {
      if (n == 0.0) to = mine.shift;
      n += (double)mine.n;
      s1 += fma((double)mine.n, mine.shift - to, mine.s1);
    }
  }
  {
    const uint64_t who = __builtin_amdgcn_ballot_w64(n > 0.0);
    const double wto = who != 0 ? lane_f64(to, (int)__builtin_ctzll(who)) : 0.0;
    const double ws1 = wave_sum_f64(n > 0.0 ? fma(n, to - wto, s1) : 0.0), wn = wave_sum_f64(n);
    if (lane == 0) lds[wave] = Sums{ws1, 0.0, wto, (long long)wn};
  }
  __syncthreads();
  Sums s{0.0, 0.0, 0.0, 0};
  if (lane < W) s = lds[lane];
  const uint64_t who = __builtin_amdgcn_ballot_w64(s.n > 0);
  to = who != 0 ? lane_f64(s.shift, (int)__builtin_ctzll(who)) : 0.0;
  n = row_sum_f64((double)s.n);
  s1 = row_sum_f64(s.n > 0 ? fma((double)s.n, s.shift - to, s.s1) : 0.0);
  const double mean = n > 0.0 ? to + s1 / n : 0.0;
  double m2 = 0.0;
  auto deviations = [&](const Sums& x) {
    const double d = x.shift - mean;
    return x.n > 0 ? fma(d, fma((double)x.n, d, 2.0 * x.s1), x.s2) : 0.0;
  };
  if (count <= W * kWave) {
    m2 = deviations(mine);
  } else {
    for (int64_t i = threadIdx.x; i < count; i += W * kWave) m2 += deviations(sets[i]);
  }
  m2 = wave_sum_f64(m2);
  if (lane == 0) lds_m2[wave] = m2;
  __syncthreads();
  m2 = row_sum_f64(lane < W ? lds_m2[lane] : 0.0);
  return Moments{n, mean, m2};
}

// The same from at most kWhMaxGroups sets about one shift.
template <int W>
__device__ __forceinline__ Moments moments_of_parts(const Sums* __restrict__ parts, int count, double* lds) {
  Sums mine{0.0, 0.0, 0.0, 0};
  static_assert(W * kWave >= kWhMaxGroups, "a thread per part");
  if ((int)threadIdx.x < count) mine = parts[threadIdx.x];
  double v[3] = {mine.s1, mine.s2, (double)mine.n};
  const double shift = parts[0].shift;
  block_sums<W>(v, lds);
  const double md = v[2] > 0.0 ? v[0] / v[2] : 0.0;
  return Moments{v[2], shift + md, fma(-v[2] * md, md, v[1])};  // s2 - n md^2: the squared deviations from the mean
}

// The rewrite, from the sums of `count` rows or parts.  Hold: items of a wave, all of them, whose loads are issued before the sums
// are merged; 0: as many as it takes, the first one's loads before that, and every next one's before the current one is stored.
template <bool Rows, int W, int Hold>
__global__ __launch_bounds__(W * kWave, W == 16 ? 8 : 4) void whiten_apply_kernel(WhArgs a, const Sums* __restrict__ sets, int64_t count) {
  __shared__ Sums lds[Rows ? W : 1];
  __shared__ double lds_d[3 * W];
  struct Held {
    f32x4 g[kWhQuads];
    uint32_t in;  // four bits per group of four
    Item im;
  };
  auto fetch = [&](int k) {
    Held h;
    h.im = item_of(a, item_index<W>(a, k));
    h.in = 0;
#pragma unroll
    for (int q = 0; q < kWhQuads; ++q) h.in |= load_quad<W>(a.adv, h.im, quad_at(q), h.g[q]) << (4 * q);
    return h;
  };
  auto store = [&](const Held& h, const Scale& s) {
#pragma unroll
    for (int q = 0; q < kWhQuads; ++q)
      store_quad(a.out + h.im.start + lane_quad<W>(h.im, quad_at(q)).at, h.g[q], (h.in >> (4 * q)) & 0xfu, s);
  };
  Held held[Hold > 0 ? Hold : 1];
#pragma unroll
  for (int i = 0; i < (Hold > 0 ? Hold : 1); ++i) held[i] = fetch(i);
  Moments m;
  if constexpr (Rows) m = moments_of_rows<W>(sets, count, lds, lds_d);
  else m = moments_of_parts<W>(sets, (int)count, lds_d);
  const Scale s = scale_of(a, m, blockIdx.x == 0 && threadIdx.x == 0);
  if constexpr (Hold > 0) {
#pragma unroll
    for (int i = 0; i < Hold; ++i) store(held[i], s);
  } else {
    for (int k = 0; item_index<W>(a, k) < (uint32_t)a.items; ++k) {
      Held nxt;
      const bool more = item_index<W>(a, k + 1) < (uint32_t)a.items;
      if (more) nxt = fetch(k + 1);
      store(held[0], s);
      if (more) held[0] = nxt;
    }
  }
}

// A small batch in one launch: one workgroup holds all positions (rows of at least four) in registers.
__global__ __launch_bounds__(kWhSmallThreads) void whiten_small_kernel(WhArgs a) {
  __shared__ double lds[3 * kWhSmallWaves];
  const uint32_t T = (uint32_t)a.T, total = (uint32_t)(a.B * a.T);
  f32x4 g[kWhSmallQuads];
  uint32_t in[kWhSmallQuads];
  const int quads = (int)((total + 4 * kWhSmallThreads - 1) / (4 * kWhSmallThreads));
#pragma unroll
  for (int u = 0; u < kWhSmallQuads; ++u) {
    in[u] = 0;
    g[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t f = ((uint32_t)u * kWhSmallThreads + threadIdx.x) * 4u;
    if (u < quads && f < total) {  // the four positions lie in one row or at the end of it and the start of the next
      const uint32_t row = f / T, t = f - row * T;
      auto valid = [&](uint32_t r) {
        const int32_t L = r < (uint32_t)a.B ? a.lengths[r] : 0;
        return L < 0 ? 0u : min((uint32_t)L, T);
      };
      const uint32_t L0 = valid(row), L1 = t + 4u > T ? valid(row + 1u) : 0u;
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) in[u] |= (t + j < T ? t + j < L0 : t + j - T < L1) ? 1u << j : 0u;
      if (in[u] == 0xfu) {
        g[u] = *(const f32x4*)(a.adv + f);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if ((in[u] >> j) & 1u) g[u][j] = a.adv[f + (uint32_t)j];
      }
    }
  }
  const double shift = batch_shift(a);
  LaneSums w;
#pragma unroll
  for (int u = 0; u < kWhSmallQuads; ++u)
    if (u < quads) w.add(g[u], in[u], shift);
  double v[3] = {w.s1, w.s2, (threadIdx.x & (kWave - 1)) == 0 ? (double)w.n : 0.0};
  block_sums<kWhSmallWaves>(v, lds);
  const double md = v[2] > 0.0 ? v[0] / v[2] : 0.0;
  const Scale s = scale_of(a, Moments{v[2], shift + md, fma(-v[2] * md, md, v[1])}, threadIdx.x == 0);
#pragma unroll
  for (int u = 0; u < kWhSmallQuads; ++u)
    if (u < quads) store_quad(a.out + ((uint32_t)u * kWhSmallThreads + threadIdx.x) * 4u, g[u], in[u], s);
}

// Items of a row: one that starts between boundaries spans up to 3 positions more.
int64_t items_per_row(int64_t T) { return (T + (T % 4 != 0 ? 3 : 0) + kWhItem - 1) / kWhItem; }

// An item for every wave of the smaller workgroups, up to what the chip holds of the larger ones.
int whiten_groups(int64_t items) {
  const int64_t want = (items + 7) / 8;
  return (int)(want < 1 ? 1 : (want > kWhMaxGroups ? kWhMaxGroups : want));
}

// The rewrite of these arguments.
template <bool Rows>
int launch_apply(const WhArgs& a, const Sums* sets, int64_t count, hipStream_t stream) {
  const int64_t waves = (int64_t)a.groups * 8;
  static_assert(kWhHold == 4, "the three sizes below");
  const bool eight = a.items <= kWhHold * waves;
  const auto kernel = a.items <= waves ? whiten_apply_kernel<Rows, 8, 1> : a.items <= 2 * waves ? whiten_apply_kernel<Rows, 8, 2>
                      : eight ? whiten_apply_kernel<Rows, 8, 4> : whiten_apply_kernel<Rows, 16, 0>;
  hipLaunchKernelGGL(kernel, dim3(a.groups), dim3((eight ? 8 : 16) * kWave), 0, stream, a, sets, count);
  return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
}

WhArgs whiten_args(const float* adv, const int32_t* lengths, int64_t B, int64_t T, float eps, int shift_mean, int unbiased,
                   float* out, double* stats) {
  WhArgs a;
  a.adv = adv;
  a.lengths = lengths;
  a.B = B;
  a.T = T;
  a.nch = items_per_row(T);
  a.items = B * a.nch;
  a.groups = whiten_groups(a.items);
  a.eps = eps;
  a.shift_mean = shift_mean;
  a.ddof = unbiased ? 1 : 0;
  a.out = out;
  a.stats = stats;
  a.part = nullptr;
  return a;
}

}  // namespace

// item_index counts in 32 bits, and past the last item by up to kWhUnroll rounds of the waves.
bool whiten_indexable(int64_t B, int64_t T) {
  constexpr int64_t kRoom = 1 << 15;
  static_assert((kWhUnroll + 1) * 16 * kWhMaxGroups <= kRoom, "room for the index of a loop's last step");
  return B * ((T + 3 + kWhItem - 1) / kWhItem) < (1ll << 32) - kRoom;
}

// Room for a partial for each 4096 positions of a row, up to the most a launch has: never more for fewer rows or steps, so that
// a buffer sized for a program's largest call serves all its calls.  (Workgroups go by items, of which 65535 positions
// have one more than 65536; 4096 positions are at most five items, five eighths of a workgroup, so there is always room.)
size_t whiten_workspace(int64_t B, int64_t T) {
  static_assert(kWhItem == 1024, "five items in 4096 positions");
  const int64_t parts = B * ((T + 4095) / 4096);
  return (size_t)(parts < 1 ? 1 : parts > kWhMaxGroups ? kWhMaxGroups : parts) * sizeof(Sums);
}

int launch_whiten(const float* adv, const int32_t* lengths, int64_t B, int64_t T, float eps, int shift_mean,
                  int unbiased, float* out, double* stats, void* workspace, hipStream_t stream) {
  WhArgs a = whiten_args(adv, lengths, B, T, eps, shift_mean, unbiased, out, stats);
  if (T >= 4 && B * T <= kWhSmall) {
    hipLaunchKernelGGL(whiten_small_kernel, dim3(1), dim3(kWhSmallThreads), 0, stream, a);
    return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
  }
  a.part = (Sums*)workspace;
  const bool eight = a.items <= kWhEightWavesTo;
  hipLaunchKernelGGL(eight ? whiten_partial_kernel<8> : whiten_partial_kernel<16>, dim3(a.groups), dim3((eight ? 8 : 16) * kWave), 0, stream, a);
  if (hipGetLastError() != hipSuccess) return ESPO_EHIP;
  return launch_apply<false>(a, a.part, a.groups, stream);
}

int launch_whiten_rows(const float* adv, const int32_t* lengths, int64_t B, int64_t T, float eps, int shift_mean,
                       int unbiased, float* out, double* stats, const AdvRowStats* rows, hipStream_t stream) {
  const WhArgs a = whiten_args(adv, lengths, B, T, eps, shift_mean, unbiased, out, stats);
  return launch_apply<true>(a, rows, B, stream);
}

}  // namespace espo
