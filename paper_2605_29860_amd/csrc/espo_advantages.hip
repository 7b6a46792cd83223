// espo_advantages: TD errors and GAE on truncated trajectories (Section 3: delta_t and
// Eq. gae; Section 4.4: failure reward at the stop step, no bootstrap past the end).
//
// A_t = delta_t + c A_{t+1} (c = gamma*lambda) is a first-order linear recurrence that
// runs backwards over each row's valid prefix [0, L).  One workgroup of 16 wavefronts owns
// one row and walks it in tiles of 4096 tokens from the tile that holds L-1 down to tile 0;
// tiles at or beyond L are only zero-filled.  Inside a tile every lane holds 4 consecutive
// tokens (one 16-byte load per input array, one 16-byte store per output array), and the
// lanes are laid out backwards: thread 0 holds the tile's last four tokens.  That turns the
// suffix sums of the recurrence into prefix sums over the lanes, which the DPP row shifts
// and row broadcasts of gfx9 compute in six steps without touching LDS; the sixteen wave
// totals are combined the same way after one trip through LDS, and a single scalar carries A
// across the tile boundary.  Only that scalar depends on the previous tile, so the next
// tile's loads are issued before the current one is reduced.
//
// The same kernel serves the terminal-reward form (the rewards of Algorithm 1: zero at every
// step that goes on, one reward at the last): no reward array is read, the last token takes
// r_fail or the row's terminal reward, and on request the value targets A_t + V(s_t) are
// stored and the padding beyond the lengths is left alone.
//
// It also serves trajectories stored back to back (extents from cu_seqlens) and rows whose length
// is no multiple of four: the workgroup then works on the span that starts at the 16-byte
// boundary at or before the row's first token, so every lane still moves 16 aligned bytes; the up
// to three tokens before the first one belong to the neighbour, come last in the backward scan
// (nothing valid depends on them) and are not stored, and neither is anything at or after the end
// of what the row owns.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/espo.h"
#include "espo_device.h"
#include "espo_host.h"

namespace espo {
namespace {

// A workgroup has W wavefronts (a template parameter of what depends on it): 16, or 8 with two spans of 256 tokens each, for tiles of
// 4096 tokens; 4 for tiles of 1024.
constexpr int kPerLane = 4;
constexpr int kWaveTokens = kWave * kPerLane;
constexpr int kPair = 2;                          // inner tiles of a workgroup of 4 waves that share a barrier
constexpr int kDppWaveShr1 = 0x138;               // lane i takes lane i-1 across the whole wave

struct AdvArgs {
  const float* rewards;          // dense form: [B, T]
  const float* terminal_reward;  // terminal form: [B]
  float* returns;                // optional [B, T]: A_t + V(s_t)
  int32_t zero_padding;          // write zeros at t >= L (else those positions are not written by whole lanes)
  const float* values;
  const int64_t* cu;             // packed form: [B + 1] extents into arrays of N tokens
  int64_t N;
  const int32_t* lengths;
  const uint8_t* stopped;
  int64_t T;
  int32_t B;  // rows; with zero padding and more than one tile per row the grid has 2 B workgroups, the second B only fill
  int32_t ordered_from;  // rows from here on (kAdvFirstRows or none) are scanned longest first
  float r_fail, gamma, c;
  float cj[kPerLane + 1];  // c^0 .. c^4
  float clane[6];          // c^(4*2^k), k = 0..5: a distance of 2^k lanes
  float cwave[5];          // c^(256*2^k), k = 0..4: a distance of 2^k waves; cwave[log2 W] spans a tile
  float* td;
  float* adv;
  const int32_t* order;    // optional [B]: the rows, longest first (padded forms)
  AdvRowStats* row_stats;  // optional [B]: sums of every row's advantages (padded forms)
  int32_t* sorted;         // optional [B - kAdvFirstRows]: the rows from kAdvFirstRows on, longest first, written by
                           //   workgroup 0 of this launch (padded forms in workgroups of 8 or 16 waves, no `order` given)
  uint32_t* sync;          // with `sorted`: [0] set once `sorted` is complete, [32] readers so far; both 0 between launches
};

// Workgroups that the chip holds at once (256 CUs x 2 of 1024 threads): the rows that are scanned first whatever
// their lengths.  Only the order of the rows that follow decides how ragged the launch's end is (measured: rows
// 512.. of 1024 longest first gives what a full order gives, 39.9 us against 45.3 in index order; rows 768.. 43.3).
constexpr int kAdvFirstRows = 512;
// The order is followed in batches of at most three rows per workgroup slot, where it decides how ragged the launch's
// end is, and only for rows of several tiles, which take longer than finding one's row (2 to 3 us); us per launch
// with / without: B = 1024, T = 16384: 39.5 / 43.0; 9000: 25.0 / 26.0; B = 1300, T = 16384: 50.3 / 53.2;
// B = 2000, T = 10000: 52.1 / 48.0, T = 3000: 30.6 / 22.6; B = 1024, T = 1500: 13.2 / 10.9.
constexpr int kAdvSelectRows = 3 * kAdvFirstRows;
constexpr int64_t kAdvSelectTokens = 8192;
// Read from a list that the launch makes, the order costs its readers one load, so it pays for shorter rows, too; us per
// launch with / without, dense: T = 4100: B = 1024: 19.5 / 17.3, 1536: 28.5 / 26.4; T = 5000: B = 800: 17.7 / 19.2,
// 1024: 20.9 / 22.4, 1536: 30.2 / 29.4; T = 8192: B = 1024: 24.1 / 25.8 (terminal rewards, padding filled: 24.2 / 26.0).
constexpr int64_t kAdvSortTokens = 4608;
// The word that says "sorted" and the count of its readers lie in different 128-byte lines: loads of the one and
// read-modify-writes of the other on the same line cost the readers 15 us per launch between them.
constexpr int kAdvSyncStride = 32;       // words
constexpr size_t kAdvSyncBytes = 256;
constexpr int64_t kAdvOnePerUnit = 256;  // rows: one for every compute unit at most
constexpr int64_t kAdvFiveArrays = 13824;  // twice the mean length
constexpr int kOrderClasses = 256;

__device__ __forceinline__ int class_of_length(int64_t L, int64_t T) {  // class 0 is the longest
  L = L < 0 ? 0 : (L > T ? T : L);
  return kOrderClasses - 1 - (int)((L * kOrderClasses) / (T + 1));
}

// Writes the rows first .. B-1 to order[0 .. B-first), longest first: a counting sort of the clipped lengths into
// 256 classes by one workgroup of W waves, 4 at least (rows of one class in no particular order; no result depends on it).  The entries
// are written past the caches that other parts of the chip do not see, and are complete when the call returns.
template <int W>
__device__ __forceinline__ void sort_rows_by_length(const int32_t* __restrict__ lengths, int32_t first, int32_t B, int64_t T,
                                                    int32_t* __restrict__ order) {
  __shared__ int count[kOrderClasses];
  __shared__ int wave_total[kOrderClasses / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  auto class_of = [&](int32_t i) { return class_of_length(lengths[i], T); };
  if (tid < kOrderClasses) count[tid] = 0;
  __syncthreads();
  for (int32_t i = first + tid; i < B; i += W * kWave) atomicAdd(&count[class_of(i)], 1);
  __syncthreads();
  int mine = 0, incl = 0;
  if (tid < kOrderClasses) {  // inclusive prefix over the classes: inside each wave, then over the four waves
    mine = count[tid];
    incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int up = __shfl_up(incl, d);
      if (lane >= d) incl += up;
    }
    if (lane == kWave - 1) wave_total[tid >> 6] = incl;
  }
  __syncthreads();
  if (tid < kOrderClasses) {
    int before = 0;
    for (int w = 0; w < (tid >> 6); ++w) before += wave_total[w];
    count[tid] = before + incl - mine;  // where the class starts
  }
  __syncthreads();
  for (int32_t i = first + tid; i < B; i += W * kWave)
    __hip_atomic_store(order + atomicAdd(&count[class_of(i)], 1), i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// The k-th of the rows first .. B-1 in order of their classes (class 0 first; inside a class by index), found by the calling workgroup for itself: every workgroup that asks gets the same permutation, so
// no memory and no waiting is needed.  All threads must call it; the result is uniform.
template <int W, typename ClassOf>
__device__ __forceinline__ int32_t kth_row_by_length(ClassOf&& class_of, int32_t first, int32_t B, int32_t k) {
  __shared__ int count[kOrderClasses];
  __shared__ int wave_total[W];
  __shared__ int s_class, s_rank, s_found;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  if (tid < kOrderClasses) count[tid] = 0;
  if (tid == 0) s_found = -1;
  __syncthreads();
  for (int32_t i = first + tid; i < B; i += W * kWave) atomicAdd(&count[class_of(i)], 1);
  __syncthreads();
  int mine = 0, incl = 0;
  if (tid < kOrderClasses) {  // inclusive prefix over the classes: inside each wave, then over the four waves
    mine = count[tid];
    incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int up = __shfl_up(incl, d);
      if (lane >= d) incl += up;
    }
    if (lane == kWave - 1) wave_total[wave] = incl;
  }
  __syncthreads();
  if (tid < kOrderClasses) {
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wave_total[w];
    const int start = before + incl - mine;  // where the class starts
    if (k >= start && k < start + mine) {
      s_class = tid;
      s_rank = k - start;
    }
  }
  __syncthreads();
  const int want_class = s_class, want_rank = s_rank;
  int seen = 0;  // rows of the class before this chunk (uniform)
  for (int32_t chunk = first; chunk < B; chunk += W * kWave) {
    const int32_t i = chunk + tid;
    const bool in = i < B && class_of(i) == want_class;
    const uint64_t who = __builtin_amdgcn_ballot_w64(in);
    if (lane == 0) wave_total[wave] = (int)__builtin_popcountll(who);
    __syncthreads();
    int before = seen, all = 0;
    for (int w = 0; w < W; ++w) {
      const int n = wave_total[w];
      before += w < wave ? n : 0;
      all += n;
    }
    if (in && before + (int)__builtin_popcountll(who & ((1ull << lane) - 1ull)) == want_rank) s_found = i;
    seen += all;
    __syncthreads();
    if (seen > want_rank) break;  // (uniform) found in this chunk
  }
  return s_found;
}

struct TileIn {
  float r[kPerLane], v[kPerLane];
  float halo;  // value of the token after the wave's span (lane 0 only)
};

// c^(unit * e) for 0 <= e < 2^Bits from the table of c^(unit * 2^k).
template <int Bits>
__device__ __forceinline__ float pow_from_table(const float* tab, int e) {
  float w = 1.0f;
#pragma unroll
  for (int k = 0; k < Bits; ++k)
    if (e & (1 << k)) w *= tab[k];
  return w;
}

// Loads the lane's 4 tokens starting at t0 and, in lane 0, the value at t0 + 4; tokens at or
// beyond L are never read.
// Positions are of type Pos: 64-bit ones of a row, or 32-bit ones of a tile.
template <bool Dense, typename Pos>
__device__ __forceinline__ TileIn load_tile(const float* __restrict__ rrow, const float* __restrict__ vrow, Pos t0,
                                            Pos L, bool want_halo) {
  TileIn in;
#pragma unroll
  for (int j = 0; j < kPerLane; ++j) { in.r[j] = 0.0f; in.v[j] = 0.0f; }
  in.halo = 0.0f;
  if (t0 + kPerLane <= L) {
    if constexpr (Dense) {
      const f32x4 a = __builtin_nontemporal_load((const f32x4*)(rrow + t0));
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) in.r[j] = a[j];
    }
    const f32x4 b = __builtin_nontemporal_load((const f32x4*)(vrow + t0));
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) in.v[j] = b[j];
  } else {
#pragma unroll
    for (int j = 0; j < kPerLane; ++j)
      if (t0 + j < L) {
        if constexpr (Dense) in.r[j] = rrow[t0 + j];
        in.v[j] = vrow[t0 + j];
      }
  }
  if (want_halo && t0 + kPerLane < L) in.halo = vrow[t0 + kPerLane];
  return in;
}

// Stores x at t0 .. t0 + 3 where the row goes on (T % 4 == 0 here).
template <typename Pos>
__device__ __forceinline__ void store4(float* __restrict__ row, Pos t0, Pos T, const float x[kPerLane]) {
  if (t0 < T) __builtin_nontemporal_store(f32x4{x[0], x[1], x[2], x[3]}, (f32x4*)(row + t0));
}

// Stores x[j] at t0 + j for lo <= t0 + j < hi (t0 a multiple of 4, the row 16-byte aligned).
template <typename Pos>
__device__ __forceinline__ void store_span(float* __restrict__ row, Pos t0, Pos lo, Pos hi, const float x[kPerLane]) {
  if (t0 >= lo && t0 + kPerLane <= hi) {
    __builtin_nontemporal_store(f32x4{x[0], x[1], x[2], x[3]}, (f32x4*)(row + t0));
    return;
  }
#pragma unroll
  for (int j = 0; j < kPerLane; ++j)
    if (t0 + j >= lo && t0 + j < hi) row[t0 + j] = x[j];
}

// One step of a weighted inclusive prefix sum over lanes: s += w * (s of the lane the DPP control names).
template <int Ctrl, int RowMask>
__device__ __forceinline__ float scan_step(float s, float w) {
  return fmaf(w, dpp_f32<Ctrl, RowMask>(0.0f, s), s);
}

// The tiles last .. 1 of a trajectory stored back to back, in a workgroup of 4 waves.  The number of waves follows from the
// mean length, so a trajectory many times as long can come this way, and four waves are alone on their SIMDs: what
// bounds them is what they issue and the chain of each tile, not memory.  These tiles lie wholly inside the trajectory and none is
// its last: nothing is checked, addresses are 32-bit offsets from a uniform base, and two tiles share a barrier while the next
// two are on their way.  us per call, with the loop below for every tile / with this / with workgroups of 16 waves:
//   1000 trajectories of 300 tokens and one of 100000: 83.6 / 40.1 / 35.0;  512 of 400, one of 16384: 16.0 / 9.7 / 10.2;
//   63 of 100, one of 30000: 25.9 / 14.3 / 11.7;  256 of 250, one of 4000: 5.9 / 5.0 / 5.2;
//   1024 of up to 500, 1000, 3800 tokens: 5.5, 5.8, 11.7 / 5.5, 5.9, 10.3 / 9.9, 10.4, 11.9.
// Takes A at the first token after tile `last`, returns A at tile 1's first.
template <bool Dense>
__device__ __forceinline__ float walk_inner(const AdvArgs& a, const float* __restrict__ r, const float* __restrict__ v, float* __restrict__ td,
                                            float* __restrict__ adv, float* __restrict__ ret, int64_t last, float carry,
                                            float w_b15, float w_b31, float w_lane, float w_wave) {
  constexpr int kTile = 4 * kWaveTokens;
  __shared__ float s_tot[2][4 * kPair];  // wave totals of a group, double-buffered
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t at = (uint32_t)(4 * kWave - 1 - threadIdx.x) * kPerLane;
  struct In {
    f32x4 r, v;
    float halo;
  };
  auto load = [&](int64_t k) {
    In in;
    in.r = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (Dense) in.r = __builtin_nontemporal_load((const f32x4*)(r + k * kTile + at));
    in.v = __builtin_nontemporal_load((const f32x4*)(v + k * kTile + at));
    in.halo = 0.0f;
    if (lane == 0) in.halo = v[k * kTile + at + kPerLane];
    return in;
  };
  In ring[2][kPair];
  auto fetch = [&](In (&to)[kPair], int64_t k) {
#pragma unroll
    for (int g = 0; g < kPair; ++g)
      if (k - g > 0) to[g] = load(k - g);
  };
  fetch(ring[0], last);
  int par = 0;
#pragma unroll 1
  for (int64_t k0 = last; k0 > 0; k0 -= kPair) {
    fetch(ring[1], k0 - kPair);
    f32x4 d[kPair], loc[kPair];
    float s[kPair];
#pragma unroll
    for (int g = 0; g < kPair; ++g) {
      if (k0 - g <= 0) break;  // (uniform)
      const In& in = ring[0][g];
      float vnext = dpp_f32<kDppWaveShr1, 0xf>(0.0f, in.v[0]);
      if (lane == 0) vnext = in.halo;
      float acc = 0.0f;
#pragma unroll
      for (int j = kPerLane - 1; j >= 0; --j) {
        d[g][j] = (in.r[j] + a.gamma * (j == kPerLane - 1 ? vnext : in.v[j + 1])) - in.v[j];
        acc = d[g][j] + a.c * acc;
        loc[g][j] = acc;
      }
      s[g] = acc;
    }
    // the scan over the lanes, step by step for all of them
#pragma unroll
    for (int g = 0; g < kPair; ++g) s[g] = scan_step<kDppRowShr1, 0xf>(s[g], a.clane[0]);
#pragma unroll
    for (int g = 0; g < kPair; ++g) s[g] = scan_step<kDppRowShr2, 0xf>(s[g], a.clane[1]);
#pragma unroll
    for (int g = 0; g < kPair; ++g) s[g] = scan_step<kDppRowShr4, 0xf>(s[g], a.clane[2]);
#pragma unroll
    for (int g = 0; g < kPair; ++g) s[g] = scan_step<kDppRowShr8, 0xf>(s[g], a.clane[3]);
#pragma unroll
    for (int g = 0; g < kPair; ++g) s[g] = scan_step<kDppBcast15, 0xa>(s[g], w_b15);
#pragma unroll
    for (int g = 0; g < kPair; ++g) {
      s[g] = scan_step<kDppBcast31, 0xc>(s[g], w_b31);
      if (lane == kWave - 1) s_tot[par][g * 4 + wave] = s[g];
    }
    __syncthreads();
    // lanes 4 g .. 4 g + 3 hold the totals of tile g; the scan over four of them does not cross into the next
    float p = lane < 4 * kPair ? s_tot[par][lane] : 0.0f;
    const float p1 = dpp_f32<kDppRowShr1, 0xf>(0.0f, p);
    p = (lane & 3) >= 1 ? fmaf(a.cwave[0], p1, p) : p;
    const float p2 = dpp_f32<kDppRowShr2, 0xf>(0.0f, p);
    p = (lane & 3) >= 2 ? fmaf(a.cwave[1], p2, p) : p;
#pragma unroll
    for (int g = 0; g < kPair; ++g) {
      const int64_t k = k0 - g;
      if (k <= 0) break;  // (uniform)
      const float before = wave > 0 ? uniform_f32(p, 4 * g + wave - 1) : 0.0f;
      const float wave_in = fmaf(w_wave, carry, before);
      carry = fmaf(a.cwave[2], carry, uniform_f32(p, 4 * g + 3));
      const float a_next = fmaf(w_lane, wave_in, dpp_f32<kDppWaveShr1, 0xf>(0.0f, s[g]));
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) loc[g][j] = fmaf(a.cj[kPerLane - j], a_next, loc[g][j]);
      __builtin_nontemporal_store(d[g], (f32x4*)(td + k * kTile + at));
      __builtin_nontemporal_store(loc[g], (f32x4*)(adv + k * kTile + at));
      if (ret) __builtin_nontemporal_store(loc[g] + ring[0][g].v, (f32x4*)(ret + k * kTile + at));
    }
#pragma unroll
    for (int g = 0; g < kPair; ++g) ring[0][g] = ring[1][g];
    par ^= 1;
  }
  return carry;
}

// Layout of the rows: [B, T] with T a multiple of four, [B, T] with any T, or back to back.
enum RowLayout { kAligned, kShifted, kPacked };

// What a workgroup has to do: its row, where the row's tokens lie and what its last token's reward is.  False: nothing.
struct Row {
  bool fill_only;      // zeros beyond the trajectory, and nothing else
  int32_t row;
  int64_t T, L, head;  // from the row's 16-byte boundary on: its end, the end of its valid part, its start
  bool last_given;     // the reward of the last token is r_last, wherever the others come from
  float r_last;
  const float *rewards, *values;
  float *td, *adv, *returns;
};

template <bool Dense, RowLayout Layout, int W>
__device__ __forceinline__ bool open_row(const AdvArgs& a, Row& r) {
  // With zero padding, the tiles wholly beyond a trajectory are filled by a workgroup of their
  // own (the second half of the grid): the two kinds of work of a row are then dispatched
  // separately, which evens out the rows (a row costs 16 bytes per valid and 8 per padded token):
  // 2 to 3 us on the B = 1024, T = 16384 batches when their rows come in order of length, nothing
  // when they come in random order.  (Ranking the rows by length inside every workgroup, 8 or 64
  // classes, cost 3 to 5 us per launch, as much as the order gains; only the order of the rows that do
  // not fit the chip at once matters, and only their scans look their row up: see below.)
  constexpr bool Packed = Layout == kPacked, kOrdered = W != 4;  // of the smallest workgroups, for short rows, the chip holds 2048, and rows differ little
  int unit = (int)blockIdx.x;
  if (kOrdered && !Packed && a.sorted) {
    // No order was given and the later rows are to be scanned longest first: workgroup 0 of this launch
    // sorts them while the first kAdvFirstRows are being scanned, and tells the others when it is done.
    // It waits for nobody and is dispatched before every workgroup that waits for it.
    if (unit == 0) {
      sort_rows_by_length<W>(a.lengths, kAdvFirstRows, a.B, a.T, a.sorted);
      if (threadIdx.x == 0) __hip_atomic_store(a.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
    unit -= 1;
  }
  r.fill_only = !Packed && unit >= a.B;
  const bool fill_only = r.fill_only;
  int row = fill_only ? unit - a.B : unit;
  // Rows in order of length: the long scans start first and the short ones fill the launch's end (the
  // workgroups that only fill take the rows the other way round: the shortest row has the most padding).
  // An entry that names no row makes its workgroup do nothing.
  if (!Packed && a.order) {
    row = a.order[fill_only ? a.B - 1 - row : row];
    if ((unsigned)row >= (unsigned)a.B) return false;
  } else if (kOrdered && !Packed && a.sorted && !fill_only && row >= a.ordered_from) {
    // one of the later scans: its row comes from the sorted list.  The last reader clears the two words, so the
    // next launch finds them as this one did.
    __shared__ int s_row;
    if (threadIdx.x == 0) {
      while (__hip_atomic_load(a.sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) __builtin_amdgcn_s_sleep(8);
      s_row = __hip_atomic_load(a.sorted + (row - kAdvFirstRows), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t readers = (uint32_t)(a.B - kAdvFirstRows);
      if (atomicInc(a.sync + kAdvSyncStride, readers - 1u) == readers - 1u)
        __hip_atomic_store(a.sync, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    row = s_row;
    if ((unsigned)row >= (unsigned)a.B) return false;
  } else if (kOrdered && !fill_only && row >= a.ordered_from) {
    // No order and nowhere to keep one: each of the later scans finds its row for itself, the
    // (row - kAdvFirstRows)-th longest of the later rows (five barriers and a few hundred LDS operations
    // before its first load, while the other workgroups of the compute unit stream).  Measured on the
    // B = 1024, T = 16384 batches: 40.6 against 43.7 us per launch; stored back to back 30.5 against 33.0.
    // Without a T, the classes of length divide up to four times the mean length.
    if constexpr (Packed) {
      const int64_t most = 4 * (a.N / a.B) + 3;
      row = kth_row_by_length<W>([&](int32_t i) { return class_of_length(a.cu[i + 1] - a.cu[i], most); }, kAdvFirstRows, a.B, row - kAdvFirstRows);
    } else {
      row = kth_row_by_length<W>([&](int32_t i) { return class_of_length(a.lengths[i], a.T); }, kAdvFirstRows, a.B, row - kAdvFirstRows);
    }
    if ((unsigned)row >= (unsigned)a.B) return false;
  }
  int64_t T = a.T;
  int64_t L, base = (int64_t)row * T, head = 0;
  if constexpr (Packed) {
    // extent clipped to the arrays; the span starts at the 16-byte boundary at or before it
    int64_t first = a.cu[row], end = a.cu[row + 1];
    first = first < 0 ? 0 : (first > a.N ? a.N : first);
    end = end > a.N ? a.N : end;
    if (end <= first) return false;
    base = first & ~(int64_t)(kPerLane - 1);
    head = first - base;
    L = end - base;
    T = L;
  } else {
    L = a.lengths[row];
    L = L < 0 ? 0 : (L > T ? T : L);
    if constexpr (Layout == kShifted) {  // positions count from the boundary: the row is [head, T), its valid part [head, L)
      head = base & (kPerLane - 1);
      base -= head;
      L = L > 0 ? L + head : 0;
      T += head;
    }
  }
  const bool stopped = a.stopped[row] != 0;
  // reward of the last token where it does not come from the reward array: r_fail after a stop
  // (Eq. failure_reward), the row's terminal reward in the terminal form
  const bool last_given = stopped || !Dense;
  float r_last = a.r_fail;
  if (!Dense && !stopped) r_last = a.terminal_reward[row];
  r.row = row;
  r.T = T;
  r.L = L;
  r.head = head;
  r.last_given = last_given;
  r.r_last = r_last;
  r.rewards = Dense ? a.rewards + base : nullptr;
  r.values = a.values + base;
  r.td = a.td + base;
  r.adv = a.adv + base;
  r.returns = a.returns ? a.returns + base : nullptr;
  return true;
}


// The sums of a row's n advantages from those of its threads: lanes, then waves, in a fixed order.
template <int W>
__device__ __forceinline__ void leave_row_stats(const AdvArgs& a, int32_t row, double s1, double s2, double shift, int64_t n) {
  __shared__ double s_stats[2][W];
  const int wave = threadIdx.x >> 6;
  s1 = wave_sum_f64(s1);
  s2 = wave_sum_f64(s2);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s_stats[0][wave] = s1;
    s_stats[1][wave] = s2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t1 = 0.0, t2 = 0.0;
    for (int w = 0; w < W; ++w) {
      t1 += s_stats[0][w];
      t2 += s_stats[1][w];
    }
    a.row_stats[row] = AdvRowStats{t1, t2, shift, (long long)n};
  }
}

template <bool Dense, RowLayout Layout, int W>
__global__ __launch_bounds__(W * kWave, W == 4 ? (Dense && Layout == kPacked ? 5 : 6) : 8) void espo_advantages_kernel(AdvArgs a) {
  constexpr bool Packed = Layout == kPacked, Span = Layout != kAligned;
  constexpr int kTile = W * kWaveTokens;
  __shared__ float s_tot[2][W];  // wave totals, double-buffered by tile parity
  Row r;
  if (!open_row<Dense, Layout, W>(a, r)) return;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t row = r.row;
  const int64_t T = r.T, L = r.L, head = r.head;
  const bool fill_only = r.fill_only, last_given = r.last_given;
  const float r_last = r.r_last;
  const float *const rrow = r.rewards, *const vrow = r.values;
  float *const drow = r.td, *const arow = r.adv, *const trow = r.returns;

  const int64_t ntiles = (T + kTile - 1) / kTile;
  const int64_t nvalid = (L + kTile - 1) / kTile;  // tiles that hold at least one valid token
  const int64_t lane_off = (int64_t)(W * kWave - 1 - tid) * kPerLane;  // backwards: thread 0 holds the last tokens

  auto put = [&](float* out, int64_t t0, const float x[kPerLane]) {  // what the row owns of four positions
    if constexpr (Span) store_span(out, t0, head, Packed ? L : T, x);
    else store4(out, t0, T, x);
  };
  // tiles wholly beyond the trajectory: outputs are exactly zero
  const float zero[kPerLane] = {0, 0, 0, 0};
  if (fill_only) {
    for (int64_t k = ntiles - 1; k >= nvalid; --k) {
      put(drow, k * kTile + lane_off, zero);
      put(arow, k * kTile + lane_off, zero);
      if (trow) put(trow, k * kTile + lane_off, zero);
    }
    return;
  }
  if (nvalid == 0) {
    if (!Packed && a.zero_padding && T <= kTile) {  // a row of one tile has no workgroup that only fills
      put(drow, lane_off, zero);
      put(arow, lane_off, zero);
      if (trow) put(trow, lane_off, zero);
    }
    if (!Packed && a.row_stats && tid == 0) a.row_stats[row] = AdvRowStats{0.0, 0.0, 0.0, 0};
    return;
  }
  // Sums of the row's advantages for the batch statistics, in double about the advantage of the row's
  // last token (r - V there: nothing is bootstrapped beyond the end), which every thread can form.
  const bool want_stats = !Packed && a.row_stats != nullptr;
  double st_shift = 0.0, st_s1 = 0.0, st_s2 = 0.0;
  if (want_stats) st_shift = (double)((last_given ? r_last : rrow[L - 1]) - vrow[L - 1]);

  // per-lane weights of the cross-row scan steps and of the carry into this lane and this wave
  const float w_b15 = pow_from_table<5>(a.clane, (lane & 15) + 1);  // from lane 15 of the row before
  const float w_b31 = pow_from_table<6>(a.clane, (lane & 31) + 1);  // from lane 31
  const float w_lane = pow_from_table<6>(a.clane, lane);            // c^(4 lane): the wave's carry-in seen from this lane
  const float w_wave = pow_from_table<4>(a.cwave, wave);            // c^(256 wave): the tile's carry-in seen from this wave

  float carry = 0.0f;  // A at the first token of the tile processed before (the later one)
  TileIn cur = load_tile<Dense>(rrow, vrow, (nvalid - 1) * kTile + lane_off, L, lane == 0);
  for (int64_t k = nvalid - 1; k >= 0; --k) {
    const int64_t t0 = k * kTile + lane_off;
    TileIn nxt;
    if (k > 0) nxt = load_tile<Dense>(rrow, vrow, Packed && W == 4 ? lane_off : t0 - kTile, L, lane == 0);  // the earlier tile, in flight during the scan

    // V_{t+1} of the lane's last token: first value of the lane that holds the following tokens
    float vnext = dpp_f32<kDppWaveShr1, 0xf>(0.0f, cur.v[0]);
    if (lane == 0) vnext = cur.halo;

    // delta_t and the recurrence over the lane's 4 tokens, later tokens first
    const int64_t rem = L - t0;  // valid tokens from t0 on (may be <= 0 or large)
    float d[kPerLane], loc[kPerLane];
    float acc = 0.0f;
    if (__builtin_amdgcn_ballot_w64(rem <= kPerLane) == 0) {  // whole wave strictly inside the trajectory
#pragma unroll
      for (int j = kPerLane - 1; j >= 0; --j) {
        const float vn = (j == kPerLane - 1) ? vnext : cur.v[j + 1];
        d[j] = (cur.r[j] + a.gamma * vn) - cur.v[j];
        acc = d[j] + a.c * acc;
        loc[j] = acc;
      }
    } else {
#pragma unroll
      for (int j = kPerLane - 1; j >= 0; --j) {
        float vn = (j == kPerLane - 1) ? vnext : cur.v[j + 1];
        if (j + 1 >= rem) vn = 0.0f;                        // no bootstrap beyond the last token
        float r = cur.r[j];
        if (last_given && j + 1 == rem) r = r_last;
        float dj = (r + a.gamma * vn) - cur.v[j];
        if (j >= rem) dj = 0.0f;
        d[j] = dj;
        acc = dj + a.c * acc;
        loc[j] = acc;
      }
    }

    // inclusive prefix over the lanes: s_i = sum_{i' <= i} c^(4 (i - i')) acc_i'
    float s = acc;
    s = scan_step<kDppRowShr1, 0xf>(s, a.clane[0]);
    s = scan_step<kDppRowShr2, 0xf>(s, a.clane[1]);
    s = scan_step<kDppRowShr4, 0xf>(s, a.clane[2]);
    s = scan_step<kDppRowShr8, 0xf>(s, a.clane[3]);
    s = scan_step<kDppBcast15, 0xa>(s, w_b15);
    s = scan_step<kDppBcast31, 0xc>(s, w_b31);
    const int par = (int)(k & 1);
    if (lane == kWave - 1) s_tot[par][wave] = s;
    __syncthreads();
    // the same scan over the wave totals, one per lane of the first row
    float p = lane < W ? s_tot[par][lane] : 0.0f;
    p = scan_step<kDppRowShr1, 0xf>(p, a.cwave[0]);
    p = scan_step<kDppRowShr2, 0xf>(p, a.cwave[1]);
    if constexpr (W > 4) {
      p = scan_step<kDppRowShr4, 0xf>(p, a.cwave[2]);
      p = scan_step<kDppRowShr8, 0xf>(p, a.cwave[3]);
    }
    // A at the first token after this wave's span
    const float before = wave > 0 ? uniform_f32(p, wave - 1) : 0.0f;
    const float wave_in = fmaf(w_wave, carry, before);
    carry = fmaf(a.cwave[W == 16 ? 4 : 2], carry, uniform_f32(p, W - 1));  // A at the tile's first token
    // A at the first token after this lane's span
    const float s_prev = dpp_f32<kDppWaveShr1, 0xf>(0.0f, s);
    const float a_next = fmaf(w_lane, wave_in, s_prev);

    float outA[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) outA[j] = (j < rem) ? fmaf(a.cj[kPerLane - j], a_next, loc[j]) : 0.0f;
    float outR[kPerLane] = {0, 0, 0, 0};  // value targets: the lambda-return A_t + V(s_t)
    if (trow) {
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) outR[j] = (j < rem) ? outA[j] + cur.v[j] : 0.0f;
    }
    if ((!Packed && a.zero_padding) || rem > 0) {  // lanes wholly beyond L only ever hold zeros
      put(drow, t0, d);
      put(arow, t0, outA);
      if (trow) put(trow, t0, outR);
    }
    if (want_stats) {
#pragma unroll
      for (int j = 0; j < kPerLane; ++j)
        if (j < rem && (!Span || t0 + j >= head)) {
          const double dd = (double)outA[j] - st_shift;
          st_s1 += dd;
          st_s2 += dd * dd;
        }
    }
    if (k > 0) cur = nxt;
    if constexpr (Packed && W == 4) {
      if (k > 1) {
        carry = walk_inner<Dense>(a, rrow, vrow, drow, arow, trow, k - 1, carry, w_b15, w_b31, w_lane, w_wave);
        k = 1;
      }
    }
  }
  if (want_stats) leave_row_stats<W>(a, row, st_s1, st_s2, st_shift, L - head);
}

// The same walk in workgroups of 8 waves, each of which has two of a tile's 16 spans of 256 tokens: the same scan over the same spans, so
// td and adv are the same bits.  For batches that give every compute unit two rows: a launch's waves start over some 4 us
// where 512 rows have 16 each, which is a third of what such a batch takes.  us per call, 16 waves -> 8, lengths U[64, T]: 512 rows, T = 8192:
// dense 12.2 -> 10.3, with the rows' sums 14.2 -> 12.0, terminal rewards with targets 13.6 -> 12.4, without the fill 10.3 -> 9.1, back to back 11.7 -> 10.9;
// 1024 rows, T = 6000: 20.2 -> 18.9; T = 16384: 39.3 -> 38.6, without the fill 27.3 -> 24.8.  (A wave's two spans next to each
// other: 40 instead of 37.4 back to back.  Four spans and 4 waves: without the fill 8.0 and 25.7, padding filled 12.6 and 49.)
template <bool Dense, RowLayout Layout>
__global__ __launch_bounds__(8 * kWave, 4) void espo_advantages_spans_kernel(AdvArgs a) {
  constexpr bool Packed = Layout == kPacked, Span = Layout != kAligned;
  constexpr int W = 8, G = 2, kSpans = W * G;
  constexpr int kTile = kSpans * kWaveTokens;
  __shared__ float s_tot[2][kSpans];  // the spans' totals, double-buffered by tile parity
  Row r;
  if (!open_row<Dense, Layout, W>(a, r)) return;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t row = r.row;
  const int64_t T = r.T, L = r.L, head = r.head;
  const bool fill_only = r.fill_only, last_given = r.last_given;
  const float r_last = r.r_last;
  const float *const rrow = r.rewards, *const vrow = r.values;
  float *const drow = r.td, *const arow = r.adv, *const trow = r.returns;

  const int64_t ntiles = (T + kTile - 1) / kTile;
  const int64_t nvalid = (L + kTile - 1) / kTile;  // tiles that hold at least one valid token
  // Span g of a tile is the lane's tokens in its wave's g-th; positions count from the tile's first token, whose address
  // is uniform (with 64-bit positions of the row the kernel did not fit its registers).
  auto place = [&](int g) { return ((kSpans - g * W) * kWave - 1 - tid) * kPerLane; };  // backwards: thread 0 holds the last tokens
  auto in_tile = [&](int64_t t, int64_t k) {  // position t of the row, a little beyond the tile's end at most if it lies farther on
    const int64_t off = t - k * kTile;
    return (int32_t)(off < 0 ? 0 : off < kTile + 8 ? off : kTile + 8);
  };
  auto put = [&](float* out, int64_t k, int g, const float x[kPerLane]) {  // what the row owns of four positions
    if constexpr (Span) store_span(out + k * kTile, place(g), in_tile(head, k), in_tile(Packed ? L : T, k), x);
    else store4(out + k * kTile, place(g), in_tile(T, k), x);
  };
  auto load = [&](int64_t k, int g) {
    return load_tile<Dense>(Dense ? rrow + k * kTile : nullptr, vrow + k * kTile, place(g), in_tile(L, k), lane == 0);
  };
  // tiles wholly beyond the trajectory: outputs are exactly zero
  const float zero[kPerLane] = {0, 0, 0, 0};
  if (fill_only) {
    for (int64_t k = ntiles - 1; k >= nvalid; --k) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        put(drow, k, g, zero);
        put(arow, k, g, zero);
        if (trow) put(trow, k, g, zero);
      }
    }
    return;
  }
  if (nvalid == 0) {
    if (!Packed && a.zero_padding && T <= kTile) {  // a row of one tile has no workgroup that only fills
#pragma unroll
      for (int g = 0; g < G; ++g) {
        put(drow, 0, g, zero);
        put(arow, 0, g, zero);
        if (trow) put(trow, 0, g, zero);
      }
    }
    if (!Packed && a.row_stats && tid == 0) a.row_stats[row] = AdvRowStats{0.0, 0.0, 0.0, 0};
    return;
  }
  // Sums of the row's advantages for the batch statistics, in double about the advantage of the row's
  // last token (r - V there: nothing is bootstrapped beyond the end), which every thread can form.
  const bool want_stats = !Packed && a.row_stats != nullptr;
  double st_shift = 0.0, st_s1 = 0.0, st_s2 = 0.0;
  if (want_stats) st_shift = (double)((last_given ? r_last : rrow[L - 1]) - vrow[L - 1]);

  // per-lane weights of the cross-row scan steps and of the carry into this lane and this wave
  const float w_b15 = pow_from_table<5>(a.clane, (lane & 15) + 1);  // from lane 15 of the row before
  const float w_b31 = pow_from_table<6>(a.clane, (lane & 31) + 1);  // from lane 31
  const float w_lane = pow_from_table<6>(a.clane, lane);            // c^(4 lane): the wave's carry-in seen from this lane
  float w_wave[G];                                                  // c^(256 span): the tile's carry-in seen from this span
#pragma unroll
  for (int g = 0; g < G; ++g) w_wave[g] = pow_from_table<4>(a.cwave, g * W + wave);

  float carry = 0.0f;  // A at the first token of the tile processed before (the later one)
  TileIn cur[G];
#pragma unroll
  for (int g = 0; g < G; ++g) cur[g] = load(nvalid - 1, g);
  for (int64_t k = nvalid - 1; k >= 0; --k) {
    TileIn nxt[G];
    if (k > 0) {  // the earlier tile, in flight during the scan
#pragma unroll
      for (int g = 0; g < G; ++g) nxt[g] = load(k - 1, g);
    }

    float d[G][kPerLane], loc[G][kPerLane], s[G];
    const int par = (int)(k & 1);
    const int32_t end = in_tile(L, k);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const TileIn& in = cur[g];
      // V_{t+1} of the lane's last token: first value of the lane that holds the following tokens
      float vnext = dpp_f32<kDppWaveShr1, 0xf>(0.0f, in.v[0]);
      if (lane == 0) vnext = in.halo;

      // delta_t and the recurrence over the lane's 4 tokens, later tokens first
      const int32_t rem = end - place(g);  // valid tokens from the lane's first on (may be <= 0 or large)
      float acc = 0.0f;
      if (__builtin_amdgcn_ballot_w64(rem <= kPerLane) == 0) {  // whole wave strictly inside the trajectory
#pragma unroll
        for (int j = kPerLane - 1; j >= 0; --j) {
          const float vn = (j == kPerLane - 1) ? vnext : in.v[j + 1];
          d[g][j] = (in.r[j] + a.gamma * vn) - in.v[j];
          acc = d[g][j] + a.c * acc;
          loc[g][j] = acc;
        }
      } else {
#pragma unroll
        for (int j = kPerLane - 1; j >= 0; --j) {
          float vn = (j == kPerLane - 1) ? vnext : in.v[j + 1];
          if (j + 1 >= rem) vn = 0.0f;                        // no bootstrap beyond the last token
          float r = in.r[j];
          if (last_given && j + 1 == rem) r = r_last;
          float dj = (r + a.gamma * vn) - in.v[j];
          if (j >= rem) dj = 0.0f;
          d[g][j] = dj;
          acc = dj + a.c * acc;
          loc[g][j] = acc;
        }
      }
      s[g] = acc;
    }
    // inclusive prefix over the lanes: s_i = sum_{i' <= i} c^(4 (i - i')) acc_i', step by step for all spans
#pragma unroll
    for (int g = 0; g < G; ++g) s[g] = scan_step<kDppRowShr1, 0xf>(s[g], a.clane[0]);
#pragma unroll
    for (int g = 0; g < G; ++g) s[g] = scan_step<kDppRowShr2, 0xf>(s[g], a.clane[1]);
#pragma unroll
    for (int g = 0; g < G; ++g) s[g] = scan_step<kDppRowShr4, 0xf>(s[g], a.clane[2]);
#pragma unroll
    for (int g = 0; g < G; ++g) s[g] = scan_step<kDppRowShr8, 0xf>(s[g], a.clane[3]);
#pragma unroll
    for (int g = 0; g < G; ++g) s[g] = scan_step<kDppBcast15, 0xa>(s[g], w_b15);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      s[g] = scan_step<kDppBcast31, 0xc>(s[g], w_b31);
      if (lane == kWave - 1) s_tot[par][g * W + wave] = s[g];
    }
    __syncthreads();
    // the same scan over the spans' totals, one per lane of the first row
    float p = lane < kSpans ? s_tot[par][lane] : 0.0f;
    p = scan_step<kDppRowShr1, 0xf>(p, a.cwave[0]);
    p = scan_step<kDppRowShr2, 0xf>(p, a.cwave[1]);
    p = scan_step<kDppRowShr4, 0xf>(p, a.cwave[2]);
    p = scan_step<kDppRowShr8, 0xf>(p, a.cwave[3]);
    const float carry_in = carry;
    carry = fmaf(a.cwave[4], carry, uniform_f32(p, kSpans - 1));  // A at the tile's first token
#pragma unroll
    for (int g = 0; g < G; ++g) {
      // A at the first token after this span
      const int span = g * W + wave;
      const float before = span > 0 ? uniform_f32(p, span - 1) : 0.0f;
      const float wave_in = fmaf(w_wave[g], carry_in, before);
      // A at the first token after this lane's tokens
      const float s_prev = dpp_f32<kDppWaveShr1, 0xf>(0.0f, s[g]);
      const float a_next = fmaf(w_lane, wave_in, s_prev);
      const int32_t rem = end - place(g);

      float outA[kPerLane];
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) outA[j] = (j < rem) ? fmaf(a.cj[kPerLane - j], a_next, loc[g][j]) : 0.0f;
      float outR[kPerLane] = {0, 0, 0, 0};  // value targets: the lambda-return A_t + V(s_t)
      if (trow) {
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) outR[j] = (j < rem) ? outA[j] + cur[g].v[j] : 0.0f;
      }
      if ((!Packed && a.zero_padding) || rem > 0) {  // lanes wholly beyond L only ever hold zeros
        put(drow, k, g, d[g]);
        put(arow, k, g, outA);
        if (trow) put(trow, k, g, outR);
      }
      if (want_stats) {
#pragma unroll
        for (int j = 0; j < kPerLane; ++j)
          if (j < rem && (!Span || place(g) + j >= in_tile(head, k))) {
            const double dd = (double)outA[j] - st_shift;
            st_s1 += dd;
            st_s2 += dd * dd;
          }
      }
    }
    if (k > 0) {
#pragma unroll
      for (int g = 0; g < G; ++g) cur[g] = nxt[g];
    }
  }
  if (want_stats) leave_row_stats<W>(a, row, st_s1, st_s2, st_shift, L - head);
}

__global__ __launch_bounds__(16 * kWave) void length_order_kernel(const int32_t* __restrict__ lengths, int32_t B, int64_t T,
                                                                  int32_t* __restrict__ order) {
  sort_rows_by_length<16>(lengths, 0, B, T, order);
}

template <RowLayout Layout>
void (*pick_kernel(bool dense, int waves))(AdvArgs) {
  if (waves == 4) return dense ? espo_advantages_kernel<true, Layout, 4> : espo_advantages_kernel<false, Layout, 4>;
  if (waves == 8) return dense ? espo_advantages_spans_kernel<true, Layout> : espo_advantages_spans_kernel<false, Layout>;
  return dense ? espo_advantages_kernel<true, Layout, 16> : espo_advantages_kernel<false, Layout, 16>;
}

}  // namespace

int launch_advantages(const float* rewards, const float* terminal_reward, const float* values, const int32_t* lengths,
                      const int64_t* cu, int64_t N, const uint8_t* stopped, int64_t B, int64_t T, float r_fail, float gamma,
                      float lambda, int zero_padding, float* td, float* adv, float* returns, const int32_t* order,
                      AdvRowStats* row_stats, int32_t* sorted, uint32_t* sync, hipStream_t stream) {
  AdvArgs a;
  a.order = order;
  a.row_stats = row_stats;
  a.rewards = rewards;
  a.terminal_reward = terminal_reward;
  a.returns = returns;
  a.zero_padding = zero_padding;
  a.values = values;
  a.lengths = lengths;
  a.cu = cu;
  a.N = N;
  a.stopped = stopped;
  a.T = T;
  a.B = (int32_t)B;
  a.r_fail = r_fail;
  a.gamma = gamma;
  const double c = (double)gamma * (double)lambda;
  a.c = (float)c;
  double power = 1.0;
  for (int j = 0; j <= kPerLane; ++j, power *= c) a.cj[j] = (float)power;
  static_assert(kPerLane == 4 && kWave == 64, "the squares below");
  power = (c * c) * (c * c);
  for (int k = 0; k < 11; ++k, power *= power) (k < 6 ? a.clane[k] : a.cwave[k - 6]) = (float)power;  // c^(4 2^k)
  a.td = td;
  a.adv = adv;
  // Workgroups of 4 waves for short rows: more rows at once, fewer waves without work, no second round of workgroups
  // (B = 1024: T = 1000: 5.3 against 14.1 us, 2048: 8.2 / 11.0, 3000: 11.0 / 13.3, 4096: 13.6 / 14.7; B = 300,
  // T = 2001: 5.9 / 7.4).  A few rows of several of their tiles are better walked by 16 (B = 8, T = 8192).
  // Trajectories stored back to back: by their mean length.
  const int64_t longest = cu ? 2 * (N / B) : T + (T % 4 != 0 ? 3 : 0);
  const bool shortrows = longest <= 8 * kWaveTokens || (longest <= 16 * kWaveTokens && B > kAdvFirstRows);
  const bool can_sort = cu == nullptr && order == nullptr && sorted != nullptr && sync != nullptr;
  a.ordered_from = !shortrows && B <= kAdvSelectRows && longest > (can_sort ? kAdvSortTokens : kAdvSelectTokens) ? kAdvFirstRows : 0x7fffffff;
  // a list that nobody reads is not made (us with / without: B = 20000, T = 1000: 94.0 / 65.8; 100000, 100: 330 / 224)
  const bool sort_here = can_sort && a.ordered_from < B;
  a.sorted = sort_here ? sorted : nullptr;
  a.sync = sort_here ? sync : nullptr;
  // Two spans a wave where every compute unit has more than one row; fewer have the chip to themselves, and more waves walk each
  // faster (8 rows of 16384: 7.7 us, with 8 waves 8.0).  Long rows back to back with rewards and targets, five arrays, are as fast or faster
  // with 16 waves (us, 16 waves / 8, lengths U[T / 16, T]: T = 16384: 300 rows 19.5 / 20.3, 512 23.2 / 24.2, 1024 37.5 / 37.9; whole rows of
  // 8192: 257 10.1 / 10.1, 320 10.9 / 11.2; but mean length 6144: 384 rows 11.4 / 10.4).  No other form is (targets of terminal rewards, U[1024, 16384],
  // 512 rows: padded 21.7 / 19.0, filled 26.0 / 25.7, back to back 20.7 / 19.5).
  const bool five = cu && rewards && returns;
  const int waves = shortrows ? 4 : B <= kAdvOnePerUnit || (five && longest > kAdvFiveArrays) ? 16 : 8;
  const int64_t tile = (shortrows ? 4 : 16) * kWaveTokens;
  const bool fillers = cu == nullptr && zero_padding && longest > tile;
  const dim3 grid((unsigned)((fillers ? 2 * B : B) + (sort_here ? 1 : 0))), block(waves * kWave);
  void (*kernel)(AdvArgs);
  if (cu) kernel = pick_kernel<kPacked>(rewards != nullptr, waves);
  else if (T % 4 == 0) kernel = pick_kernel<kAligned>(rewards != nullptr, waves);
  else kernel = pick_kernel<kShifted>(rewards != nullptr, waves);
  hipLaunchKernelGGL(kernel, grid, block, 0, stream, a);
  return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
}

size_t advantages_workspace_layout(int64_t B, size_t* stats_offset, size_t* sorted_offset) {
  // the two words of `sync` come first, so that they are where they were whatever B a call has
  const size_t stats = (size_t)B * sizeof(AdvRowStats);
  const size_t later = B > kAdvFirstRows ? (size_t)(B - kAdvFirstRows) : 0;
  if (stats_offset) *stats_offset = kAdvSyncBytes;
  if (sorted_offset) *sorted_offset = kAdvSyncBytes + stats;
  return kAdvSyncBytes + stats + ((later * sizeof(int32_t) + 15) & ~(size_t)15);
}

int launch_length_order(const int32_t* lengths, int64_t B, int64_t T, int32_t* order, hipStream_t stream) {
  hipLaunchKernelGGL(length_order_kernel, dim3(1), dim3(16 * kWave), 0, stream, lengths, (int32_t)B, T, order);
  return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
}

}  // namespace espo
