// espo_step: one decode step of ESPO rollout collection (Algorithm 1 body) on gfx950.
//
// One workgroup of 16 wavefronts owns one row.  The row is streamed exactly once through
// 16-byte nontemporal loads; a wave iteration covers a tile of 512 consecutive vocabulary
// indices, 8 per lane, so that each aligned group of 8 lanes holds exactly one 64-index
// block of the random stream.
//   phase 1 (streaming, HBM bound): per lane the running maximum and the softmax sum
//     against a lazily advanced per-lane reference; per block the maximum logit (three
//     DPP steps) and an fp32 upper bound ub_q >= max_v (y_v + G_v) built from the block's
//     largest Gumbel variate M_q, kept in LDS.  Each lane group also keeps the raw data of
//     the block with the largest bound it has seen, so that phase 2 seldom re-reads memory.
//   phase 2 (a handful of indices, behind two barriers): every lane scores the largest logit it
//     has kept, the best score found rules out every block with a lower bound, and each wave
//     looks at what is left of its own blocks (many of them go to a list for the whole workgroup,
//     which is reduced to the indices whose own bound y_v + M_q still reaches the score
//     attained, and those are scored one per thread).  Scores are first formed in fp32 with a
//     proven error margin; if the best two cannot be told apart within that margin, the
//     indices that reach the fp32 winner's lower end are scored again in double, which
//     decides exactly.
//   One lane then runs the scalar chain regret -> normalise/clip -> smoothed state -> stop
//   test (Eq. step_gap, Eq. normalized_gap, Eq. smoothed_score, Eq. stop_rule).
// Pruning only ever discards indices that provably cannot attain the maximum, so the
// token equals the exhaustive double-precision argmax with lowest-index tie-break.
//
// The entropy of the sampling distribution (one more accumulator in phase 1) is a template
// parameter, so that the plain step pays nothing for it.  Filtered draws (top-p / top-k) have a
// kernel of their own, which streams the row the same way but collects its largest logits
// instead of bounding its blocks (see "filtered draws" below).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "../../include/espo.h"
#include "espo_device.h"
#include "espo_host.h"

namespace espo {
namespace {

// A workgroup has W wavefronts (a template parameter of everything below that depends on it): 16 or 8 (plan_step), or 4
// where a caller of the diagnostics entry point forces them.
constexpr int kTile = 512;                        // indices per wave iteration
constexpr int kGroups = kTile / kDrawBlock;       // draw blocks per tile = lane groups per wave
constexpr int kMaxChunks = 64;                    // a row is split over at most this many workgroups (one lane each in the combine)
constexpr int kRing = 4;                          // 16-byte loads kept in flight per lane
constexpr int kCandCap = 1024;                    // candidate indices kept for a row with a long survivor list
constexpr float kRescaleAt = 64.0f;               // advance a lane's softmax reference when topped by 2^64

// What the workgroup of one chunk hands to the combine: the chunk's largest logit, its softmax sums relative to that logit,
// and its exact local winner (score known to within +-e): m, sum, sumw, s, e, x, v.  Each goes into the workspace as a
// 64-bit word of its own with this mark above it, so that a word is either there as a whole or recognised as not there.
constexpr uint32_t kMailMark = 0x4553504Fu;
constexpr int kMailWords = 7, kMailRoom = 8;  // words of a chunk, and what it has room for

struct StepArgs {
  const void* logits;
  int64_t row_stride;
  int32_t V, ntiles, nblocks;
  float inv_tau, k2;   // 1/temperature (fp32 division) and inv_tau * log2(e)
  float ref_lead;      // a lane's softmax reference is advanced once a logit tops it by this much (2^64 in the sum)
  float margin_scale;  // scales the fp32 score margin (1 in production)
  uint32_t key0, key1;
  int32_t step;
  const float* values;
  float mu_g, rsd, clip_c, alpha_s, oma, beta, eps;
  int32_t stop_enabled, eos_id, stop_mode, simulate;
  float stop_threshold;
  float top_p;    // nucleus filter on the draw, active for 0 < top_p < 1
  int32_t top_k;  // top-k filter on the draw, active for top_k > 0
  float* z;
  uint8_t* alive;
  int32_t* stop_step;
  int32_t* tokens;
  float* regret;
  float* logprob;
  float* entropy;
  // a row split over `nch` workgroups: workgroup (row, c) streams `chunk_tiles` tiles, one more for the first `chunk_extra` chunks
  int32_t nch, chunk_tiles, chunk_extra;
  // Where the chunks leave what they found, all left zero for live rows: [B][kMailRoom][nch] words.  A row's words are read by lanes that
  // hold a chunk each, so word j of all chunks is one access (us per launch, eight planes with four words of every row each -> this:
  // bf16 V = 152064, B = 1: 8.85 -> 8.48, 64: 11.02 -> 10.79; f32 V = 150001, B = 64: 14.1 -> 13.6, 320: 42.7 -> 41.7).
  unsigned long long* mail;
};


// ---------------------------------------------------------------- row access
// The raw words of a lane's 8 elements.  Kept as scalars on purpose: the ring of loads in
// flight is carried around the streaming loop, and per-word values keep that rotation in
// plain 32-bit registers.
template <int DT>
struct Raw {
  static constexpr int kWords = DT == ESPO_BF16 ? 4 : 8;
  uint32_t w[kWords];
};

template <int DT>
constexpr int elem_bytes() { return DT == ESPO_BF16 ? 2 : 4; }

// The lane's 8 consecutive elements starting at element e0 (a multiple of 8, e0 < V).  The row
// pitch is a multiple of 4 floats only, so the second half of an fp32 group is read from the
// row's last group of four if it would start at or beyond V (those elements are masked later).
template <int DT>
__device__ __forceinline__ Raw<DT> load_raw(const void* row, uint32_t e0, uint32_t V) {
  Raw<DT> r;
  const char* p = (const char*)row + (size_t)(e0 * (uint32_t)elem_bytes<DT>());
  const u32x4 t = __builtin_nontemporal_load((const u32x4*)p);
  r.w[0] = t.x; r.w[1] = t.y; r.w[2] = t.z; r.w[3] = t.w;
  if constexpr (DT == ESPO_F32) {
    const uint32_t last4 = (V - 1u) & ~3u;
    const uint32_t e1 = e0 + 4u < last4 ? e0 + 4u : last4;
    const u32x4 u = __builtin_nontemporal_load((const u32x4*)((const char*)row + (size_t)(e1 * 4u)));
    r.w[4] = u.x; r.w[5] = u.y; r.w[6] = u.z; r.w[7] = u.w;
  }
  return r;
}

// The same for a tile that lies wholly inside the row: `tile` is the tile's first element
// (wave-uniform, so the address stays a scalar base plus a constant lane offset).
template <int DT>
__device__ __forceinline__ Raw<DT> load_raw_inner(const void* tile, uint32_t lane_bytes) {
  Raw<DT> r;
  const char* p = (const char*)tile + lane_bytes;
  const u32x4 t = __builtin_nontemporal_load((const u32x4*)p);
  r.w[0] = t.x; r.w[1] = t.y; r.w[2] = t.z; r.w[3] = t.w;
  if constexpr (DT == ESPO_F32) {
    const u32x4 u = __builtin_nontemporal_load((const u32x4*)(p + 16));
    r.w[4] = u.x; r.w[5] = u.y; r.w[6] = u.z; r.w[7] = u.w;
  }
  return r;
}

// The same words in LDS.
template <int DT>
__device__ __forceinline__ Raw<DT> pack_load(const uint32_t* raw) {
  Raw<DT> r;
#pragma unroll
  for (int h = 0; h < Raw<DT>::kWords / 4; ++h) {
    const u32x4 t = ((const u32x4*)raw)[h];
    r.w[4 * h] = t.x; r.w[4 * h + 1] = t.y; r.w[4 * h + 2] = t.z; r.w[4 * h + 3] = t.w;
  }
  return r;
}
template <int DT>
__device__ __forceinline__ void pack_store(uint32_t* raw, const Raw<DT>& r) {
#pragma unroll
  for (int h = 0; h < Raw<DT>::kWords / 4; ++h)
    ((u32x4*)raw)[h] = u32x4{r.w[4 * h], r.w[4 * h + 1], r.w[4 * h + 2], r.w[4 * h + 3]};
}

template <int DT>
__device__ __forceinline__ void unpack(const Raw<DT>& r, float x[8]) {
  if constexpr (DT == ESPO_BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __builtin_bit_cast(float, r.w[i] << 16);
      x[2 * i + 1] = __builtin_bit_cast(float, r.w[i] & 0xFFFF0000u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __builtin_bit_cast(float, r.w[i]);
  }
}

__device__ __forceinline__ float max8(const float x[8]) {
  return fmaxf(fmaxf(fmaxf(fmaxf(fmaxf(x[0], x[1]), x[2]), fmaxf(fmaxf(x[3], x[4]), x[5])), x[6]), x[7]);
}

template <int DT>
__device__ __forceinline__ float elem_at(const void* base, int64_t idx) {
  if constexpr (DT == ESPO_BF16)
    return __builtin_bit_cast(float, (uint32_t)((const uint16_t*)base)[idx] << 16);
  else
    return ((const float*)base)[idx];
}

// Logits at or below this are masked like -inf, whatever they are filled with (often the type's lowest value): they hold
// no probability beside any other logit and no search offers them.
constexpr float kMaskedBelow = -1e30f;
constexpr float kNoReference = 1e30f;  // a lane's softmax reference before its first logit that counts

// The negated reference of a lane's softmax sum at logit g.  A masked g over the temperature may overflow; the reference then
// stays where it is before the first logit, so that masked logits add nothing (and no infinity).
__device__ __forceinline__ float lane_reference(float g, float k2) { return fminf(-g * k2, kNoReference); }

// The weight of logit x beside the row maximum m, on the scale of the softmax sum (in which the rounding of every lane's
// reference cancels).  The difference comes first: as 2^(x k2 - m k2) with m k2 rounded, all weights of a row would be off by
// a common factor, up to 4e-5 for logits around 1000 times the temperature, which is more than the 1e-5 trusted below.
__device__ __forceinline__ float weight_below(float x, float m, float k2) { return __builtin_amdgcn_exp2f((x - m) * k2); }

// ---------------------------------------------------------------- scores
// A candidate for the argmax: score s = y + G known to within +-e, its index and logit.
template <typename F>
struct Cand {
  F s;
  float e;
  int32_t v;
  float x;
};

// Running state of the search: the best candidate and `hi2`, the largest upper end s + e
// among all other scored indices.  The winner is certain iff best.s - best.e > hi2.
template <typename F>
struct Search {
  Cand<F> best;
  F hi2;
  __device__ __forceinline__ void init() {
    best = Cand<F>{(F)-__builtin_huge_val(), 0.0f, -1, 0.0f};
    hi2 = (F)-__builtin_huge_val();
  }
  __device__ __forceinline__ void offer(const Cand<F>& c) {
    if (c.v < 0 || c.v == best.v) return;  // nothing, or the element that already leads
    if (c.s > best.s || (c.s == best.s && (uint32_t)c.v < (uint32_t)best.v)) {
      if (best.v >= 0) hi2 = hi2 > best.s + (F)best.e ? hi2 : best.s + (F)best.e;
      best = c;
    } else {
      hi2 = hi2 > c.s + (F)c.e ? hi2 : c.s + (F)c.e;
    }
  }
  __device__ __forceinline__ void merge(const Search& o) {
    hi2 = hi2 > o.hi2 ? hi2 : o.hi2;
    offer(o.best);
  }
  __device__ __forceinline__ F lower() const { return best.v >= 0 ? best.s - (F)best.e : (F)-__builtin_huge_val(); }
};

template <typename F>
__device__ __forceinline__ Search<F> wave_merge(Search<F> s) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Search<F> o;
    o.best.s = __shfl_xor(s.best.s, off);
    o.best.e = __shfl_xor(s.best.e, off);
    o.best.v = __shfl_xor(s.best.v, off);
    o.best.x = __shfl_xor(s.best.x, off);
    o.hi2 = __shfl_xor(s.hi2, off);
    s.merge(o);
  }
  return s;
}

// -ln u(word) in the working precision.  fp32: |ln u| >= ln 2 for u < 1/2, and log1p keeps
// full relative accuracy for u >= 1/2 (1 - u is exact in fp32).
template <typename F>
__device__ __forceinline__ F neg_log_uniform(uint32_t word);
template <>
__device__ __forceinline__ double neg_log_uniform<double>(uint32_t word) { return -log(uniform_f64(word)); }
template <>
__device__ __forceinline__ float neg_log_uniform<float>(uint32_t word) {
  return -__builtin_amdgcn_logf((float)(2u * (word >> 9) + 1u) * (1.0f / 16777216.0f)) * kLn2;
}
// fp32 ln and exp from the hardware log2 / exp2.  Measured over all inputs that occur here
// (every positive float in [2^-26, 64) for ln, every u(w); [-40, 8] for exp): relative error
// below 1.7e-7 for ln, also next to 1, and below 2e-6 for exp; a GPU test re-measures this.
__device__ __forceinline__ float flog(float x) { return __builtin_amdgcn_logf(x) * kLn2; }
__device__ __forceinline__ double flog(double x) { return log(x); }
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }
__device__ __forceinline__ double fexp(double x) { return exp(x); }

// Error margin of an fp32 score y + G.  With ln accurate to 1.7e-7 and exp to 2e-6 (relative):
// -ln u carries 1.7e-7, M_q = ln n - ln(-ln u) at most 5e-6 for |M_q| <= 25, exp(-M_q) at most
// 7e-6 relative (4e-7 where it is formed as (-ln u)/n), G = -ln(exp(-M_q) - ln u) at most
// 1.1e-5, and the product and sum forming y + G add 2^-23 (|y| + |G|).  The margin below is
// more than three times that.
__device__ __forceinline__ float score_margin(const StepArgs& a, float y) {
  return a.margin_scale * (4e-5f + 2.5e-7f * fabsf(y));
}

// The block-level part of the draw for block q: its largest variate M_q, exp(-M_q), and the
// index that receives M_q.
template <typename F>
struct BlockDraw {
  F M, emM;
  int32_t vpos;
};

template <typename F>
__device__ __forceinline__ BlockDraw<F> block_draw(const StepArgs& a, int row, int q) {
  const int32_t first = q * kDrawBlock;
  const int32_t n = a.V - first < kDrawBlock ? a.V - first : kDrawBlock;
  const Philox4 pb = philox4x32_10((uint32_t)(q >> 2), (uint32_t)a.step, (uint32_t)row, kTagBlock, a.key0, a.key1);
  const uint32_t wb = (q & 3) == 0 ? pb.w[0] : (q & 3) == 1 ? pb.w[1] : (q & 3) == 2 ? pb.w[2] : pb.w[3];
  BlockDraw<F> d;
  d.M = flog((F)n) - flog(neg_log_uniform<F>(wb));
  d.emM = fexp(-d.M);
  d.vpos = first + (int32_t)((wb >> 3) & 63u);
  if (n < kDrawBlock) {  // ragged last block: own position draw
    const Philox4 pr = philox4x32_10((uint32_t)q, (uint32_t)a.step, (uint32_t)row, kTagRagged, a.key0, a.key1);
    d.vpos = first + (int32_t)(((uint64_t)pr.w[0] * (uint64_t)n) >> 32);
  }
  return d;
}

// Scores index v (logit x) of a block with draw d and offers it to the search, unless its
// upper bound y + M_q (+ margins) cannot reach `bound`, a score already known to be attained,
// or its logit is not above `floor` (-inf: only masked entries are left out).
template <typename F>
__device__ __forceinline__ void score_index(const StepArgs& a, int row, int32_t v, float x, const BlockDraw<F>& d,
                                            F bound, float floor, Search<F>& st) {
  const F y = (F)x * (F)a.inv_tau;
  const float e = sizeof(F) == 4 ? score_margin(a, (float)y) : 0.0f;
  if (x > floor && (y + d.M) + (F)(2.0f * e) >= bound) {   // masked (-inf) and filtered entries never win
    F G = d.M;
    if (v != d.vpos) {
      const Philox4 p = philox4x32_10((uint32_t)(v >> 2), (uint32_t)a.step, (uint32_t)row, kTagElem, a.key0, a.key1);
      const uint32_t w = (v & 3) == 0 ? p.w[0] : (v & 3) == 1 ? p.w[1] : (v & 3) == 2 ? p.w[2] : p.w[3];
      G = -flog(d.emM + neg_log_uniform<F>(w));
    }
    st.offer(Cand<F>{y + G, e, v, x});
  }
}

// Scores the 64 indices of block q, one per lane.  `data` points at the block's 64 elements.
template <int DT, typename F>
__device__ __forceinline__ void visit_block(const StepArgs& a, int row, int q, const void* data, F bound, float floor,
                                            Search<F>& st) {
  const int lane = threadIdx.x & (kWave - 1);
  const BlockDraw<F> d = block_draw<F>(a, row, q);
  const int32_t v = q * kDrawBlock + lane;
  if (v < a.V) score_index<F>(a, row, v, elem_at<DT>(data, lane), d, bound, floor, st);
}

// The scalar chain regret -> normalised, clipped regret -> smoothed state -> stop test.
// Every operation is a single correctly rounded fp32 operation in the order written
// (contraction off), so a host re-computation reproduces z and the stop decision bit for bit.
struct ChainOut {
  float g, z;
  bool stop;
};

constexpr uint32_t kTagStop = 0x53544F50u;  // counter word 3 of the coin of the random stop mode

__device__ __forceinline__ ChainOut scalar_chain(const StepArgs& a, int row, float m, float x_a, float z_prev, float value) {
#pragma clang fp contract(off)
  const float d = m - x_a;
  const float g = d * a.inv_tau;                                    // Eq. step_gap
  const float n = (g - a.mu_g) * a.rsd;
  const float gt = fminf(fmaxf(n, -a.clip_c), a.clip_c);            // Eq. normalized_gap
  const float t = a.oma * gt;
  const float zn = __builtin_fmaf(a.alpha_s, z_prev, t);            // Eq. smoothed_score
  bool stop;
  if (a.stop_mode == ESPO_STOP_VALUE_ONLY) {
    stop = value < a.stop_threshold;
  } else if (a.stop_mode == ESPO_STOP_REGRET_ONLY) {
    stop = zn > a.stop_threshold;
  } else if (a.stop_mode == ESPO_STOP_RANDOM) {
    const Philox4 p = philox4x32_10(0u, (uint32_t)a.step, (uint32_t)row, kTagStop, a.key0, a.key1);
    stop = (float)(2u * (p.w[0] >> 9) + 1u) * (1.0f / 16777216.0f) < a.stop_threshold;  // u(w) is exact in fp32
  } else {
    const float thr = a.beta * fmaxf(value, a.eps);
    stop = zn > thr;                                                // Eq. stop_rule (strict)
  }
  return ChainOut{g, zn, a.stop_enabled && stop};
}

// What one lane does at the end of a row: the scalar chain on the sampled logit, then the row's outputs.
template <int DT, bool Entropy, bool Sum>
__device__ __forceinline__ void finish_row(const StepArgs& a, int row, const void* rowp, int32_t tok, float x_a, float m,
                                           float S, float Sw, float z_prev, float value) {
  if (tok < 0) { tok = 0; x_a = elem_at<DT>(rowp, 0); }  // row of -inf only: unspecified, stay in range
  const ChainOut c = scalar_chain(a, row, m, x_a, z_prev, value);
  a.tokens[row] = tok;
  a.regret[row] = c.g;
  a.z[row] = c.z;
  if (Sum && a.logprob) a.logprob[row] = -c.g - flog(S);
  if constexpr (Entropy)  // H = ln S - E_pi[y - y_max] >= 0; rounding can leave S a few ulp below 1
    a.entropy[row] = fmaxf(flog(S) - kLn2 * Sw / S, 0.0f);
  if (a.eos_id >= 0 && tok == a.eos_id) {
    a.alive[row] = 0;  // natural end
  } else if (c.stop) {
    if (a.simulate) {  // bookkeeping only: the first stop step is recorded, decoding goes on
      if (a.stop_step[row] < 0) a.stop_step[row] = a.step;
    } else {
      a.alive[row] = 0;  // absorbing failure (Eq. failure_reward): the trajectory ends here
      a.stop_step[row] = a.step;
    }
  }
}

// ---------------------------------------------------------------- shared memory
// Blocks are named by their index q in the row everywhere (survivor lists, own); the
// per-block tables only cover the workgroup's chunk and are reached through the accessors, which
// subtract q0, the chunk's first block (a multiple of 8).
struct StepShared {
  float* mu;        // [nslots][2] per block slot (tile * 8 + group): upper bound of M_q (phase 1 only; phase 2
                    //   keeps its survivor list there), and the bound of the block's best score
  uint32_t* wq;     // [nslots] the block's word of the random stream
  int q0;           // first block of the chunk
  __device__ __forceinline__ float& mub(int q) const { return mu[2 * (q - q0)]; }
  __device__ __forceinline__ float& ub(int q) const { return mu[2 * (q - q0) + 1]; }
  __device__ __forceinline__ uint32_t& word(int q) const { return wq[q - q0]; }
  __device__ __forceinline__ float& blockmax(int q) const { return bmx[q - q0]; }
  __device__ __forceinline__ int& surv(int k) const { return ((int*)mu)[2 * k]; }
  void* top_raw;    // [8 W][64 elements] data of each lane group's best block
  float* m;         // [W] wave maxima
  float* sum;       // [W] wave softmax sums, relative to the wave's own maximum
  float* sumw;      // [W] wave sums of 2^t t, t = (y_v - y_max) log2 e with the wave's y_max (entropy output only)
  double* res_s;    // [W] per-wave search results
  double* res_hi2;
  float* res_e;
  int* res_v;
  float* res_x;
  float* lo;        // [W] score each wave knows to be attained
  int* own;         // [W][8] blocks that a wave has to read again
  float* fres;      // [W][8] per-wave results of the fp32 search: s, e, x, hi2, v
  int32_t* cand_v;  // [kCandCap] long survivor lists: indices that can still win ...
  float* cand_x;    // [kCandCap] ... and their logits
  int* ncand;       // [1]
  int* nsurv;       // [1]
  int* bkey;        // [1] best attained score published during long survivor lists (order-preserving key)
  float floor;      // only logits above this take part in the search (what counts as masked, or more if the draw is filtered)
  float* bmx;       // [nslots] largest logit of every block (filtered draws only, else null)
};

template <int DT, bool Filter, int W>
__device__ __forceinline__ StepShared carve(unsigned char* base, int nslots, int q0) {
  constexpr int kStepWaves = W, kSlots = W * kGroups;
  StepShared s;
  s.floor = kMaskedBelow;
  s.q0 = q0;
  size_t off = 0;
  auto take = [&](size_t bytes) { void* p = base + off; off += (bytes + 15) & ~(size_t)15; return p; };
  s.res_s = (double*)take(kStepWaves * 8);
  s.res_hi2 = (double*)take(kStepWaves * 8);
  s.top_raw = take((size_t)kSlots * kDrawBlock * elem_bytes<DT>());
  s.m = (float*)take(kStepWaves * 4);
  s.sum = (float*)take(kStepWaves * 4);
  s.sumw = (float*)take(kStepWaves * 4);
  s.res_e = (float*)take(kStepWaves * 4);
  s.res_v = (int*)take(kStepWaves * 4);
  s.res_x = (float*)take(kStepWaves * 4);
  s.lo = (float*)take(kStepWaves * 4);
  s.own = (int*)take(kSlots * 4);
  s.fres = (float*)take(8 * kStepWaves * 4);
  s.cand_v = (int32_t*)take(kCandCap * 4);
  s.cand_x = (float*)take(kCandCap * 4);
  s.nsurv = (int*)take(16);
  s.bkey = s.nsurv + 1;
  s.ncand = s.nsurv + 2;
  s.mu = (float*)take((size_t)nslots * 8);
  s.wq = (uint32_t*)take((size_t)nslots * 4);
  s.bmx = Filter ? (float*)take((size_t)nslots * 4) : nullptr;
  return s;
}

// Dynamic LDS of a workgroup of `waves` wavefronts whose chunk has `ntiles` tiles (what carve() lays out).
[[maybe_unused]] size_t step_lds_bytes(int dt, int ntiles, bool filter, int waves) {
  const size_t esz = dt == ESPO_BF16 ? 2 : 4;
  const size_t nslots = (size_t)ntiles * kGroups, slots = (size_t)waves * kGroups;
  return 2 * (size_t)waves * 8 + slots * kDrawBlock * esz + slots * 4 + 15 * (size_t)waves * 4 + 16 + 2 * kCandCap * 4 +
         ((nslots * 8 + 15) & ~(size_t)15) + (filter ? 2 : 1) * ((nslots * 4 + 15) & ~(size_t)15);
}

// The streaming loop stores a block's bound as the plain fma(y_max, 1/tau, bound of M_q); what
// that fma may have rounded away (2^-24 relative) is added back where bounds are compared.
__device__ __forceinline__ float ub_rounded_up(float u) { return fmaf(fabsf(u), 2e-7f, u); }

// Whether block b can hold a logit that takes part in the search: always, unless the draw is
// filtered; then only if its largest logit is above the floor.
__device__ __forceinline__ bool holds_eligible(const StepShared& sh, int q) { return sh.bmx == nullptr || sh.blockmax(q) > sh.floor; }

// ---------------------------------------------------------------- phase 2
// Lanes below this one whose bit is set in `mask`.
__device__ __forceinline__ int rank_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ int float_key(float f) {  // order-preserving map to signed int
  const int b = __builtin_bit_cast(int, f);
  return b >= 0 ? b : b ^ 0x7fffffff;
}

template <typename F>
__device__ __forceinline__ float round_down_f32(F v) {
  float f = (float)v;
  if ((F)f > v) f = __builtin_bit_cast(float, __builtin_bit_cast(int32_t, f) + (f > 0.0f ? -1 : 1));
  if (f == 0.0f && v < (F)0) f = -1e-37f;
  return f;
}

// Merges the lanes' and then the waves' search states in a fixed order; returns the same
// result in every thread.  All threads of the workgroup must call it.
template <typename F, int W>
__device__ __forceinline__ Search<F> combine_search(const StepShared& sh, Search<F> st) {
  constexpr int kStepWaves = W;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  st = wave_merge(st);
  if (lane == 0) {
    sh.res_s[wave] = (double)st.best.s;
    sh.res_hi2[wave] = (double)st.hi2;
    sh.res_e[wave] = st.best.e;
    sh.res_v[wave] = st.best.v;
    sh.res_x[wave] = st.best.x;
  }
  __syncthreads();
  Search<F> all;
  all.init();
#pragma unroll 1
  for (int w = 0; w < kStepWaves; ++w) {  // fixed order: deterministic
    Search<F> o;
    o.best = Cand<F>{(F)sh.res_s[w], sh.res_e[w], sh.res_v[w], sh.res_x[w]};
    o.hi2 = (F)sh.res_hi2[w];
    all.merge(o);
  }
  return all;
}

// Finds the argmax over the row in double.  `bound` is a score that is known to be attained or exceeded: every block whose own bound
// reaches it is scored, one block per wave visit.  Returns the winner, the same in every thread; all threads of
// the workgroup must call it.
template <int DT, int W>
__device__ __forceinline__ Search<double> find_argmax(const StepArgs& a, const StepShared& sh, const void* rowp, int row,
                                                      int nslots, double bound) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) *sh.nsurv = 0;
  __syncthreads();
  const float bound_f = round_down_f32(bound);
  for (int b = sh.q0 + tid; b < sh.q0 + nslots; b += W * kWave) {
    const float u = sh.ub(b);
    if (u > kMaskedBelow && ub_rounded_up(u) >= bound_f && holds_eligible(sh, b)) sh.surv(atomicAdd(sh.nsurv, 1)) = b;
  }
  __syncthreads();
  const int nsurv = *sh.nsurv;
  Search<double> st;
  st.init();
#pragma unroll 1
  for (int k = wave; k < nsurv; k += W) {
    const int q = sh.surv(k);
    visit_block<DT, double>(a, row, q, (const char*)rowp + (size_t)q * kDrawBlock * elem_bytes<DT>(), bound, sh.floor, st);
    bound = fmax(bound, (double)wave_max(round_down_f32(st.lower())));  // best score this wave has seen, rounded down
  }
  return combine_search<double, W>(sh, st);
}

// ---------------------------------------------------------------- phase 2 in fp32
// State of the fp32 search, per lane while blocks are visited and wave-uniform once reduced:
// the best index scored (score s known to within +-e, logit x) and hi2, the largest upper
// end s + e among all other scored indices.  The winner is certain iff s - e > hi2.
struct Best {
  float s, e, x, hi2;
  int32_t v;
};

__device__ __forceinline__ Best no_best() { return Best{kNegInf, 0.0f, 0.0f, kNegInf, -1}; }

// The block-level part of an fp32 score, from the block's random word: its largest variate M_q = ln n - ln(-ln u),
// exp(-M_q) = (-ln u) / n, and the index that receives M_q.
struct FastDraw {
  float M, emM;
  int32_t vpos;
};

__device__ __forceinline__ FastDraw fast_draw(const StepArgs& a, int row, int32_t q, uint32_t wb) {
  const int32_t first = q * kDrawBlock;
  const int32_t n = a.V - first < kDrawBlock ? a.V - first : kDrawBlock;
  const float nlb = neg_log_uniform<float>(wb);
  FastDraw d;
  d.M = flog((float)n) - flog(nlb);
  d.emM = nlb * __builtin_amdgcn_rcpf((float)n);
  d.vpos = first + (int32_t)((wb >> 3) & 63u);
  if (n < kDrawBlock) {  // ragged last block: own position draw
    const Philox4 pr = philox4x32_10((uint32_t)q, (uint32_t)a.step, (uint32_t)row, kTagRagged, a.key0, a.key1);
    d.vpos = first + (int32_t)(((uint64_t)pr.w[0] * (uint64_t)n) >> 32);
  }
  return d;
}

// Offers index v (logit x) with variate G to the lane's state.  An index is offered at most once in a search.
// `v_named` is what the state calls the index (the index itself, or the index with a flag on top).
__device__ __forceinline__ void offer_score(const StepArgs& a, int32_t v_named, float x, float G, bool valid, Best& st) {
  const float y = x * a.inv_tau;
  const float sc = y + G;
  const float e = score_margin(a, y);
  if (valid) {
    if (sc > st.s) {
      st.hi2 = fmaxf(st.hi2, st.s + st.e);
      st.s = sc; st.e = e; st.x = x; st.v = v_named;
    } else {
      st.hi2 = fmaxf(st.hi2, sc + e);
    }
  }
}

// The index's own word of the random stream.  (The four words are formed before one is picked: left to itself the compiler
// puts the last rounds of each behind a branch.)
__device__ __forceinline__ uint32_t element_word(const StepArgs& a, int row, int32_t v) {
  Philox4 p = philox4x32_10((uint32_t)(v >> 2), (uint32_t)a.step, (uint32_t)row, kTagElem, a.key0, a.key1);
  asm("" : "+v"(p.w[0]), "+v"(p.w[1]), "+v"(p.w[2]), "+v"(p.w[3]));
  const uint32_t low = (v & 1) ? p.w[1] : p.w[0], high = (v & 1) ? p.w[3] : p.w[2];
  return (v & 2) ? high : low;
}

// Scores index v (logit x) in fp32 and offers it to the lane's state, with `d` the draw of its block.
__device__ __forceinline__ void score_with(const StepArgs& a, int row, int32_t v, int32_t v_named, float x, const FastDraw& d,
                                           bool valid, Best& st) {
  float G = -flog(d.emM + neg_log_uniform<float>(element_word(a, row, v)));
  G = v == d.vpos ? d.M : G;
  offer_score(a, v_named, x, G, valid, st);
}
__device__ __forceinline__ void score_drawn(const StepArgs& a, int row, int32_t v, int32_t v_named, float x, uint32_t wb,
                                            bool valid, Best& st) {
  score_with(a, row, v, v_named, x, fast_draw(a, row, v >> 6, wb), valid, st);
}

__device__ __forceinline__ void score_element(const StepArgs& a, const StepShared& sh, int row, int32_t v, float x,
                                              bool valid, Best& st) {
  score_drawn(a, row, v, v, x, sh.word(v >> 6), valid && x > sh.floor, st);  // masked (-inf) and filtered entries never win
}

// Scores the 64 indices of block q, one per lane.
template <int DT>
__device__ __forceinline__ void fast_visit(const StepArgs& a, const StepShared& sh, const void* rowp, int row, int q,
                                           Best& st) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t first = q * kDrawBlock;
  const int32_t n = a.V - first < kDrawBlock ? a.V - first : kDrawBlock;
  const float x = elem_at<DT>((const char*)rowp + (size_t)first * elem_bytes<DT>(), lane < n ? lane : n - 1);  // stay inside the row
  score_element(a, sh, row, first + lane, x, lane < n, st);
}

// For a row with a long survivor list: instead of scoring every index of every surviving
// block, the blocks' logits are only compared with the bound (index v can win only if
// y_v + M_q reaches it); the few indices that pass are collected and then scored by all threads
// at once.  The blocks are read again from the row, laid out as in phase 1: a lane group of 8
// lanes per block, 16 bytes per lane, so one load of a wave covers 8 blocks; with four loads in
// flight the workgroup covers 512 blocks per trip to memory (a flat row at temperature 1 has a
// hundred survivors and more; one block per load took a trip per 64 of them).
template <int DT, int W>
__device__ __forceinline__ void collect_candidates(const StepArgs& a, const StepShared& sh, const void* rowp, int nsurv,
                                                   float bound) {
  constexpr int kStepWaves = W, kLoads = 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane >> 3;
  const uint32_t sub = (uint32_t)(lane & 7) * 8u;  // the lane's 8 elements within its block
  const uint32_t last_group = (uint32_t)(a.V - 1) & ~7u;
#pragma unroll 1
  for (int base = wave * kGroups; base < nsurv; base += kLoads * kStepWaves * kGroups) {
    int qs[kLoads];
    Raw<DT> raw[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int k = base + j * kStepWaves * kGroups + grp;
      qs[j] = k < nsurv ? sh.surv(k) : -1;
      // a group without a block reads block 0 and drops it; a ragged last block is masked below
      const uint32_t e0 = (uint32_t)(qs[j] < 0 ? 0 : qs[j]) * kDrawBlock + sub;
      raw[j] = load_raw<DT>(rowp, e0 < last_group ? e0 : last_group, (uint32_t)a.V);
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      if (qs[j] < 0) continue;
      float x[8];
      unpack<DT>(raw[j], x);
      const int32_t first = qs[j] * kDrawBlock;
      const int32_t n = a.V - first < kDrawBlock ? a.V - first : kDrawBlock;
      const float M = flog((float)n) - flog(neg_log_uniform<float>(sh.word(qs[j])));
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int32_t v = first + (int32_t)sub + u;
        const float y = x[u] * a.inv_tau;
        if (v < a.V && x[u] > sh.floor && (y + M) + 2.0f * score_margin(a, y) >= bound) {
          const int i = atomicAdd(sh.ncand, 1);
          if (i < kCandCap) {
            sh.cand_v[i] = v;
            sh.cand_x[i] = x[u];
          }
        }
      }
    }
  }
}

// The exact decision for a row whose best fp32 scores overlap: `lower` is a score known to be
// attained (the fp32 winner's lower end), so only indices with y_v + M_q at or above it can
// be the maximum.  They are collected as above, usually two or three, and scored in double
// by one thread each.  Returns false if they do not fit the candidate buffer (then the
// caller searches block by block); all threads of the workgroup must call it.
template <int DT, int W>
__device__ __forceinline__ bool exact_among_candidates(const StepArgs& a, const StepShared& sh, const void* rowp, int row,
                                                       int nslots, float lower, Search<double>& out) {
  constexpr int kStepThreads = W * kWave;
  const int tid = threadIdx.x;
  if (tid == 0) {
    *sh.nsurv = 0;
    *sh.ncand = 0;
  }
  __syncthreads();
  for (int b = sh.q0 + tid; b < sh.q0 + nslots; b += kStepThreads) {
    const float u = sh.ub(b);
    if (u > kMaskedBelow && ub_rounded_up(u) >= lower && holds_eligible(sh, b)) sh.surv(atomicAdd(sh.nsurv, 1)) = b;
  }
  __syncthreads();
  collect_candidates<DT, W>(a, sh, rowp, *sh.nsurv, lower);
  __syncthreads();
  const int ncand = *sh.ncand;
  if (ncand > kCandCap) return false;
  Search<double> st;
  st.init();
  for (int i = tid; i < ncand; i += kStepThreads) {
    const int32_t v = sh.cand_v[i];
    const BlockDraw<double> d = block_draw<double>(a, row, v >> 6);
    score_index<double>(a, row, v, sh.cand_x[i], d, -__builtin_huge_val(), sh.floor, st);
  }
  out = combine_search<double, W>(sh, st);
  return true;
}

// The lane that holds the highest score, the lowest index among equals, or -1; wave-uniform.  `smax` is that score.
__device__ __forceinline__ int best_lane(const Best& st, float smax) {
  const bool cand = st.v >= 0 && st.s == smax;
  uint64_t mask = __builtin_amdgcn_ballot_w64(cand);
  if (mask == 0) return -1;
  if ((mask & (mask - 1)) != 0) {  // (rare)
    const uint32_t vmin = wave_min_u32(cand ? (uint32_t)st.v : 0xffffffffu);
    mask = __builtin_amdgcn_ballot_w64(cand && (uint32_t)st.v == vmin);
  }
  return (int)__builtin_ctzll(mask);
}

// Combines the states of 64 lanes, or of the first 16, into one.
template <bool Row = false>
__device__ __forceinline__ Best wave_best(const Best& st) {
  const float smax = Row ? row_max(st.s) : wave_max(st.s);
  const int src = best_lane(st, smax);
  if (src < 0) return no_best();
  const float other = (int)(threadIdx.x & (kWave - 1)) == src ? st.hi2 : fmaxf(st.hi2, st.s + st.e);
  Best r;
  r.s = smax;
  r.v = __builtin_amdgcn_readlane(st.v, src);
  r.e = uniform_f32(st.e, src);
  r.x = uniform_f32(st.x, src);
  r.hi2 = Row ? row_max(other) : wave_max(other);
  return r;
}

__device__ __forceinline__ float key_float(int k) { return __builtin_bit_cast(float, k >= 0 ? k : k ^ 0x7fffffff); }

// A wave's state, to LDS: the lane that holds the best writes it itself.
template <int W>
__device__ __forceinline__ void publish_wave(float* fres, const Best& st) {
  static_assert(W <= 16, "row_max: a lane per wave");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int src = best_lane(st, wave_max(st.s));
  const float hi2 = wave_max(lane == src ? st.hi2 : fmaxf(st.hi2, st.s + st.e));
  float* const to = fres + wave * 8;
  if (lane == (src < 0 ? 0 : src)) {  // (without a best, lane 0 holds an empty state like every other)
    *(f32x4*)to = f32x4{st.s, st.e, st.x, hi2};
    to[4] = __builtin_bit_cast(float, st.v);
  }
}

// Every wave's state, merged; the same in every wave.
template <int W>
__device__ __forceinline__ Best merge_waves(const float* fres) {
  const int lane = threadIdx.x & (kWave - 1);
  Best t = no_best();
  if (lane < W) {
    const f32x4 from = *(const f32x4*)(fres + lane * 8);
    t.s = from[0];
    t.e = from[1];
    t.x = from[2];
    t.hi2 = from[3];
    t.v = __builtin_bit_cast(int32_t, fres[lane * 8 + 4]);
  }
  return wave_best<true>(t);
}

// The fp32 search over the row, behind two barriers.  Every lane group still has in LDS the 64 logits of `q_top`, the block
// with the largest bound among those it has streamed, 8 of them at `my_raw` of each lane.  Before the first barrier each
// lane scores the largest of its 8, and the lane that holds the index that received the block's M_q scores that one,
// which needs no random word of its own: 8 blocks per wave, one Philox call.  The best lower end s - e found that way
// is a score known to be attained.  After the barrier a wave looks through its own blocks only: what else of them reaches
// that score is scored in place, at most kGroups blocks read again from the row; with more than that to read the
// wave puts them on a list for the whole workgroup, which reduces it to the indices that can still win.  Of 152064 logits
// at temperature 0.6 a row has 0.7 (16 waves) to 1.2 (8 waves) such blocks on average, none in half of the rows; at
// temperature 1.0 2.7 and 7.8.  (One block per wave scored whole, two with 8 waves, then the survivors of the row
// dealt to the waves through a list and a barrier of its own left 4 and, at temperature 1.0, 40 to 46.)
// Bound by what a wave issues, about 4.4 cycles an instruction, since the last waves to end their streaming have the
// compute unit to themselves: so a maximum is one instruction a step (espo_device.h), blocks' bounds are read ahead of the
// barrier, and the lane that holds a wave's best hands it on itself.  us per launch from a graph, before -> now, V = 152064 bf16,
// all rows live: B = 1: 11.5 -> 10.2, 64: 14.0 -> 12.8 (both with the cheaper combine of step_row), 512: 34.5 -> 33.2,
// 1024: 59.4 -> 57.5; at temperature 1.0 / 1.3, B = 512: 39.7 -> 36.5 / 65.3 -> 37.6; all logits equal, B = 512: 32.9 -> 32.3.
// Short rows of flat logits pay for it, 0.3 to 0.6 us: their best block is looked at a second time, behind the barrier (means over 60 steps, all logits equal,
// B = 1, V = 8000: 6.3 -> 6.7; 255, 32000: 8.2 -> 8.7; normal logits at temperature 3, 255, 32000: 8.4 -> 9.2).  (Leaving out there, or in the branch for several
// indices a lane, what cannot beat the index that received M_q: 3 to 5 % slower on all other rows.)
// Returns the wave-uniform result, the same in every wave; all threads of the workgroup must call it.
template <int DT, bool Filter, int W>
__device__ __forceinline__ Best fast_argmax(const StepArgs& a, const StepShared& sh, const void* rowp, int row, int my_tiles,
                                            int q_top, float top_ub, const char* my_raw) {
  constexpr int kStepThreads = W * kWave;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = lane >> 3;
  const uint32_t sub = (uint32_t)(lane & 7) * 8u;  // the lane's 8 elements within a block
  Best st = no_best();
  Raw<DT> raw = pack_load<DT>((const uint32_t*)my_raw);  // this lane's 8 logits of the group's best block (those at or beyond V are -inf there)
  FastDraw d = {};
  uint32_t scored = 0;  // which of the lane's 8 logits need no more looking at
  if (q_top >= 0) {     // (the same in the lanes of a group)
    const int32_t v0 = q_top * kDrawBlock + (int32_t)sub;
    float x[8];
    unpack<DT>(raw, x);
    const float top = max8(x);
    int at = 7;
#pragma unroll
    for (int j = 6; j >= 0; --j) at = x[j] == top ? j : at;
    d = fast_draw(a, row, q_top, sh.word(q_top));
    const int drawn = d.vpos - v0;
    const bool mine = (uint32_t)drawn < 8u;
    const float xd = elem_at<DT>(my_raw, mine ? drawn : 0);
    // above the floor of a filtered draw few waves hold anything, and the random words are most of the work
    if (!Filter || __builtin_amdgcn_ballot_w64(top > sh.floor) != 0) score_with(a, row, v0 + at, v0 + at, top, d, top > sh.floor, st);
    offer_score(a, d.vpos, xd, d.M, mine && drawn != at && xd > sh.floor, st);  // (vpos is below V)
    scored = 1u << at | (mine ? 1u << drawn : 0u);
  }
  const float lo = wave_max(st.s - st.e);
  if (lane == 0) sh.lo[wave] = lo;
  if (tid == 0) {
    *sh.nsurv = 0;
    *sh.ncand = 0;
  }
  // this wave's blocks, except the groups' best: block k & 7 of its tile k >> 3
  const int slots = my_tiles * kGroups;
  const int q_first = sh.q0 + wave * kGroups;
  const int skip = __shfl(q_top, (lane & 7) * 8);
  auto block_at = [&](int k) { return q_first + (k >> 3) * (W * kGroups) + (k & 7); };
  auto bound_of = [&](int k) {  // of block k, rounded up; -inf for one that cannot win or is none of these
    if (k >= slots) return kNegInf;
    const int b = block_at(k);
    const float u = sh.ub(b);
    return u > kMaskedBelow && b != skip && holds_eligible(sh, b) ? ub_rounded_up(u) : kNegInf;
  };
  // Read before the barrier: all blocks of a wave for V up to 196608 (16 waves) or 163840.  None in the general search of a filtered draw,
  // which few rows need and which shares its registers with the draw from the lists.
  constexpr int kAhead = Filter ? 0 : W == 16 ? 3 : 5;
  float ahead[Filter ? 1 : kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    ahead[i] = kNegInf;
    if (i * kWave < slots) ahead[i] = bound_of(i * kWave + lane);  // (wave-uniform)
  }
  __syncthreads();
  // (a row without a candidate so far has no bound: every block with a logit that counts is then looked at)
  const float bound = fmaxf(row_max(lane < W ? sh.lo[lane] : kNegInf), -3.0e38f);
  int nown = 0;  // blocks whose bound reaches the best score found so far
  auto look = [&](auto&& use) {
    auto one = [&](int k0, float u) {
      const bool in = u >= bound;
      const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
      if (mask != 0) use(k0 + lane, in, mask);
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) one(i * kWave, ahead[i]);
#pragma unroll 1
    for (int k0 = kAhead * kWave; k0 < slots; k0 += kWave) one(k0, bound_of(k0 + lane));  // (wave-uniform)
  };
  look([&](int k, bool in, uint64_t mask) {
    const int at = nown + rank_below(mask);
    if (in && at < kGroups) sh.own[wave * kGroups + at] = block_at(k);
    nown += (int)__builtin_popcountll(mask);
  });
  if (nown > kGroups) {  // too many to read again one after the other: to the workgroup's list
    look([&](int k, bool in, uint64_t mask) {
      int base = 0;
      if (lane == 0) base = atomicAdd(sh.nsurv, (int)__builtin_popcountll(mask));
      base = __builtin_amdgcn_readfirstlane(base);
      if (in) sh.surv(base + rank_below(mask)) = block_at(k);
    });
    nown = 0;
  }
  // the groups' best blocks once more, then the wave's list, a block per lane group
  int q = q_top >= 0 && ub_rounded_up(top_ub) >= bound ? q_top : -1;
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 1) {
      if (nown == 0) break;
      asm volatile("" ::: "memory");  // the list was written by this wave's other lanes (LDS keeps a wave's order)
      q = grp < nown ? sh.own[wave * kGroups + grp] : -1;
      const uint32_t last_group = (uint32_t)(a.V - 1) & ~7u;
      const uint32_t e0 = (uint32_t)(q < 0 ? 0 : q) * kDrawBlock + sub;  // a group without a block reads block 0 and drops it
      raw = load_raw<DT>(rowp, e0 < last_group ? e0 : last_group, (uint32_t)a.V);
      if (q >= 0) d = fast_draw(a, row, q, sh.word(q));
      scored = 0;
    }
    if (__builtin_amdgcn_ballot_w64(q >= 0) == 0) continue;
    const int32_t v0 = q * kDrawBlock + (int32_t)sub;
    float x[8];
    unpack<DT>(raw, x);
    uint32_t todo = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float y = x[j] * a.inv_tau;
      todo |= x[j] > sh.floor && (y + d.M) + 2.0f * score_margin(a, y) >= bound ? 1u << j : 0u;
    }
    todo &= ~scored & (q < 0 ? 0u : a.V - v0 >= 8 ? 0xffu : a.V > v0 ? (1u << (a.V - v0)) - 1u : 0u);
    while (__builtin_amdgcn_ballot_w64(todo != 0) != 0) {
      const uint64_t many = __builtin_amdgcn_ballot_w64((todo & (todo - 1)) != 0);
      int32_t v;
      float xv;
      bool valid;
      FastDraw dv = d;
      if (many == 0) {  // one for each lane at most (the usual case): all at once
        const int j = __builtin_ctz(todo | 0x100u) & 7;
        xv = x[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) xv = i == j ? x[i] : xv;
        v = v0 + j;
        valid = todo != 0;
        todo = 0;
      } else {  // several (equal logits, flat rows): one group's block, an index per lane
        const int from = (int)__builtin_ctzll(many) & ~7;
        valid = (__shfl(todo, from + grp) >> (lane & 7) & 1) != 0;
        v = __builtin_amdgcn_readlane(v0, from) + lane;
        if (pass == 0)
          xv = elem_at<DT>(my_raw + ((from - (lane & ~7)) * 8 - (int)sub) * elem_bytes<DT>(), lane);
        else
          xv = elem_at<DT>(rowp, v < a.V ? v : a.V - 1);
        dv.M = uniform_f32(d.M, from);
        dv.emM = uniform_f32(d.emM, from);
        dv.vpos = __builtin_amdgcn_readlane(d.vpos, from);
        todo = grp == from >> 3 ? 0u : todo;
      }
      score_with(a, row, v, v, xv, dv, valid, st);
    }
  }
  publish_wave<W>(sh.fres, st);
  __syncthreads();
  const int nsurv = *sh.nsurv;
  if (nsurv > 0) {  // blocks that some wave left to all
    const float reached = row_max(lane < W ? sh.fres[lane * 8] - sh.fres[lane * 8 + 1] : kNegInf);
    if (tid == 0) *sh.bkey = float_key(reached);
    collect_candidates<DT, W>(a, sh, rowp, nsurv, reached);
    __syncthreads();
    const int ncand = *sh.ncand;
    if (ncand <= kCandCap) {
      for (int i = tid; i < ncand; i += kStepThreads) score_element(a, sh, row, sh.cand_v[i], sh.cand_x[i], true, st);
    } else {  // tie-heavy rows: block by block, skipping what the waves' best scores rule out
#pragma unroll 1
      for (int k = wave; k < nsurv; k += W) {
        const int c = sh.surv(k);
        if (ub_rounded_up(sh.ub(c)) < key_float(*sh.bkey)) continue;
        fast_visit<DT>(a, sh, rowp, row, c, st);
        const float low = wave_max(st.s - st.e);
        if (lane == 0) atomicMax(sh.bkey, float_key(low));
      }
    }
    publish_wave<W>(sh.fres, st);
    __syncthreads();
  }
  return merge_waves<W>(sh.fres);
}

// Softmax sums over parts of a row, one part per lane (its largest logit, and its sums relative to that), moved to the
// largest of all; wave-uniform.
struct RowSums {
  float m, S, Sw;
};

template <bool Entropy, bool Row>
__device__ __forceinline__ RowSums merge_sums(const StepArgs& a, float m_c, float S_c, float Sw_c) {
  RowSums r;
  r.m = Row ? row_max(m_c) : wave_max(m_c);
  const float shift = (m_c - r.m) * a.k2;
  const float f = __builtin_amdgcn_exp2f(shift);
  r.S = wave_sum(S_c > 0.0f ? S_c * f : 0.0f);
  r.Sw = 0.0f;
  if constexpr (Entropy) r.Sw = wave_sum(S_c > 0.0f ? f * fmaf(shift, S_c, Sw_c) : 0.0f);
  return r;
}

// ---------------------------------------------------------------- the kernel
// alive[row] == 0, read through the scalar data path: the aligned 32-bit word that holds the flag (it
// lies in the same page as the flag, so the read cannot fault wherever the array ends).  A workgroup
// whose row is done holds its place in the dispatcher's queue until it knows; the scalar path tells
// it sooner than a vector load.  The kernel writes the flag later with a vector store, after this
// read, and never reads it again.
__device__ __forceinline__ bool row_is_done(const uint8_t* alive, int row) {
  const uintptr_t addr = (uintptr_t)(alive + row);
  const uint32_t* word = (const uint32_t*)(addr & ~(uintptr_t)3);
  uint32_t bits;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(bits) : "s"(word) : "memory");
  return ((bits >> (8u * (uint32_t)(addr & 3))) & 0xffu) == 0u;
}

template <int DT, bool Entropy, bool Filter, bool Sum, int W>
__device__ __forceinline__ void step_row(const StepArgs& a, unsigned char* smem_raw) {
  static_assert(Sum || (!Entropy && !Filter), "entropy and filtered draws need the softmax sum");
  constexpr int kStepWaves = W, kStepThreads = W * kWave, kSlots = W * kGroups;
  const int tid = threadIdx.x;
  // workgroup (row, chunk) owns tiles [tile0, tile1) of the row
  const int nch = Filter ? 1 : a.nch;
  const int row = (int)blockIdx.x;
  const int chunk = Filter ? 0 : (int)blockIdx.y;
  if (row_is_done(a.alive, row)) {  // done rows are not decoded (Algorithm 1, loop condition)
    if (tid == 0 && chunk == 0) {
      a.tokens[row] = -1;
      a.regret[row] = 0.0f;
      if (a.logprob) a.logprob[row] = 0.0f;
      if (Entropy) a.entropy[row] = 0.0f;
    }
    return;
  }
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = lane >> 3;
  const int ntiles = a.ntiles;  // of the row
  const int tile0 = Filter ? 0 : chunk * a.chunk_tiles + min(chunk, a.chunk_extra);
  const int ctiles = Filter ? ntiles : a.chunk_tiles + (chunk < a.chunk_extra ? 1 : 0);
  const int tile1 = tile0 + ctiles;
  const int nslots = ctiles * kGroups;  // block slots of the chunk incl. the non-existent ones of the row's last tile
  const StepShared sh = carve<DT, Filter, W>(smem_raw, nslots, tile0 * kGroups);
  const void* rowp = (const char*)a.logits + (size_t)row * (size_t)a.row_stride * elem_bytes<DT>();

  // ------------------------------------------------------------ phase 1: stream the chunk
  // Wave iteration i handles tile tile0 + i*W + wave.  Lanes whose 16-byte group starts at or beyond
  // V (the row's last tile only) read the last valid group instead and are masked below.
  const int my_tiles = wave < ctiles ? (ctiles - wave + kStepWaves - 1) / kStepWaves : 0;
  const uint32_t last_group = (uint32_t)(a.V - 1) & ~7u;
  // the last 16-byte group of the chunk: where the first ring's loads of a wave with fewer tiles go
  const uint32_t chunk_last = tile1 == ntiles ? last_group : (uint32_t)tile1 * kTile - 8u;
  uint32_t lane_off = (uint32_t)lane * 8u;
  uint32_t lane_bytes = lane_off * (uint32_t)elem_bytes<DT>();
  auto load_tile = [&](int t) {  // t is wave-uniform
    if (t != ntiles - 1) return load_raw_inner<DT>((const char*)rowp + (size_t)t * kTile * elem_bytes<DT>(), lane_bytes);
    const uint32_t e0 = (uint32_t)t * kTile + lane_off;  // last tile: may be ragged
    return load_raw<DT>(rowp, e0 < last_group ? e0 : last_group, (uint32_t)a.V);
  };
  // The first ring of loads is issued by every wave, whether it has that many tiles or not
  // (addresses beyond the chunk fall back on its last group): with a fixed number of loads in
  // flight the compiler can wait for exactly the one a ring slot needs.
  Raw<DT> ring[kRing];
#pragma unroll
  for (int d = 0; d < kRing; ++d) {
    const uint32_t e0 = (uint32_t)(tile0 + d * kStepWaves + wave) * kTile + lane_off;
    ring[d] = load_raw<DT>(rowp, e0 < chunk_last ? e0 : chunk_last, (uint32_t)a.V);
  }
  // While the first loads are in flight: M_q bounds of the chunk's blocks, four per Philox call
  // (the chunk starts at a multiple of 8 blocks, so the calls' groups of four line up).
  for (int c = tid; c * 4 < nslots; c += kStepThreads) {
    const int b0 = sh.q0 + c * 4;
    const Philox4 p = philox4x32_10((uint32_t)(b0 >> 2), (uint32_t)a.step, (uint32_t)row, kTagBlock, a.key0, a.key1);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int b = b0 + j;
      float mub = kNegInf;
      if (b < a.nblocks) {
        const int32_t n = a.V - b * kDrawBlock < kDrawBlock ? a.V - b * kDrawBlock : kDrawBlock;
        mub = (__builtin_amdgcn_logf((float)n) * kLn2 + 2e-6f) + gumbel_upper_f32(p.w[j]);
        mub += 1e-5f + 4e-7f * fabsf(mub);  // room for the rounding of y_max + M_q below
      }
      if (c * 4 + j < nslots) {
        sh.mub(b) = mub;
        sh.word(b) = p.w[j];
      }
    }
  }
  __syncthreads();

  // Softmax sum against a lazily advanced per-lane reference: the lane accumulates
  // sum_v 2^(x_v k2 + nrk) with nrk = -(reference logit) * k2; the final combine multiplies
  // by 2^-(m k2 + nrk), so the rounding of nrk itself cancels.  `lead` is the logit beyond
  // which the reference has to move up (the sum would grow past 2^64 per term otherwise).
  float nrk = kNoReference;
  float lead = kNegInf;
  float sum = 0.0f;
  float sumw = 0.0f;         // entropy output: sum_v 2^t_v t_v with t_v = x_v k2 + nrk (see below)
  float mx = kNegInf;        // largest logit this lane group has seen
  float top_ub = kNegInf;    // largest block bound this lane group has seen, and its block
  int top_q = -1;
  char* const my_raw = (char*)sh.top_raw + ((size_t)(wave * kGroups + grp) * kDrawBlock + (lane & 7) * 8) * elem_bytes<DT>();
  float* const bmx_lane = Filter ? sh.bmx + (wave * kGroups + grp) : nullptr;
  float* const mu_lane = sh.mu + 2 * (wave * kGroups + grp);  // this lane group's entry of tile `wave`; 256 floats per iteration

  // One wave iteration over ring slot d, tile index i of this wave.  `Steady` iterations are
  // those that need no checks: the tile is whole, not the row's last, and its ring slot is
  // refilled with a tile that is not the last either.
  auto iteration = [&](auto steady, int d, int i) {
    constexpr bool Steady = decltype(steady)::value;
    const int t = tile0 + i * kStepWaves + wave;
    float* const mu = mu_lane + (size_t)i * (2 * kStepWaves * kGroups);
    const float mub = mu[0];  // asked for before the tile is waited for
    float x[8];
    unpack<DT>(ring[d], x);
    if (!Steady && (t + 1) * kTile > a.V) {  // ragged last tile: indices at or beyond V do not exist
      const int32_t e0 = t * kTile + (int32_t)lane_off;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (e0 + j >= a.V) x[j] = kNegInf;
      if constexpr (DT == ESPO_BF16) {  // and in what is kept of the tile
#pragma unroll
        for (int j = 0; j < 4; ++j)
          ring[d].w[j] = (__builtin_bit_cast(uint32_t, x[2 * j]) >> 16) | (__builtin_bit_cast(uint32_t, x[2 * j + 1]) & 0xFFFF0000u);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) ring[d].w[j] = __builtin_bit_cast(uint32_t, x[j]);
      }
    }
    const float gm = max8(x);
    if constexpr (Sum) {
      if (__builtin_amdgcn_ballot_w64(gm > lead) != 0) {  // rare after the first tile
        asm volatile("" ::: "memory");  // keep this rare path out of the straight-line code
        if (gm > lead) {  // move this lane's reference up to gm
          const float nrk_new = lane_reference(gm, a.k2);
          const float shift = nrk_new - nrk;  // every t_v moves by this much
          const float f = __builtin_amdgcn_exp2f(shift);
          if (Entropy) sumw = f * fmaf(shift, sum, sumw);
          sum *= f;
          nrk = nrk_new;
          lead = gm + a.ref_lead;
        }
      }
    }
    if constexpr (!Sum) {
      // nobody asked for the log-probability, the entropy or a filtered draw: token, regret and
      // state need the row maximum only, and the eight fma / exp2 / add per lane are left out
    } else if constexpr (!Entropy) {
      float acc0 = __builtin_amdgcn_exp2f(fmaf(x[0], a.k2, nrk));
      float acc1 = __builtin_amdgcn_exp2f(fmaf(x[1], a.k2, nrk));
#pragma unroll
      for (int j = 2; j < 8; j += 2) {
        acc0 += __builtin_amdgcn_exp2f(fmaf(x[j], a.k2, nrk));
        acc1 += __builtin_amdgcn_exp2f(fmaf(x[j + 1], a.k2, nrk));
      }
      sum += acc0 + acc1;
    } else {
      // The entropy needs sum_v pi_v ln pi_v = (ln 2 / S) sum_v 2^t_v t_v - ln S.  t_v is kept
      // above -200: 2^t_v is 0 in fp32 from far above that, so the sum is unchanged and a
      // masked logit (-inf) contributes 0 * -200 instead of 0 * -inf.
      float acc0 = 0.0f, acc1 = 0.0f, w0 = 0.0f, w1 = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float t0 = fmaxf(fmaf(x[j], a.k2, nrk), -200.0f), t1 = fmaxf(fmaf(x[j + 1], a.k2, nrk), -200.0f);
        const float e0 = __builtin_amdgcn_exp2f(t0), e1 = __builtin_amdgcn_exp2f(t1);
        acc0 += e0;
        acc1 += e1;
        w0 = fmaf(e0, t0, w0);
        w1 = fmaf(e1, t1, w1);
      }
      sum += acc0 + acc1;
      sumw += w0 + w1;
    }
    // upper bound of every perturbed score in the lane group's block: y_max + M_q
    const float bm = group8_max(gm);
    const float ub = fmaf(bm, a.inv_tau, mub);
    mu[1] = ub;  // the 8 lanes of the group store the same value
    if constexpr (Filter) bmx_lane[(size_t)i * (kStepWaves * kGroups)] = bm;
    mx = fmaxf(mx, bm);
    if (ub > top_ub) {  // keep the data of the block with the group's largest bound
      top_ub = ub;
      top_q = t * kGroups + grp;
      *(u32x4*)my_raw = u32x4{ring[d].w[0], ring[d].w[1], ring[d].w[2], ring[d].w[3]};
      if constexpr (DT == ESPO_F32) *(u32x4*)(my_raw + 16) = u32x4{ring[d].w[4], ring[d].w[5], ring[d].w[6], ring[d].w[7]};
    }
    if (Steady)  // refill this ring slot
      ring[d] = load_raw_inner<DT>((const char*)rowp + (size_t)(t + kRing * kStepWaves) * kTile * elem_bytes<DT>(), lane_bytes);
    else if (i + kRing < my_tiles)
      ring[d] = load_tile(t + kRing * kStepWaves);
  };
  // Steady passes: all kRing tiles and their refills lie before this wave's last tile.
  const int steady_end = my_tiles > 2 * kRing ? ((my_tiles - kRing - 1) / kRing) * kRing : 0;
  int i0 = 0;
#pragma unroll 1
  for (; i0 < steady_end; i0 += kRing) {
#pragma unroll
    for (int d = 0; d < kRing; ++d) iteration(std::true_type{}, d, i0 + d);
  }
#pragma unroll 1
  for (; i0 < my_tiles; i0 += kRing) {
#pragma unroll
    for (int d = 0; d < kRing; ++d)
      if (i0 + d < my_tiles) iteration(std::false_type{}, d, i0 + d);  // wave-uniform
  }
  // The wave's largest logit and its share of the softmax sums relative to that.  All of it, like the first scores of the
  // search, comes before the barrier: the waves of a workgroup end their streaming microseconds apart.
  const float mw = wave_max(mx);
  if (lane == 0) sh.m[wave] = mw;
  if constexpr (Sum) {
    const float shift = -fmaf(mw, a.k2, nrk);  // from this lane's reference to the wave's maximum
    const float f = __builtin_amdgcn_exp2f(shift);
    const float tot = wave_sum(sum > 0.0f ? sum * f : 0.0f);
    if (lane == 0) sh.sum[wave] = tot;
    if constexpr (Entropy) {
      const float totw = wave_sum(sum > 0.0f ? f * fmaf(shift, sum, sumw) : 0.0f);
      if (lane == 0) sh.sumw[wave] = totw;
    }
  }
  float z_prev = 0.0f, value = 0.0f;  // wanted at the very end: fetched now, off the critical path
  if (tid == 0) {
    z_prev = a.z[row];
    value = a.values[row];
  }

  // ------------------------------------------------------------ phase 2: argmax of y + G
  auto row_sums = [&]() {  // after a barrier: the waves' shares put together (in a fixed order, the same in every wave)
    return merge_sums<Entropy, true>(a, lane < kStepWaves ? sh.m[lane] : kNegInf, Sum && lane < kStepWaves ? sh.sum[lane] : 0.0f,
                               Entropy && lane < kStepWaves ? sh.sumw[lane] : 0.0f);
  };
  int32_t tok;
  float x_a;
  float s_a = kNegInf, e_a = 0.0f;  // the winner's score as a float known to within +-e_a (what the combine of a split row compares)
  // the argmax over the indices whose logit is above shx.floor: fp32 search, decided in double where needed
  auto search = [&](const StepShared& shx) {
    const Best fast = fast_argmax<DT, Filter, W>(a, shx, rowp, row, my_tiles, top_q, top_ub, my_raw);
    tok = fast.v;
    x_a = fast.x;
    s_a = fast.s;
    e_a = fast.e;
    if (fast.v >= 0 && !(fast.s - fast.e > fast.hi2)) {
      // the two best fp32 scores overlap within their margins: decide in double (rare)
      __syncthreads();  // everyone has read the fp32 results
      Search<double> exact;
      if (!exact_among_candidates<DT, W>(a, shx, rowp, row, nslots, fast.s - fast.e, exact)) {
        __syncthreads();
        exact = find_argmax<DT, W>(a, shx, rowp, row, nslots, (double)fast.s - (double)fast.e);
      }
      tok = exact.best.v;
      x_a = exact.best.x;
      s_a = (float)exact.best.s;                 // rounded to float: within 2^-24 relative of the double score
      e_a = fmaf(fabsf(s_a), 1.2e-7f, 1e-30f);
    }
  };
  RowSums sums;
  if constexpr (!Filter) {
    search(sh);
  } else {
    __syncthreads();  // the waves' maxima and sums are in place
    sums = row_sums();
    tok = -1;         // a row without a finite logit keeps this
    x_a = 0.0f;
  }

  if constexpr (Filter) {
    // The general search of a filtered draw, for the rows that filtered_row hands on (ties that fill its lists, a
    // kept set of thousands of logits, a winner whose membership fp32 cannot tell).  The kept set is
    // {v : the mass (the number) of strictly larger logits is below p (k)}, an upper set in the logit, so the
    // winner of the unfiltered search is the token if it is kept, and otherwise the search is repeated above it:
    // whether it is kept follows from the mass (number) of the logits above its own.  The floor rises strictly, so
    // the loop ends, after 1/p rounds on average.  A table of the blocks' largest logits, filled while streaming,
    // names the blocks that hold any; up to two thirds of the row's blocks are read again block by block, more of
    // them by one more pass over the row.  Sums within 1e-5 of p times the softmax sum are formed again in double
    // over the whole row, in the oracle's arithmetic.
    const bool by_count = a.top_k > 0;
    const float m = sums.m, total = sums.S;
    const float want = a.top_p * total;
    float mass = 0.0f, count = 0.0f;

    auto measure = [&](float floor_x) {  // mass and number of the logits above floor_x
      __syncthreads();  // whatever used the scratch before is over in every wave
      if (tid == 0) *sh.nsurv = 0;
      __syncthreads();
      for (int b = tid; b < nslots; b += kStepThreads)  // blocks that hold a logit above the floor
        if (sh.bmx[b] > floor_x) sh.surv(atomicAdd(sh.nsurv, 1)) = b;
      __syncthreads();
      const int nabove = *sh.nsurv;
      float acc_m = 0.0f, acc_n = 0.0f;
      auto add = [&](const Raw<DT>& raw, int32_t v0, bool valid) {
        float x[8];
        unpack<DT>(raw, x);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const bool above = valid && v0 + u < a.V && x[u] > floor_x;
          acc_m += above ? weight_below(x[u], m, a.k2) : 0.0f;
          acc_n += above ? 1.0f : 0.0f;  // counts stay exact in fp32: V < 2^24
        }
      };
      constexpr int kLoads = 4, kDeep = DT == ESPO_F32 ? 5 : 6;  // (with 6 of fp32 a register goes to scratch)
      if (3 * nabove <= 2 * nslots) {
        // the listed blocks only, laid out as in phase 1: a lane group of 8 lanes per block, 16 bytes per lane
        const uint32_t sub = (uint32_t)(lane & 7) * 8u;
#pragma unroll 1
        for (int base = wave * kGroups; base < nabove; base += kLoads * kStepWaves * kGroups) {
          int qs[kLoads];
          Raw<DT> raw[kLoads];
#pragma unroll
          for (int j = 0; j < kLoads; ++j) {
            const int k = base + j * kStepWaves * kGroups + grp;
            qs[j] = k < nabove ? sh.surv(k) : -1;
            // a group without a block reads block 0 and drops it; a ragged last block is masked
            const uint32_t e0 = (uint32_t)(qs[j] < 0 ? 0 : qs[j]) * kDrawBlock + sub;
            raw[j] = load_raw<DT>(rowp, e0 < last_group ? e0 : last_group, (uint32_t)a.V);
          }
#pragma unroll
          for (int j = 0; j < kLoads; ++j) add(raw[j], qs[j] * kDrawBlock + (int32_t)sub, qs[j] >= 0);
        }
      } else {
#pragma unroll 1
        for (int i0 = 0; i0 < my_tiles; i0 += kDeep) {
          Raw<DT> raw[kDeep];
#pragma unroll
          for (int d = 0; d < kDeep; ++d)
            if (i0 + d < my_tiles) raw[d] = load_tile((i0 + d) * kStepWaves + wave);
#pragma unroll
          for (int d = 0; d < kDeep; ++d)
            if (i0 + d < my_tiles) add(raw[d], ((i0 + d) * kStepWaves + wave) * kTile + (int32_t)lane_off, true);
        }
      }
      acc_m = wave_sum(acc_m);
      acc_n = wave_sum(acc_n);
      if (lane == 0) {
        sh.res_s[wave] = (double)acc_m;
        sh.fres[wave] = acc_n;
      }
      __syncthreads();
      mass = 0.0f;
      count = 0.0f;
      for (int w = 0; w < kStepWaves; ++w) {  // fixed order, the same in every thread
        mass += (float)sh.res_s[w];
        count += sh.fres[w];
      }
    };

    StepShared above = sh;
    if (a.top_k == 1 && m > kNegInf) {  // kept: what equals the row maximum; one search above the largest float below it
      const int32_t bits = __builtin_bit_cast(int32_t, m);
      above.floor = m == 0.0f ? -1.401298464e-45f : __builtin_bit_cast(float, bits + (m > 0.0f ? -1 : 1));
    }
    while (m > kNegInf) {  // (a row without a finite logit has no winner)
      asm volatile("" : "+v"(lane_off), "+v"(lane_bytes));  // no address that follows from them is kept in registers from round to round
      search(above);
      if (tok < 0 || a.top_k == 1) break;
      measure(x_a);
      bool kept;
      if (by_count) {
        kept = count < (float)a.top_k;
      } else if (fabsf(mass - want) > 1e-5f * total) {
        kept = mass < want;
      } else {  // too close for fp32: the same two sums in double, y and y_max formed as the oracle forms them
        const double inv = (double)a.inv_tau, y_max = (double)m * inv;
        double dm = 0.0, ds = 0.0;
#pragma unroll 1
        for (int i = 0; i < my_tiles; ++i) {
          const int t = i * kStepWaves + wave;
          const Raw<DT> raw = load_tile(t);
          float x[8];
          unpack<DT>(raw, x);
          const int32_t e0 = t * kTile + (int32_t)lane_off;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (e0 + u < a.V && x[u] > kNegInf) {
              const double e = exp((double)x[u] * inv - y_max);
              ds += e;
              if (x[u] > x_a) dm += e;
            }
          }
        }
        dm = wave_sum_f64(dm);
        ds = wave_sum_f64(ds);
        __syncthreads();
        if (lane == 0) {
          sh.res_s[wave] = dm;
          sh.res_hi2[wave] = ds;
        }
        __syncthreads();
        double dmass = 0.0, dtotal = 0.0;
        for (int w = 0; w < kStepWaves; ++w) {
          dmass += sh.res_s[w];
          dtotal += sh.res_hi2[w];
        }
        kept = dmass < (double)a.top_p * dtotal;
      }
      if (kept) break;
      above.floor = x_a;
      __syncthreads();  // the sums have been read by everyone
    }
  }

  // ------------------------------------------------------------ finalize: one lane
  if (wave != 0) return;
  if constexpr (!Filter) sums = row_sums();
  float m = sums.m, S = sums.S, Sw = sums.Sw;  // over the chunk
  if constexpr (!Filter) {
    if (nch > 1) {
      // A row split over nch workgroups: each leaves its chunk's result in the workspace and then looks at what all of them
      // have left; the one that finds every result there finishes the row.  The last to write does find them all: its
      // own have been acknowledged before it looks, and so have the others'.  Two may: they come to the same outputs, from a z that both
      // have read before either could write it.  Nobody waits for another workgroup.  Words are written and read with
      // device-scope atomic accesses, which bypass the caches that are private to a part of the chip.  (A device-scope
      // fence would do too, but writes back and invalidates a whole L2 per workgroup: measured, 50 ns
      // of serialised work per workgroup, 100 us per launch.  A ticket taken by compare-and-swap after the results
      // is one more trip through memory, and one more again where two chunks take it at a time: 7200 cycles from the search
      // to the outputs of B = 64, V = 152064 bf16, against 5000 now; B = 4, V = 150001 fp32 with the entropy, 8 chunks: 13.8 -> 11.3 us,
      // the shorter search included.)  A word without the mark is not there, so the workspace may hold anything before the launch; who
      // finishes a row leaves its words zero, so that nothing of this launch can pass for a result in a later one.
      unsigned long long* const row_mail = a.mail + (size_t)row * (size_t)(nch * kMailRoom);
      asm volatile("" : "+v"(z_prev) : : "memory");  // z has arrived before this chunk's words let another one finish the row and write it
      {
        const uint32_t w = lane == 0 ? __builtin_bit_cast(uint32_t, m) : lane == 1 ? __builtin_bit_cast(uint32_t, S)
                           : lane == 2 ? __builtin_bit_cast(uint32_t, Sw) : lane == 3 ? __builtin_bit_cast(uint32_t, s_a)
                           : lane == 4 ? __builtin_bit_cast(uint32_t, e_a) : lane == 5 ? __builtin_bit_cast(uint32_t, x_a) : (uint32_t)tok;
        if (lane < kMailWords) __hip_atomic_store(row_mail + lane * nch + chunk, (unsigned long long)kMailMark << 32 | w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // acknowledged before the others' words are read
      }
      // lane c holds chunk c (nch <= 64); the other lanes hold a chunk without any finite logit
      float m_c = kNegInf, S_c = 0.0f, Sw_c = 0.0f;
      Best win = no_best();
      bool there = true;
      if (lane < nch) {
        uint32_t w[kMailWords];
#pragma unroll
        for (int j = 0; j < kMailWords; ++j) {
          const unsigned long long word = __hip_atomic_load(row_mail + j * nch + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          w[j] = (uint32_t)word;
          there = there && (uint32_t)(word >> 32) == kMailMark;
        }
        m_c = __builtin_bit_cast(float, w[0]);
        S_c = __builtin_bit_cast(float, w[1]);
        Sw_c = __builtin_bit_cast(float, w[2]);
        win.s = __builtin_bit_cast(float, w[3]);
        win.e = __builtin_bit_cast(float, w[4]);
        win.x = __builtin_bit_cast(float, w[5]);
        win.v = (int32_t)w[6];
        if (win.v < 0) win = no_best();
      }
      if (__builtin_amdgcn_ballot_w64(!there) != 0) return;
      // all of the row's bytes of the workspace: sixteen to a lane, one store unless a caller forces more than sixteen chunks
      // (behind the row's own results they would hold up the end of the launch: 0.2 us)
      for (int k = lane * 2; k < nch * kMailRoom; k += 2 * kWave) *(u32x4*)(row_mail + k) = u32x4{0u, 0u, 0u, 0u};
      sums = merge_sums<Entropy, false>(a, m_c, S_c, Sw_c);  // the chunks' sums are relative to their own maxima
      m = sums.m;
      S = sums.S;
      Sw = sums.Sw;
      // every chunk's winner is its exact argmax, so the row's is the best of them: decided in fp32
      // where the margins allow, else by scoring those few indices in double
      const Best top = wave_best(win);
      tok = top.v;
      x_a = top.x;
      if (top.v >= 0 && !(top.s - top.e > top.hi2)) {
        Search<double> st;
        st.init();
        if (win.v >= 0) {
          const BlockDraw<double> d = block_draw<double>(a, row, win.v >> 6);
          score_index<double>(a, row, win.v, win.x, d, -__builtin_huge_val(), kNegInf, st);
        }
        st = wave_merge(st);
        tok = st.best.v;
        x_a = st.best.x;
      }
    }
  }
  if (lane == 0) finish_row<DT, Entropy, Sum>(a, row, rowp, tok, x_a, m, S, Sw, z_prev, value);
}

template <int DT, bool Entropy, bool Sum, int W>
// Registers: workgroups of 8 waves get up to 80 (three of them fit on a compute unit, in registers and in LDS) and use 73;
// one of 16 waves, which has a compute unit to itself (plan_step), may have 128 and uses 73 too.  Workgroups of 4 waves, which
// the diagnostics entry point alone launches, are held to 64 and keep some 15 registers in scratch.
__global__ __launch_bounds__(W * kWave, W == 8 ? 6 : W == 16 ? 4 : 8) void espo_step_kernel(StepArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  step_row<DT, Entropy, false, Sum, W>(a, smem_raw);
}

// ---------------------------------------------------------------- filtered draws
// The filtered token is the argmax of y + G over the kept set {x >= x*}, an upper set in the logit,
// so neither a block's bound nor any index below x* is needed: what is needed is the row's largest
// logits.  They are collected while the row streams.  A wave keeps the raw 16 (fp32: 32) bytes of
// every lane whose 8 logits hold one above the wave's threshold, in an LDS list of its own (no
// atomics, no barrier); when the list grows past kCompactAt the wave raises its threshold to about
// the kKeep-th largest of the packs' maxima and drops the rest.  Every logit of the row above
// T = the largest of the waves' thresholds is then in LDS, some 800 packs of a long row, and nothing
// is read from memory again:
//   1. row maximum m, T, softmax sum S;
//   2. the logits above T are binned by value (256 bins of equal width), weights 2^t as integers in
//      units of 2^-31 of S (1 for top-k), so the sums do not depend on their order;
//   3. the bins' prefix sum tells whether the mass (number) above T exceeds p S (k) and names the bin
//      with the edge of the kept set; logits in bins before it are kept, those in it are compared with
//      each other;
//   4. the kept logits are scored, one per thread, and the best one is the token.
// Sums within 1e-5 of p S are not trusted: such a logit takes part in the search, and if it wins, or
// if the kept set reaches below T, or a list does not hold what it has to, the row goes through the
// general search of step_row from the start.
// Bound by the streaming like the plain draw: B = 512, V = 152064 bf16, us per launch, against a
// search for the edge that read the row's blocks again after a trial floor: top-p 0.7 at temperature
// 0.6 / 0.8 / 1.0: 35.0 / 34.8 / 35.6 (44.1 / 48.7 / 67.3), top-k 50 at 1.0: 35.3 (48.8), the plain
// draw at 1.0: 36.4 (now 32.2 / 32.2 / 36.1, 32.5, the plain draw 33.7).  B = 100, V = 50003, top-k 50: 13.6 (24.9; now 12.3).  What is
// left after the last tile is five barriers: sums, bins, edge, kept logits, scores.  The lists' room is what two workgroups of 8 waves on a
// compute unit leave (73 KB of LDS each); 16 waves are used below 256 rows (13.6 against 16.0 us there).
constexpr int kKeptCap2 = 3072, kEdgeBins = 256, kEdgeMembers = 256;
constexpr int32_t kInDoubt = 1 << 30;  // on top of an index whose membership of the kept set fp32 cannot tell

template <int DT, int W>
struct CollectLimits {  // packs of a wave's list: room, when it is compacted, what is kept then; tiles between two checks
  static constexpr int kRoom = W == 8 ? (DT == ESPO_BF16 ? 448 : 256) : (DT == ESPO_BF16 ? 320 : 192);
  static constexpr int kCheckTiles = W == 8 && DT == ESPO_BF16 ? 2 : 1;
  static constexpr int kCompactAt = kRoom - kCheckTiles * kWave;
  static constexpr int kKeep = (DT == ESPO_BF16 ? 160 : 112) * 8 / W;
};

// What a compaction leaves of a wave's list.  A nucleus may need all of it.  Of a top-k draw a wave keeps little more than k packs, so that
// fewer logits are binned and collected afterwards, but no fewer than that: the row's largest logits may all be this wave's (common
// tokens with neighbouring indices), and with fewer than k of them above T the row has to be read again.  us, what a nucleus gets / so /
// a share of 10 k for each wave, k = 20: V = 50003 bf16, B = 100, synthetic rows 13.1 / 11.8 / 11.6, their largest logits within one tile 14.4 / 12.5 / 34.5;
// V = 152064, B = 300: 30.7 / 26.6 / 26.2, 32.1 / 26.5 / 60.8; k = 50, V = 50003, B = 100: 13.4 / 12.9 / 11.9, 14.9 / 14.6 / 32.4.
// From two thirds of kKeep on, k packs at the least make the lists longer than they have to be (k = 128, B = 300: 20.4 -> 21.1).
struct Kept {
  int least, most;
};
template <int DT, int W>
__device__ __forceinline__ Kept packs_kept(const StepArgs& a) {
  constexpr int kAll = CollectLimits<DT, W>::kKeep;
  if (a.top_k == 0 || a.top_k > kAll * 2 / 3) return Kept{kAll / 2, kAll};
  const int most = min(max(a.top_k * 8 / 5, 16), kAll);
  return Kept{max(a.top_k, most / 2), most};
}

template <int DT, int W>
struct FilterShared {
  uint32_t* raw;     // [W][kRoom][words] the packs ...
  uint16_t* id;      // [W][kRoom] ... and which 8 indices of the row each holds
  uint16_t* kept;    // [kKeptCap2] logits kept for sure: pack * 8 + position
  uint32_t* bins;    // [kEdgeBins]
  float* mem_x;      // [kEdgeMembers] logits in the edge's bin, their weights, and where they are
  uint32_t* mem_w;
  uint16_t* mem_at;
  float *m, *thr, *low, *least, *sum, *sumw;  // [W]
  float* fres;       // [W][8]
  double *res_s, *res_hi2;
  float* res_e;
  int* res_v;
  float* res_x;
  int *nkept, *nmem, *nover;
  int* edge;         // [4] weight of all bins, the two edges' bins, the weight above the first of them
};

template <int DT, int W>
__host__ __device__ constexpr size_t filter_lds_bytes() {
  constexpr size_t packs = (size_t)W * CollectLimits<DT, W>::kRoom;
  return packs * (DT == ESPO_BF16 ? 16 : 32) + packs * 2 + kKeptCap2 * 2 + kEdgeBins * 4 + kEdgeMembers * 10 +
         W * (6 + 8 + 3) * 4 + W * 16 + 32;
}

template <int DT, int W>
__device__ __forceinline__ FilterShared<DT, W> carve_filter(unsigned char* base) {
  constexpr size_t packs = (size_t)W * CollectLimits<DT, W>::kRoom;
  FilterShared<DT, W> f;
  size_t off = 0;
  auto take = [&](size_t bytes) { void* p = base + off; off += bytes; return p; };  // sizes are multiples of 16 down to `m`
  f.raw = (uint32_t*)take(packs * (DT == ESPO_BF16 ? 16 : 32));
  f.res_s = (double*)take(W * 8);
  f.res_hi2 = (double*)take(W * 8);
  f.bins = (uint32_t*)take(kEdgeBins * 4);
  f.mem_x = (float*)take(kEdgeMembers * 4);
  f.mem_w = (uint32_t*)take(kEdgeMembers * 4);
  f.m = (float*)take(W * 4);
  f.thr = (float*)take(W * 4);
  f.low = (float*)take(W * 4);
  f.least = (float*)take(W * 4);
  f.sum = (float*)take(W * 4);
  f.sumw = (float*)take(W * 4);
  f.fres = (float*)take(8 * W * 4);
  f.res_e = (float*)take(W * 4);
  f.res_v = (int*)take(W * 4);
  f.res_x = (float*)take(W * 4);
  f.nkept = (int*)take(16);
  f.nmem = f.nkept + 1;
  f.nover = f.nkept + 2;
  f.edge = (int*)take(16);
  f.id = (uint16_t*)take(packs * 2);
  f.kept = (uint16_t*)take(kKeptCap2 * 2);
  f.mem_at = (uint16_t*)take(kEdgeMembers * 2);
  return f;
}

// The lane's logits; those at or beyond V, which a ragged row's last pack holds, become -inf.
template <int DT>
__device__ __forceinline__ void pack_unpack(const Raw<DT>& r, int32_t v0, int32_t V, float x[8]) {
  unpack<DT>(r, x);
  if (v0 + 8 > V) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (v0 + j >= V) x[j] = kNegInf;
  }
}

// Raises a wave's threshold to a value that at most `keep.most` of the list's packs reach beyond and drops the
// others.  (Packs that tie at the threshold are dropped as well: what is kept is everything above it.)
template <int DT, int W>
__device__ __forceinline__ void compact_list(uint32_t* raw, uint16_t* id, int32_t V, const Kept& keep, int& n, float& thr) {
  using Lim = CollectLimits<DT, W>;
  constexpr int kRounds = Lim::kRoom / kWave, kWords = Raw<DT>::kWords;
  const int lane = threadIdx.x & (kWave - 1);
  float pm[kRounds];
  float top = kNegInf, bottom = kNegInf;  // bottom: of the negated maxima
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int i = r * kWave + lane;
    pm[r] = kNegInf;
    if (i < n) {
      float x[8];
      pack_unpack<DT>(pack_load<DT>(raw + i * kWords), (int32_t)id[i] * 8, V, x);
      pm[r] = max8(x);
      bottom = fmaxf(bottom, -pm[r]);
    }
    top = fmaxf(top, pm[r]);
  }
  float hi = wave_max(top), lo = -wave_max(bottom);  // none above hi; the search leaves at most `keep.most` above hi
#pragma unroll 1
  for (int it = 0; it < 12; ++it) {
    const float mid = 0.5f * lo + 0.5f * hi;
    int c = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) c += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(pm[r] > mid));
    if (c > keep.most) {
      lo = mid;
    } else {
      hi = mid;
      if (c >= keep.least) break;
    }
  }
  thr = hi;
  int kept = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {  // in place: an entry never moves up, and a round reads before it writes
    const bool stays = pm[r] > thr;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(stays);
    if (stays) {
      const int i = r * kWave + lane, to = kept + rank_below(mask);
      const Raw<DT> p = pack_load<DT>(raw + i * kWords);
      const uint16_t which = id[i];
      pack_store<DT>(raw + to * kWords, p);
      id[to] = which;
    }
    kept += (int)__builtin_popcountll(mask);
  }
  n = kept;
}

// The two forms of the collected logits, seen by one thread.  An entry is named by its place `at` in the list.
template <int DT, int W>
struct PackList {  // the wave's packs of 8, some 250 of them; each lane owns every 64th
  static constexpr int kRoom = CollectLimits<DT, W>::kRoom, kRounds = kRoom / kWave;
  const FilterShared<DT, W>& f;
  int n;          // packs of this wave
  int32_t V;
  // of each of this lane's packs: the bin of its largest logit (kEdgeBins: none above T), and from bit 16 on
  // which of its logits are above T (most packs in the list hold one)
  uint32_t info[kRounds];
  float mass;  // of all logits above T, set by a draw that reaches below it
  __device__ __forceinline__ int count() const {  // this lane's logits above T
    int c = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) c += (int)__builtin_popcount(info[r] >> 16);
    return c;
  }
  __device__ __forceinline__ uint32_t place(int r) const {
    return (uint32_t)((threadIdx.x >> 6) * kRoom + r * kWave + (threadIdx.x & (kWave - 1))) * 8u;
  }
  __device__ __forceinline__ float logit(uint32_t at) const { return elem_at<DT>((const char*)f.raw, (int64_t)at); }
  __device__ __forceinline__ int32_t index(uint32_t at) const { return (int32_t)f.id[at >> 3] * 8 + (int32_t)(at & 7u); }
  template <typename Bin, typename Weight>
  __device__ __forceinline__ void fill_bins(float bottom, Bin&& bin_of, Weight&& weight_of) {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      info[r] = kEdgeBins;
      const int i = r * kWave + (int)(threadIdx.x & (kWave - 1));
      if (i < n) {
        float x[8];
        const uint32_t at = place(r);
        pack_unpack<DT>(pack_load<DT>(f.raw + (at >> 3) * Raw<DT>::kWords), index(at), V, x);
        uint32_t over = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) over |= x[j] > bottom ? 1u << j : 0u;
        if (over != 0) info[r] = (uint32_t)bin_of(max8(x)) | (over << 16);
        for (; over != 0; over &= over - 1) {
          const float xo = logit(at + (uint32_t)__builtin_ctz(over));
          atomicAdd(&f.bins[bin_of(xo)], weight_of(xo));
        }
      }
    }
  }
  // use(at, x, bin) for this thread's logits above T in bins up to last_bin
  template <typename Bin, typename Use>
  __device__ __forceinline__ void for_each(float, int last_bin, Bin&& bin_of, Use&& use) const {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      if ((int)(info[r] & 0xffffu) > last_bin) continue;
      for (uint32_t over = info[r] >> 16; over != 0; over &= over - 1) {
        const uint32_t at = place(r) + (uint32_t)__builtin_ctz(over);
        const float x = logit(at);
        const int b = bin_of(x);
        if (b <= last_bin) use(at, x, b);
      }
    }
  }
};

template <int DT, int W>
struct LogitList {  // single logits with their indices, in the space of the packs
  static constexpr int kBytes = CollectLimits<DT, W>::kRoom * (DT == ESPO_BF16 ? 16 : 32);  // of one wave
  static constexpr int kRoom = kBytes / (DT == ESPO_BF16 ? 6 : 8) / 8 * 8;
  const FilterShared<DT, W>& f;
  int n;  // logits of this wave
  float mass;
  __device__ __forceinline__ int32_t* index_area() const { return (int32_t*)f.raw; }                             // [W][kRoom]
  __device__ __forceinline__ void* logit_area() const { return index_area() + W * kRoom; }            // [W][kRoom]
  __device__ __forceinline__ float logit(uint32_t at) const { return elem_at<DT>(logit_area(), (int64_t)at); }
  __device__ __forceinline__ int32_t index(uint32_t at) const { return index_area()[at]; }
  __device__ __forceinline__ void put(int wave, int i, int32_t v, float x) const {
    const int at = wave * kRoom + i;
    index_area()[at] = v;
    if constexpr (DT == ESPO_BF16) ((uint16_t*)logit_area())[at] = (uint16_t)(__builtin_bit_cast(uint32_t, x) >> 16);
    else ((float*)logit_area())[at] = x;
  }
  template <typename Bin, typename Weight>
  __device__ __forceinline__ void fill_bins(float, Bin&& bin_of, Weight&& weight_of) {
    for (int i = threadIdx.x & (kWave - 1); i < n; i += kWave) {
      const float x = logit((threadIdx.x >> 6) * kRoom + i);
      atomicAdd(&f.bins[bin_of(x)], weight_of(x));
    }
  }
  template <typename Bin, typename Use>
  __device__ __forceinline__ void for_each(float, int last_bin, Bin&& bin_of, Use&& use) const {
    for (int i = threadIdx.x & (kWave - 1); i < n; i += kWave) {
      const uint32_t at = (threadIdx.x >> 6) * kRoom + i;
      const float x = logit(at);
      const int b = bin_of(x);
      if (b <= last_bin) use(at, x, b);
    }
  }
};

enum DrawResult { kDrawn, kReachesBelow, kUndecided };

// The draw from one of them: all logits of the row above `bottom` (< m) are in the list.  The same result in
// every thread; f.bins and the two counters are zero and the list is complete when it is called.
template <int DT, int W, typename List>
__device__ __forceinline__ DrawResult draw_from_list(const StepArgs& a, const FilterShared<DT, W>& f, List& list, int row, float m,
                                                     float S, float bottom, int32_t& tok, float& x_a) {
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool by_count = a.top_k > 0;
  // ---------------------------------------------------------- bins
  const float want = a.top_p * S;
  const float slack = by_count ? 0.0f : 1e-5f * S;  // what an fp32 sum may be off by
  const float per_logit = (float)kEdgeBins / (m - bottom);
  const float scale = by_count ? 1.0f : 2147483648.0f / (S * 1.001f);
  auto bin_of = [&](float x) {  // rounding is monotone: a larger logit never lands in a later bin
    return (int)min((uint32_t)(int)((m - x) * per_logit), (uint32_t)kEdgeBins - 1u);
  };
  auto weight_of = [&](float x) {
    return by_count ? 1u : (uint32_t)(weight_below(x, m, a.k2) * scale + 0.5f);
  };
  list.fill_bins(bottom, bin_of, weight_of);
  __syncthreads();
  // the weight above each bin, and the last bins that have logits and less than the two limits above them: the two edges
  // (kept for sure, may be kept) lie in these bins or between them.  One wave works them out while the others wait: all of
  // them together, four to a SIMD, took 1900 cycles for what this one, alone on its own, does in 1000 (V = 30000 bf16, top-p 0.7, B = 30: 12.0 -> 11.6 us, the
  // sums formed ahead of the first barrier included).
  static_assert(kEdgeBins == 4 * kWave, "four bins per lane");
  if (wave == 0) {
    const float limit_f = by_count ? (float)a.top_k : (want + slack) * scale;
    const float limit_sure_f = by_count ? (float)a.top_k : (want - slack) * scale;
    const uint32_t limit = limit_f < 1.0f ? 1u : limit_f < 4.0e9f ? (uint32_t)limit_f : 4000000000u;
    const uint32_t limit_sure = limit_sure_f < 1.0f ? 1u : limit_sure_f < 4.0e9f ? (uint32_t)limit_sure_f : 4000000000u;
    const u32x4 h = ((const u32x4*)f.bins)[lane];
    const uint32_t lane_total = h[0] + h[1] + h[2] + h[3];
    uint32_t incl = lane_total;
    incl += dpp_u32<kDppRowShr1, 0xf>(0u, incl);
    incl += dpp_u32<kDppRowShr2, 0xf>(0u, incl);
    incl += dpp_u32<kDppRowShr4, 0xf>(0u, incl);
    incl += dpp_u32<kDppRowShr8, 0xf>(0u, incl);
    incl += dpp_u32<kDppBcast15, 0xa>(0u, incl);
    incl += dpp_u32<kDppBcast31, 0xc>(0u, incl);
    uint32_t above[4];
    above[0] = incl - lane_total;
#pragma unroll
    for (int u = 1; u < 4; ++u) above[u] = above[u - 1] + h[u - 1];
    float best = -1.0f, best_sure = -1.0f;
    uint32_t above_best = 0;  // the weight above the lane's best_sure
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (h[u] != 0 && above[u] < limit) best = (float)(4 * lane + u);
      if (h[u] != 0 && above[u] < limit_sure) {
        best_sure = (float)(4 * lane + u);
        above_best = above[u];
      }
    }
    const int last = (int)wave_max(best);       // the bin of the largest logit at least: nothing is above it
    const int edge = (int)wave_max(best_sure);  // not after `last`: its limit is the smaller one
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    const uint32_t at_edge = (uint32_t)__builtin_amdgcn_readlane((int)above_best, edge >> 2);
    if (lane == 0) {
      f.edge[0] = (int)total;
      f.edge[1] = last;
      f.edge[2] = edge;
      f.edge[3] = (int)at_edge;
    }
  }
  __syncthreads();
  const uint32_t total = (uint32_t)f.edge[0], above_edge = (uint32_t)f.edge[3];
  const int last_bin = __builtin_amdgcn_readfirstlane(f.edge[1]), edge_bin = __builtin_amdgcn_readfirstlane(f.edge[2]);
  if (by_count ? total < (uint32_t)a.top_k : !((float)total / scale - want > slack)) {
    list.mass = (float)total / scale;
    return kReachesBelow;
  }
  // ---------------------------------------------------------- the kept logits, and the edge bin's members
  list.for_each(bottom, last_bin, bin_of, [&](uint32_t at, float x, int b) {
    if (b < edge_bin) {
      const int c = atomicAdd(f.nkept, 1);
      if (c < kKeptCap2) f.kept[c] = (uint16_t)at;
    } else {
      const int c = atomicAdd(f.nmem, 1);
      if (c < kEdgeMembers) {
        f.mem_x[c] = x;
        f.mem_w[c] = weight_of(x);
        f.mem_at[c] = (uint16_t)at;
      }
    }
  });
  __syncthreads();
  const int nkept = *f.nkept, nmem = *f.nmem;
  if (nkept > kKeptCap2 || nmem > kEdgeMembers) return kUndecided;
  // ---------------------------------------------------------- scores
  auto word_of = [&](int32_t v) {
    const int q = v >> 6;
    const Philox4 pb = philox4x32_10((uint32_t)(q >> 2), (uint32_t)a.step, (uint32_t)row, kTagBlock, a.key0, a.key1);
    return (q & 3) == 0 ? pb.w[0] : (q & 3) == 1 ? pb.w[1] : (q & 3) == 2 ? pb.w[2] : pb.w[3];
  };
  bool take_member = false, sure_member = true;
  const int my_member = W * kWave - 1 - tid;  // the other end of the workgroup from the kept logits, which are usually few
  if (my_member < nmem) {  // (the largest logit of the bins after last_bin has the limit above it: not kept, nor is anything after it)
    const float xc = f.mem_x[my_member];
    uint32_t w_above = above_edge;
#pragma unroll 4
    for (int o = 0; o < nmem; ++o) w_above += f.mem_x[o] > xc ? f.mem_w[o] : 0u;
    const float m_above = (float)w_above / scale;
    sure_member = by_count ? w_above < (uint32_t)a.top_k : m_above < want - slack;
    take_member = by_count ? w_above < (uint32_t)a.top_k : m_above < want + slack;
  }
  Best st = no_best();
  // one loop for both: this thread's share of the kept logits, then its member of the edge bin
#pragma unroll 1
  for (int i = tid; i < nkept + W * kWave; i += W * kWave) {
    const bool member = i >= nkept;
    if (member ? !take_member : false) break;
    const uint32_t at = member ? f.mem_at[my_member] : f.kept[i];
    const int32_t v = list.index(at);
    score_drawn(a, row, v, member && !sure_member ? v | kInDoubt : v, list.logit(at), word_of(v), true, st);
    if (member) break;
  }
  publish_wave<W>(f.fres, st);
  __syncthreads();
  const Best all = merge_waves<W>(f.fres);
  tok = all.v;
  x_a = all.x;
  if (!(all.s - all.e > all.hi2)) {
    // the two best fp32 scores overlap within their margins: those that reach the winner's lower end, in double
    const double lower = (double)all.s - (double)all.e;
    Search<double> exact;
    exact.init();
#pragma unroll 1
    for (int i = tid; i < nkept + W * kWave; i += W * kWave) {
      const bool member = i >= nkept;
      if (member ? !take_member : false) break;
      const uint32_t at = member ? f.mem_at[my_member] : f.kept[i];
      const int32_t v = list.index(at);
      const BlockDraw<double> d = block_draw<double>(a, row, v >> 6);
      Search<double> one;
      one.init();
      score_index<double>(a, row, v, list.logit(at), d, lower, kNegInf, one);
      if (one.best.v >= 0 && member && !sure_member) one.best.v |= kInDoubt;
      exact.merge(one);
      if (member) break;
    }
    StepShared sh{};
    sh.res_s = f.res_s; sh.res_hi2 = f.res_hi2; sh.res_e = f.res_e; sh.res_v = f.res_v; sh.res_x = f.res_x;
    exact = combine_search<double, W>(sh, exact);
    tok = exact.best.v;
    x_a = exact.best.x;
  }
  return tok >= kInDoubt ? kUndecided : kDrawn;  // the winner may be one of the few logits whose sums are too close to p to tell
}

// The filtered draw of one row from its largest logits.  False (the same in every thread, nothing written): the
// row needs the general search.
template <int DT, bool Entropy, int W>
__device__ __forceinline__ bool filtered_row(const StepArgs& a, unsigned char* smem_raw, int row) {
  using Lim = CollectLimits<DT, W>;
  constexpr int kWords = Raw<DT>::kWords;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const FilterShared<DT, W> f = carve_filter<DT, W>(smem_raw);
  const void* rowp = (const char*)a.logits + (size_t)row * (size_t)a.row_stride * elem_bytes<DT>();

  // ------------------------------------------------------------ the row streams once, as in step_row
  const int ntiles = a.ntiles;
  const int my_tiles = wave < ntiles ? (ntiles - wave + W - 1) / W : 0;
  const uint32_t last_group = (uint32_t)(a.V - 1) & ~7u;
  const uint32_t lane_off = (uint32_t)lane * 8u;
  const uint32_t lane_bytes = lane_off * (uint32_t)elem_bytes<DT>();
  auto load_tile = [&](int t) {  // t is wave-uniform
    if (t != ntiles - 1) return load_raw_inner<DT>((const char*)rowp + (size_t)t * kTile * elem_bytes<DT>(), lane_bytes);
    const uint32_t e0 = (uint32_t)t * kTile + lane_off;  // last tile: may be ragged
    return load_raw<DT>(rowp, e0 < last_group ? e0 : last_group, (uint32_t)a.V);
  };
  Raw<DT> ring[kRing];
#pragma unroll
  for (int d = 0; d < kRing; ++d) {  // issued by every wave, whether it has that many tiles or not
    const uint32_t e0 = (uint32_t)(d * W + wave) * kTile + lane_off;
    ring[d] = load_raw<DT>(rowp, e0 < last_group ? e0 : last_group, (uint32_t)a.V);
  }
  for (int b = tid; b < kEdgeBins; b += W * kWave) f.bins[b] = 0;
  if (tid == 0) {
    *f.nkept = 0;
    *f.nmem = 0;
  }

  float nrk = kNoReference, lead = kNegInf, sum = 0.0f, sumw = 0.0f;  // the lane's softmax sum against its lazy reference
  float mx = kNegInf;
  uint32_t* const my_raw = f.raw + (size_t)wave * Lim::kRoom * kWords;
  uint16_t* const my_id = f.id + (size_t)wave * Lim::kRoom;
  int n = 0;                    // packs in this wave's list (wave-uniform)
  float thr = kMaskedBelow;     // every logit above it that the wave has seen is in the list
  float low = __builtin_huge_valf();  // the smallest pack maximum this lane has put there
  const Kept keep = packs_kept<DT, W>(a);
  bool flooded = false;         // a compaction found most of the list tied at its threshold
  int dry = 0;                  // passes since then that have left the list next to empty

  auto iteration = [&](auto steady, int d, int i) {
    constexpr bool Steady = decltype(steady)::value;
    const int t = i * W + wave;
    float x[8];
    unpack<DT>(ring[d], x);
    if (!Steady && (t + 1) * kTile > a.V) {  // ragged last tile: indices at or beyond V do not exist
      const int32_t e0 = t * kTile + (int32_t)lane_off;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (e0 + j >= a.V) x[j] = kNegInf;
    }
    const float gm = max8(x);
    mx = fmaxf(mx, gm);
    if (__builtin_amdgcn_ballot_w64(gm > lead) != 0) {  // rare after the first tile
      asm volatile("" ::: "memory");  // keep this rare path out of the straight-line code
      if (gm > lead) {  // move this lane's reference up to gm
        const float nrk_new = lane_reference(gm, a.k2);
        const float shift = nrk_new - nrk;
        const float g = __builtin_amdgcn_exp2f(shift);
        if (Entropy) sumw = g * fmaf(shift, sum, sumw);
        sum *= g;
        nrk = nrk_new;
        lead = gm + a.ref_lead;
      }
    }
    if constexpr (!Entropy) {
      float acc0 = __builtin_amdgcn_exp2f(fmaf(x[0], a.k2, nrk));
      float acc1 = __builtin_amdgcn_exp2f(fmaf(x[1], a.k2, nrk));
#pragma unroll
      for (int j = 2; j < 8; j += 2) {
        acc0 += __builtin_amdgcn_exp2f(fmaf(x[j], a.k2, nrk));
        acc1 += __builtin_amdgcn_exp2f(fmaf(x[j + 1], a.k2, nrk));
      }
      sum += acc0 + acc1;
    } else {  // t kept above -200: see step_row
      float acc0 = 0.0f, acc1 = 0.0f, w0 = 0.0f, w1 = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float t0 = fmaxf(fmaf(x[j], a.k2, nrk), -200.0f), t1 = fmaxf(fmaf(x[j + 1], a.k2, nrk), -200.0f);
        const float e0 = __builtin_amdgcn_exp2f(t0), e1 = __builtin_amdgcn_exp2f(t1);
        acc0 += e0;
        acc1 += e1;
        w0 = fmaf(e0, t0, w0);
        w1 = fmaf(e1, t1, w1);
      }
      sum += acc0 + acc1;
      sumw += w0 + w1;
    }
    const bool in = gm > thr;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
    if (mask != 0) {
      if (in) {
        const int at = n + rank_below(mask);
        pack_store<DT>(my_raw + at * kWords, ring[d]);
        my_id[at] = (uint16_t)(t * kWave + lane);
        low = fminf(low, gm);
      }
      n += (int)__builtin_popcountll(mask);
    }
    if (Steady)
      ring[d] = load_raw_inner<DT>((const char*)rowp + (size_t)(t + kRing * W) * kTile * elem_bytes<DT>(), lane_bytes);
    else if (i + kRing < my_tiles)
      ring[d] = load_tile(t + kRing * W);
    if ((d + 1) % Lim::kCheckTiles == 0 && n >= Lim::kCompactAt) {
      compact_list<DT, W>(my_raw, my_id, a.V, keep, n, thr);
      flooded = flooded || 4 * n < keep.most;
    }
  };
  const int steady_end = my_tiles > 2 * kRing ? ((my_tiles - kRing - 1) / kRing) * kRing : 0;
  int i0 = 0;
#pragma unroll 1
  for (; i0 < steady_end; i0 += kRing) {
#pragma unroll
    for (int d = 0; d < kRing; ++d) iteration(std::true_type{}, d, i0 + d);
    // Ties at the wave's largest logits: the kept set most likely reaches down to them, and they are not in the
    // list.  Given up early, such a row costs the general search and a few tiles (all logits equal, V = 152064, bf16 / fp32: B = 64: 23.6 / 35.1 us,
    // streamed to the end 26.2 / 38.6, the general search alone 22.9 / 31.0).
    if (flooded && (n == 0 || (8 * n < keep.most && ++dry == 2))) {
      thr = __builtin_huge_valf();  // nothing is above it: the row is handed on
      i0 = my_tiles;
      break;
    }
  }
#pragma unroll 1
  for (; i0 < my_tiles; i0 += kRing) {
#pragma unroll
    for (int d = 0; d < kRing; ++d)
      if (i0 + d < my_tiles) iteration(std::false_type{}, d, i0 + d);  // wave-uniform
  }
  // the wave's extremes, and its share of the softmax sums relative to its own maximum (see step_row)
  const float mw = wave_max(mx), loww = -wave_max(-low), leastw = -wave_max(-mx);
  {
    const float shift = -fmaf(mw, a.k2, nrk);
    const float g = __builtin_amdgcn_exp2f(shift);
    const float tot = wave_sum(sum > 0.0f ? sum * g : 0.0f);
    float totw = 0.0f;
    if constexpr (Entropy) totw = wave_sum(sum > 0.0f ? g * fmaf(shift, sum, sumw) : 0.0f);
    if (lane == 0) {
      f.least[wave] = leastw;
      f.m[wave] = mw;
      f.thr[wave] = thr;
      f.low[wave] = loww;
      f.sum[wave] = tot;
      f.sumw[wave] = totw;
    }
  }
  float z_prev = 0.0f, value = 0.0f;  // wanted at the very end: fetched now, off the critical path
  if (tid == 0) {
    z_prev = a.z[row];
    value = a.values[row];
  }
  __syncthreads();

  // ------------------------------------------------------------ m, T and S
  const RowSums sums = merge_sums<Entropy, true>(a, lane < W ? f.m[lane] : kNegInf, lane < W ? f.sum[lane] : 0.0f,
                                                 lane < W ? f.sumw[lane] : 0.0f);
  const float m = sums.m, S = sums.S;
  float bottom = row_max(lane < W ? f.thr[lane] : kNegInf);  // every logit above it is in a list
  if (!(bottom > kMaskedBelow)) {  // no list was ever compacted: the smallest pack maximum leaves a logit of every pack above
    const float lowest = -row_max(lane < W ? -f.low[lane] : kNegInf);
    const int32_t bits = __builtin_bit_cast(int32_t, lowest);
    bottom = lowest == 0.0f ? -1.401298464e-45f : __builtin_bit_cast(float, bits + (lowest > 0.0f ? -1 : 1));
  }
  int32_t tok = -1;
  float x_a = 0.0f;
  if (m > kNegInf) {
    if (!(bottom < m)) return false;  // ties at the row's largest logit fill a list
    PackList<DT, W> packs{f, n, a.V, {}, 0.0f};
    DrawResult res = draw_from_list<DT, W>(a, f, packs, row, m, S, bottom, tok, x_a);
    if (res == kReachesBelow) {
      // A flat row: the row is read once more and its single logits above a lower floor are collected, the smallest
      // of the lanes' largest logits.  (Of n lanes with V / n values each, about n ln n values of the row lie above the
      // smallest maximum: 3200 with 8 waves, 7100 with 16, whatever V is.)
      if (a.top_k == 0) {
        // How many logits it would take: those in the list, and for the missing mass more than as many of the threshold's
        // weight, since the weights fall on.  Where that is more than a draw has room for, the row is not read for
        // nothing (us, V = 152064, rows of normal logits: deviation 2, p = 0.9, B = 64: 84 -> 67; deviation 1, p = 0.7, B = 512: 187 -> 156).
        // With a factor of 1.25 fewer rows are spared (synthetic rows at temperature 1.3, p = 0.9, B = 64: 85 instead of 70); with
        // 2.5 rows that fit are sent away (temperature 1.3, p = 0.7, B = 512: 111 instead of 78).
        const float mine = wave_sum((float)packs.count());
        if (lane == 0) atomicAdd(f.nkept, (int)mine);
        __syncthreads();
        const float missing = a.top_p * S - packs.mass;
        if ((float)*f.nkept + 1.6f * missing / weight_below(bottom, m, a.k2) > (float)(kKeptCap2 + kEdgeMembers)) return false;
      }
      const float floor2 = -row_max(lane < W ? -f.least[lane] : kNegInf);
      if (!(floor2 < bottom && floor2 > kMaskedBelow)) return false;
      __syncthreads();  // the packs and the bins have been read by everyone
      for (int b = tid; b < kEdgeBins; b += W * kWave) f.bins[b] = 0;
      if (tid == 0) {
        *f.nkept = 0;
        *f.nmem = 0;
        *f.nover = 0;
      }
      LogitList<DT, W> logits{f, 0, 0.0f};
      constexpr int kDeep = 6;
#pragma unroll 1
      for (int i1 = 0; i1 < my_tiles; i1 += kDeep) {
        Raw<DT> raw[kDeep];
#pragma unroll
        for (int d = 0; d < kDeep; ++d)
          if (i1 + d < my_tiles) raw[d] = load_tile((i1 + d) * W + wave);
#pragma unroll
        for (int d = 0; d < kDeep; ++d) {
          if (i1 + d < my_tiles) {
            float x[8];
            const int32_t v0 = ((i1 + d) * W + wave) * kTile + (int32_t)lane_off;
            pack_unpack<DT>(raw[d], v0, a.V, x);
            if (__builtin_amdgcn_ballot_w64(max8(x) > floor2) != 0) {
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const uint64_t mask = __builtin_amdgcn_ballot_w64(x[j] > floor2);
                if (mask != 0) {
                  const int i = logits.n + rank_below(mask);
                  if (x[j] > floor2 && i < LogitList<DT, W>::kRoom) logits.put(wave, i, v0 + j, x[j]);
                  logits.n += (int)__builtin_popcountll(mask);
                }
              }
            }
          }
        }
      }
      __syncthreads();  // the counters are zero
      if (logits.n > LogitList<DT, W>::kRoom && lane == 0) *f.nover = 1;
      __syncthreads();
      if (*f.nover != 0) return false;
      res = draw_from_list<DT, W>(a, f, logits, row, m, S, floor2, tok, x_a);
    }
    if (res != kDrawn) return false;
  }

  if (wave != 0) return true;
  if (lane == 0) finish_row<DT, Entropy, true>(a, row, rowp, tok, x_a, m, S, sums.Sw, z_prev, value);
  return true;
}

template <int DT, bool Entropy, int W>
// Registers: 118 per lane (fp32 125) of at most 128, none in scratch: two workgroups of 8 waves on a compute unit or one of 16.  With the
// search's bounds read ahead, addresses kept over its rounds and six fp32 loads in flight it was 128 and 12 to 36 bytes of scratch
// (us, fp32 normal logits, top-p 0.9, V = 152064, B = 64: 114 -> 99; 256: 139 -> 125; synthetic rows at temperature 1.3, B = 64: 115 -> 105).
__global__ __launch_bounds__(W * kWave, 4) void espo_filtered_kernel(StepArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int row = (int)blockIdx.x;
  // top-k 1 needs the row maximum and its ties only, which the general search finds with less work per tile than the
  // lists take (us, V = 30000 bf16, B = 30: 8.8, through the lists 13.4; V = 60000, B = 300: 15.9 against 20.4).
  // A kept set of more logits than a draw from the lists has room for goes there at once, too (top-k 4000, B = 64, V = 152064:
  // 73 -> 38).
  if (a.top_k != 1 && a.top_k <= kKeptCap2 + kEdgeMembers && !row_is_done(a.alive, row)) {
    if (filtered_row<DT, Entropy, W>(a, smem_raw, row)) return;
    __syncthreads();  // the general search uses the same shared memory
  }
  step_row<DT, Entropy, true, true, W>(a, smem_raw);
}

template <int DT, int W>
const void* pick_kernel(bool sum, bool filter, bool entropy) {
  if constexpr (W >= 8) {
    if (filter) return entropy ? (const void*)espo_filtered_kernel<DT, true, W> : (const void*)espo_filtered_kernel<DT, false, W>;
  }
  if (!sum) return (const void*)espo_step_kernel<DT, false, false, W>;
  return entropy ? (const void*)espo_step_kernel<DT, true, true, W> : (const void*)espo_step_kernel<DT, false, true, W>;
}

template <int DT>
const void* pick_kernel(int waves, bool sum, bool filter, bool entropy) {
  return waves == 16 ? pick_kernel<DT, 16>(sum, filter, entropy) : waves == 8 ? pick_kernel<DT, 8>(sum, filter, entropy)
         : waves == 4 ? pick_kernel<DT, 4>(sum, filter, entropy) : nullptr;
}

}  // namespace

// This file is compiled once per logit type (the kernels take most of the build's time): with ESPO_STEP_F32
// defined for the fp32 kernels alone, without it for the bf16 kernels and everything below.
#ifdef ESPO_STEP_F32
const void* step_kernel_f32(int waves, bool sum, bool filter, bool entropy) { return pick_kernel<ESPO_F32>(waves, sum, filter, entropy); }
#else
const void* step_kernel_f32(int waves, bool sum, bool filter, bool entropy);
const void* step_kernel_bf16(int waves, bool sum, bool filter, bool entropy) { return pick_kernel<ESPO_BF16>(waves, sum, filter, entropy); }

namespace {

// Measures what score_margin assumes about the hardware transcendentals: the largest relative
// error of flog over every u(w) and over positive floats from 2^-26 to 64, and of fexp over
// [-40, 8], against the double-precision library functions.  out[0..2] hold the maxima as
// float bit patterns (non-negative floats order like unsigned integers).
__global__ void math_error_kernel(uint32_t* out) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;  // 2^23 threads
  float e_u = 0.0f, e_ln = 0.0f, e_exp = 0.0f;
  {
    const float u = (float)(2u * i + 1u) * (1.0f / 16777216.0f);  // every value u(w) takes
    const double ref = log((double)u);
    e_u = (float)fabs(((double)flog(u) - ref) / ref);
  }
  {
    // exponents -26..5 (32 of them), 2^18 mantissas each, spread over the 2^23 mantissa values
    const uint32_t bits = ((101u + (i >> 18)) << 23) | ((i & 0x3ffffu) * 32u + (i >> 18));
    const float x = __builtin_bit_cast(float, bits);
    const double ref = log((double)x);
    if (x != 1.0f) e_ln = (float)fabs(((double)flog(x) - ref) / ref);
  }
  {
    const float x = -40.0f + 48.0f * ((float)i * (1.0f / 8388608.0f));
    const double ref = exp((double)x);
    e_exp = (float)fabs(((double)fexp(x) - ref) / ref);
  }
  e_u = wave_max(e_u);
  e_ln = wave_max(e_ln);
  e_exp = wave_max(e_exp);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    atomicMax(out + 0, __builtin_bit_cast(uint32_t, e_u));
    atomicMax(out + 1, __builtin_bit_cast(uint32_t, e_ln));
    atomicMax(out + 2, __builtin_bit_cast(uint32_t, e_exp));
  }
}

}  // namespace

int launch_math_errors(float* out, hipStream_t stream) {
  hipLaunchKernelGGL(math_error_kernel, dim3(1u << 15), dim3(256), 0, stream, (uint32_t*)out);
  return hipGetLastError() == hipSuccess ? ESPO_OK : ESPO_EHIP;
}

// ---------------------------------------------------------------- launch configuration
// How a call is laid out on the GPU.  Unless it is split (own_split below), one workgroup streams a row: 8 waves, three
// workgroups to a compute unit, from 256 rows on; 16 waves for smaller batches, where a compute unit has one row at most and more
// waves stream it faster.  A workgroup of 16 waves has a compute unit to itself, and by the library's choice a launch never has more of
// them than there are compute units (255 whole rows, 64 in 4 chunks, 85 in 3, 128 in 2): from 257 on the others would be a second generation.
// us, 16 waves / 8, V = 152064 bf16, at temperature 0.6 | with the entropy at 1.0: 128 rows 16.1 / 16.9 | 19.9 / 22.6, 200: 16.5 / 17.0 | 20.5 / 23.2, 255: 18.1 / 17.7 |
// 21.1 / 23.5, 256: 19.2 / 17.5 | 20.9 / 23.2; 257: 28.1 / 23.2 | 32.4 / 28.2, 512: 36.3 / 29.3 | 38.3 / 34.0, 1024: 68.0 / 53.4 | 74.2 / 62.7; V = 32000: 200: 9.8 / 10.1 | 11.2 / 13.1,
// 300: 16.0 / 11.9 | 18.2 / 14.9; fp32 V = 100000: 128: 21.4 / 21.8, 255: 24.2 / 24.1, 257: 37.3 / 33.0.  With half of the rows done it is the live ones that
// count (300 rows: 15.9 / 23.5, 400: 28.0 / 23.9, 1024: 54.2 / 36.3), which the host does not know.  A filtered draw has the same two sizes,
// with more registers per wave: two workgroups of 8 waves to a compute unit.  The diagnostics
// entry point can force the waves per workgroup and a split of every row into `chunks` runs of
// tiles, each streamed by a workgroup of its own and combined by the one that finds all results there.  Where all compute
// units have rows enough, no split pays (B = 512, V = 152064 bf16, all rows live): 30.8 us unsplit, 45.7 us in 2 chunks
// of 16 waves, 36.0 us in 2 chunks of 8 waves, 38.9 us in 8 chunks of 4 waves (which keep some registers in scratch): every chunk pays for a search of its
// own and the row for two more trips through memory (a chunk's result written, then all of them read), which is
// more than the finer grain gains.  (Also measured and left out:
// 512 resident workgroups that claim rows from a counter in the workspace instead of one workgroup
// per row, meant to make rows that are done cost a claim instead of a workgroup: 512 device-scope
// atomics on one address take 50 ns each, and a launch of B = 1024 live rows went from 56 to 82 us.)

size_t step_workspace(int64_t B, int chunks) { return (size_t)B * (size_t)chunks * kMailRoom * sizeof(unsigned long long); }

constexpr int64_t kEightWavesFrom = 256;
constexpr int kComputeUnits = 256;

// How the library itself splits the rows of a plain draw, given a workspace: chunks per row and waves per chunk.
// A compute unit takes 4.9 to 8.3 us to stream a bf16 row of 152064 logits (its vector units are the limit: some 45
// operations per tile and wave, 8 of them exponentials) while, below 256 rows, others have none, or, just above,
// have one row where some have two.  A split costs two more trips through memory (results written, then the
// other chunks' results), 2 to 3 us, so it pays for long rows only; how long follows from how much a row's workgroup is held up by
// others that stream beside it, and for fp32 rows, whose sums hide behind the loads, from more rows on.  us per launch, one workgroup
// per row -> split, with log-probabilities / without (all rows live, synthetic language-model rows, temperature 0.6):
//   up to 64 rows, 4 chunks:
//     bf16 from 256 KB on: V = 131500: B = 1: 14.6 -> 11.4 / 11.2 -> 10.2, 64: 15.9 -> 13.3 / 14.0 -> 12.1; 152064: 64: 16.6 -> 13.7
//     f32, B <= 32, from 384 KB on: V = 100000: B = 1: 13.4 -> 12.9 / 12.3 -> 12.1, 32: 17.4 -> 14.4 / 16.4 -> 13.9; but V = 75000:
//       B = 4: 10.9 -> 11.5 / 9.9 -> 10.9, 17: 11.7 -> 12.5 / 10.7 -> 12.1, 32: 14.6 -> 13.8 / 14.1 -> 13.3
//     f32, B = 33 to 64, from 256 KB on: V = 66000: 33: 14.3 -> 13.4 / 13.9 -> 12.9, 64: 16.2 -> 13.7 / 15.8 -> 13.4
//     8 chunks up to 16 rows from 512 KB on (f32 V = 200000, B = 16: 31.8 -> 14.8, in 4 chunks 17.3).
//   65 to 128 rows, 2 chunks:
//     bf16 from 288 KB on: V = 151936: B = 65: 16.8 -> 15.5 / 13.8 -> 14.0, 128: 17.0 -> 15.9 / 14.9 -> 14.8; but V = 140000: 65:
//       16.3 -> 15.3 / 13.4 -> 14.2, 128: 16.4 -> 16.1 / 14.0 -> 15.2
//     f32 beyond 256 KB: V = 66000: 65: 16.3 -> 15.8 / 15.6 -> 15.5, 128: 17.8 -> 16.5 / 17.4 -> 16.2; but V = 65536 (eight tiles
//       for each of 16 waves): 65: 15.2 -> 15.5 / 14.6 -> 15.2
//   129 to 256 rows: f32 V = 150001: B = 200: 36.0 -> 35.0, 256: 36.6 -> 37.5; bf16: 18.9 -> 21.9.  Not split.
//   257 to 400 rows of f32 from 512 KB on, 3 chunks: V = 131072: B = 257: 41.8 -> 37.1, 350: 47.5 -> 45.1, 400: 49.3 -> 48.4;
//     V = 150001: 57.4 -> 44.8 at 300 (with half the rows done 53.2 -> 33.5).  V = 80000, B = 400: 33.7 -> 36.0: not split.
//   401 to 512 rows: V = 140000, B = 480: 54.9 -> 57.2 in 2 chunks, 59.0 in 3; 512: 56.1 -> 59.1, 63.8: not split.
//   513 to 640 rows of f32 from 512 KB on (more rows than two a compute unit), 2 chunks: V = 131500: B = 513: 66.5 -> 61.0,
//     570: 76.0 -> 68.4; V = 150001, B = 640: 88.4 -> 81.7.  bf16 V = 150001, B = 320: 30.3 -> 29.8, 512: 34.9 -> 40.8: not split.
// These lines were drawn with a search and a combine that took twice as long.  Into how many chunks a row goes was measured again
// since: as many as give every compute unit one of 8 waves, as long as that is 3, 4, 8 or 16 to a row, or two of them where
// that takes 5.  us per launch, chunks before -> now, with log-probabilities / without:
//   16 of 8 waves up to 16 rows: f32 V = 150001: B = 1: 10.7 -> 9.3 / 9.9 -> 8.9, 4: 10.5 -> 9.7 / 9.8 -> 9.1, 16: 10.3 -> 9.8 / 9.7 -> 9.3 (32 of 4
//     waves, with registers in scratch, B = 4: 10.1); bf16 V = 152064, B = 1: 10.8 -> 9.4 / 9.6 -> 8.9, 16: 11.4 -> 9.8 / 9.9 -> 9.1
//   8 of 8 waves from 17 to 32: f32 V = 150001, B = 32: 13.2 -> 11.4 / 12.6 -> 10.7; bf16 V = 201000, B = 32: 12.3 -> 10.7
//   33 to 64: 4 stay (B = 64: bf16 8 of 8 waves 11.6 -> 12.6, f32 14.6 -> 15.4).
//   3 from 65 to 85: f32, 2 chunks / 3: V = 66000, B = 65: 13.0 / 11.2, 85: 13.4 / 11.8; 100000, 85: 16.0 / 14.1; 200000, 85: 23.7 / 19.5; but 88 rows: 13.7 / 14.5, 16.1 / 17.8,
//     23.7 / 26.6.  bf16 V = 201000, B = 85, 16 waves: 15.7 -> 14.2.
//   5 of f32 from 86 to 102, 2 chunks / 5: B = 102: V = 66000 14.0 / 13.6, 100000 16.4 / 15.8, 150001 20.9 / 19.7, 390000 42.9 / 37.2, with the entropy at temperature 1.0
//     16.7 / 15.5, 19.4 / 17.9, 24.3 / 22.4, 45.9 / 40.0 (B = 94, V = 66000: 12.8 / 13.3, 16.0 / 15.1); but 104 rows: 13.8 / 14.9, 16.2 / 16.9, 20.7 / 22.6, 42.7 / 46.3.  bf16 V = 152064: 14.2 -> 14.6: not.
//   4 of f32 from 257 to 320 (five to a compute unit at most), from 576 KB on, 3 chunks / 4: B = 288: V = 147456 39.0 / 37.9, 150001 42.6 / 40.5, 200000 50.5 / 48.5, 390000 104.1 / 100.5;
//     320: 40.1 / 39.6, 44.1 / 42.6, 52.2 / 50.3, 108.1 / 103.9 (with half of the rows done 30.6 / 31.1, 32.7 / 33.4, 38.2 / 40.0, 78.4 / 72.3); but 336 rows: 40.9 / 43.1, 44.3 / 46.2, 53.0 / 55.7,
//     and below, B = 320: V = 131072 36.9 / 37.1, with the entropy 39.5 / 40.9, 140000 39.0 / 39.3, 41.7 / 42.5.
// A chunk of bf16 beyond 32 rows is streamed by 16 waves (at temperature 1.0, V = 152064, B = 64: 8 waves 7 % slower), every other by 8.
struct RowSplit {
  int chunks, waves;
};

RowSplit own_split(int dt, int64_t B, int64_t V) {
  const bool bf16 = dt == ESPO_BF16;
  const int64_t row_bytes = V * (bf16 ? 2 : 4);
  constexpr int64_t kKB = 1024, kVeryLong = 512 * kKB;
  constexpr RowSplit whole{1, 0};
  if (B <= 64) {
    if (row_bytes < (!bf16 && B <= 32 ? 384 * kKB : 256 * kKB)) return whole;
    if (B <= 32) return RowSplit{B <= 16 ? 16 : 8, 8};
    return RowSplit{4, bf16 ? 16 : 8};
  }
  if (B <= 128) {
    if (bf16 ? row_bytes < 288 * kKB : row_bytes <= 256 * kKB) return whole;
    if (B <= kComputeUnits / 3) return RowSplit{3, bf16 ? 16 : 8};
    if (!bf16 && B <= 2 * kComputeUnits / 5) return RowSplit{5, 8};
    return RowSplit{2, bf16 ? 16 : 8};
  }
  if (!bf16 && row_bytes >= kVeryLong) {
    if (B > 256 && B <= 400) return RowSplit{B <= 5 * kComputeUnits / 4 && row_bytes >= 576 * kKB ? 4 : 3, 8};
    if (B > 512 && B <= 640) return RowSplit{2, 8};
  }
  return whole;
}

StepPlan plan_step(int dt, int64_t B, int64_t V, bool filter, int waves, int chunks) {
  StepPlan p;
  const int ntiles = (int)((V + kTile - 1) / kTile);
  p.waves = waves > 0 ? waves : B >= kEightWavesFrom ? 8 : 16;
  int nch = filter || chunks <= 0 ? 1 : chunks;
  if (!filter && waves <= 0 && chunks <= 0) {
    const RowSplit own = own_split(dt, B, V);
    nch = own.chunks;
    if (nch > 1) p.waves = own.waves;
  }
  if (nch > ntiles) nch = ntiles;
  if (nch > kMaxChunks) nch = kMaxChunks;
  p.chunks = nch;
  const int ctiles = (ntiles + nch - 1) / nch;
  auto lds = [&](int w) {
    const size_t tables = step_lds_bytes(dt, ctiles, filter, w);
    if (!filter) return tables;
    const size_t lists = dt == ESPO_BF16 ? (w == 8 ? filter_lds_bytes<ESPO_BF16, 8>() : filter_lds_bytes<ESPO_BF16, 16>())
                                         : (w == 8 ? filter_lds_bytes<ESPO_F32, 8>() : filter_lds_bytes<ESPO_F32, 16>());
    return std::max(tables, lists);
  };
  p.lds = lds(p.waves);
  if (filter && waves <= 0 && p.lds > kMaxStepLds) p.lds = lds(p.waves = 8);  // the widest vocabularies: 8 waves need less
  p.workspace = nch > 1 ? step_workspace(B, nch) : 0;
  return p;
}

int launch_step(const void* logits, int dt, int64_t B, int64_t V, int64_t row_stride, float temperature,
                uint64_t seed, int32_t step, const float* values, const espo_params& p, float margin_scale,
                float* z, uint8_t* alive, int32_t* stop_step, int32_t* tokens, float* regret, float* logprob,
                float* entropy, void* workspace, const StepPlan& plan, hipStream_t stream) {
  StepArgs a;
  a.logits = logits;
  a.V = (int32_t)V;
  a.row_stride = row_stride;
  a.ntiles = (int)((V + kTile - 1) / kTile);
  a.nblocks = (int)((V + kDrawBlock - 1) / kDrawBlock);
  a.inv_tau = 1.0f / temperature;
  a.k2 = a.inv_tau * kLog2e;
  a.ref_lead = kRescaleAt / a.k2;
  a.margin_scale = margin_scale;
  a.key0 = (uint32_t)(seed & 0xffffffffu);
  a.key1 = (uint32_t)(seed >> 32);
  a.step = step;
  a.values = values;
  a.mu_g = p.mu_g;
  a.rsd = 1.0f / sqrtf(p.var_g + p.delta);
  a.clip_c = p.clip_c;
  a.alpha_s = p.alpha_s;
  a.oma = 1.0f - p.alpha_s;
  a.beta = p.beta;
  a.eps = p.eps;
  a.stop_enabled = p.stop_enabled;
  a.eos_id = p.eos_id;
  a.stop_mode = p.stop_mode;
  a.simulate = p.simulate;
  a.stop_threshold = p.stop_threshold;
  a.top_p = p.top_p;
  a.top_k = p.top_k;
  a.z = z;
  a.alive = alive;
  a.stop_step = stop_step;
  a.tokens = tokens;
  a.regret = regret;
  a.logprob = logprob;
  a.entropy = entropy;
  a.nch = plan.chunks;
  a.chunk_tiles = a.ntiles / plan.chunks;
  a.chunk_extra = a.ntiles % plan.chunks;
  a.mail = plan.chunks > 1 ? (unsigned long long*)workspace : nullptr;

  // the entropy output costs two more vector operations per logit: its own instantiation
  // and so does a filtered draw (more passes over the row)
  const bool filter = (p.top_p > 0.0f && p.top_p < 1.0f) || p.top_k > 0;
  if (plan.lds > kMaxStepLds) return ESPO_ERANGE;
  if (filter && (plan.waves < 8 || plan.chunks != 1)) return ESPO_EINVAL;
  if (plan.chunks > a.ntiles || plan.chunks > kMaxChunks || (int64_t)B * plan.chunks > 0x7fffffff) return ESPO_ERANGE;
  // and a step that is asked for neither log-probabilities nor either of these needs no softmax sum at all
  const bool sum = logprob != nullptr || entropy != nullptr || filter;
  const bool ent = entropy != nullptr;
  const void* const kernel = dt == ESPO_BF16 ? step_kernel_bf16(plan.waves, sum, filter, ent) : step_kernel_f32(plan.waves, sum, filter, ent);
  if (!kernel) return ESPO_EINVAL;
  if (plan.lds > 64 * 1024) {  // beyond the default limit the kernel has to be told (very large vocabularies)
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxStepLds) != hipSuccess)
      return ESPO_EHIP;
  }
  const dim3 grid((unsigned)B, (unsigned)plan.chunks), block((unsigned)(plan.waves * kWave));
  void* args[] = {&a};
  return hipLaunchKernel(kernel, grid, block, args, plan.lds, stream) == hipSuccess ? ESPO_OK : ESPO_EHIP;
}

#endif  // ESPO_STEP_F32

}  // namespace espo
