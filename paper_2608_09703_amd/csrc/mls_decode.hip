// The head step of nested speculative decoding (paper section 2, paragraph
// "Speculative Decoding"; the measured setting of section 3, "Speculative
// Decoding Throughput": greedy or nucleus top-p 0.9 sampling at temperature
// 0.4, a smaller sub-model drafting gamma tokens and a larger one verifying).
//
// 1. head_logits_kernel: logits[t][v] = sum_k o[t][k] W[v][k] in fp32, on the
//    MFMA tile core (tiles from 64 vocabulary rows x 32 tokens to 192 x 128, by
//    the rule at head_tile); the fp32 tile is staged in LDS and leaves the block
//    as 16-byte stores of token-major rows.
//    Decode batches are small, so the [rows, V] logits are cheap next to the
//    head itself.
// 2. sample_kernel: one 1024-thread block per row. The row's sampling
//    distribution is softmax(l / temperature) restricted to the nucleus: the
//    most probable tokens (ties: lower index first) up to and including the
//    first one at which the kept mass reaches top_p. The nucleus threshold is
//    the largest exp-weight value theta whose "weight >= theta" mass still
//    reaches top_p of the total (found as described below); tokens tied at theta are kept in
//    index order as far as needed. A draw with uniform u returns the smallest
//    index whose cumulative kept weight in index order exceeds u times the
//    kept total.
// 3. verify_kernel: one block per sequence tests its gamma drafts: the draft
//    token x is kept when u * q(x) < p(x); at the first rejection the next
//    token is drawn from max(0, p - q); if all are kept, one more token is drawn
//    from the verifier's distribution after the drafts. Greedy mode compares
//    with the verifier's argmax (lowest index on ties).
//
// All reductions run in a fixed order, so results are bitwise reproducible.
#include <math.h>

#include "mls_core.h"
#include "mls_device.h"
#include "mls_launch.h"
#include "mls_wave.h"

namespace mls {

namespace {

// ---------------------------------------------------------------------------
// 1. head logits
// ---------------------------------------------------------------------------

template <class Mma, typename E>
__global__ __launch_bounds__(Mma::NT, Mma::kBM == 64 ? 1 : 2) void head_logits_kernel(HeadArgs a) {
  constexpr int BM = Mma::kBM;  // vocabulary rows
  constexpr int BN = Mma::kBN;  // tokens
  constexpr int FM = Mma::FM;
  constexpr int FN = Mma::FN;
  constexpr int NT = Mma::NT;
  constexpr int kChunks = BM / 4;          // 16-byte chunks (4 floats) per token row of the tile
  constexpr int kSw = kChunks & -kChunks;  // chunk swizzle span: XOR stays inside aligned groups
  // the fp32 tile leaves in one pass, or in one pass per wave column when it
  // is larger than the stage memory
  constexpr int kPasses = (BN * BM * 4 + Mma::kSmemBytes - 1) / Mma::kSmemBytes;
  constexpr int kTok = BN / kPasses;  // tokens per pass
  static_assert(kPasses == 1 || kPasses == Mma::kWGN, "one pass, or one per wave column");
  static_assert(kTok * BM * 4 <= Mma::kSmemBytes, "a pass fits in the stage memory");
  __shared__ __attribute__((aligned(16))) char smem[Mma::kSmemBytes];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % Mma::kWGM;
  const int wn = wave / Mma::kWGM;
  const int bl = xcd_remap(blockIdx.x, gridDim.x);
  int vt, tt;
  tile_coords(bl, a.n_vt, a.n_tt, a.group_v, vt, tt);
  const int64_t vbase = (int64_t)vt * BM;
  const int64_t tbase = (int64_t)tt * BN;
  const int64_t kb = a.d * E::kBytes;

  Mma mma;
  mma.run(static_cast<const char*>(a.W), kb, vbase, a.V, static_cast<const char*>(a.o), kb, tbase,
          a.T, kb, smem, tid);

  // stage: token row t of a pass holds kChunks chunks of 4 vocabulary entries,
  // chunk c at c ^ (t % kSw)
  float* st = reinterpret_cast<float*>(smem);
  const bool vec = (a.V & 3) == 0;
#pragma unroll
  for (int ps = 0; ps < kPasses; ++ps) {
    if (ps > 0) __syncthreads();  // every read of the previous pass is done
    if (kPasses == 1 || wn == ps) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const int t = Mma::col_of(wn, fn, lane) - ps * kTok;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) {
            const int v0 = Mma::row_of(wm, fm, rg * 4, lane);  // multiple of 4
            const float4 w = make_float4(mma.acc[fm][fn][rg * 4], mma.acc[fm][fn][rg * 4 + 1],
                                         mma.acc[fm][fn][rg * 4 + 2], mma.acc[fm][fn][rg * 4 + 3]);
            *reinterpret_cast<float4*>(st + t * BM + (((v0 >> 2) ^ (t & (kSw - 1))) << 2)) = w;
          }
      }
    }
    __syncthreads();
    for (int idx = tid; idx < kTok * kChunks; idx += NT) {
      const int t = idx / kChunks;
      const int c = idx % kChunks;
      const int64_t tg = tbase + ps * kTok + t;
      const int64_t v = vbase + 4 * c;
      if (tg >= a.T || v >= a.V) continue;
      const float4 w = *reinterpret_cast<const float4*>(st + t * BM + ((c ^ (t & (kSw - 1))) << 2));
      float* out = a.logits + tg * a.V + v;
      if (vec) {
        // whole lines, non-temporal (decode step 0.74 -> 0.72 ms: draft heads
        // 0.141 -> 0.126 ms, verifier head 3 % faster)
        store16_nt(out, make_uint4(__float_as_uint(w.x), __float_as_uint(w.y), __float_as_uint(w.z),
                                   __float_as_uint(w.w)));
      } else {
        const float x[4] = {w.x, w.y, w.z, w.w};
        for (int q = 0; q < 4 && v + q < a.V; ++q) out[q] = x[q];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// 2./3. per-row sampling distribution
// ---------------------------------------------------------------------------
//
// One 1024-thread block per row. Element i of a thread sits at vocabulary
// index v = 64 EPT wave + 64 i + lane: each wave owns a contiguous range of
// 64 EPT tokens, a slab i of it is one coalesced 256-byte load, and index
// order is (wave, slab, lane).
//
// Nucleus threshold. With `total` the sum of the row's exp weights and
// P = top_p * total, theta is the largest weight value whose mass
// S(theta) = sum(weight >= theta) still reaches P. S(c) >= P for some c puts
// theta at c or above, and every kept token among the weights >= c.
// 1. A close c for the price of a few LDS atomics: the largest weight of each
//    of a thread's kGroups runs of elements (4,096 in a row) enters a histogram
//    of mass over the weights' upper bits. From the top down, the first bin
//    edge c at which these maxima alone hold P has S(c) >= P, and where the
//    nucleus is small against the number of runs, c lies little below theta.
// 2. The weights >= c, a few per wave, move in index order to an LDS list; one
//    wave finds theta among them, resolves ties and draws.
// 3. Rows whose nucleus is too large for step 1 or the list take a radix
//    selection over all weights >= c0 = (1 - top_p) total / V (the weights
//    below c0 hold less than (1 - top_p) of the mass): a histogram of 64-bit
//    fixed-point masses (2^-44; sums do not depend on the order of the atomics)
//    over eight bins per octave names the bin that holds theta; if the weights
//    from that bin's lower edge up still overflow the list, three more levels
//    over the remaining bits give theta itself.
//
// The kernel lasts as long as one row's serial chain on its CU: load and
// maximum 4.7 us at V = 49,152, exp weights and sum 2.7 us (both bound by the
// CU), then barriers, scans of the thread's elements and the list wave. At 102
// such rows (nucleus 0.9 at temperature 0.4) a launch took 24 us with a list of
// every weight >= c0 (some 2,000 of them), three bound raises on it and a
// four-way threshold search, and 22 us with the radix selection for every row;
// it takes 15.5 us (one row: 20 -> 12 us; the records of 714 verifier rows:
// 73 -> 51 us).

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kMaxEPT = 64;
constexpr int kRunMax = 16;              // candidate entries per lane of the list wave
constexpr int kMaxCand = 64 * kRunMax;   // candidates one wave holds
constexpr int kSmallCand = 4 * 64;       // lists searched with 4 entries per lane
constexpr int kGroups = 4;               // runs of a thread's elements with a maximum each
constexpr int kRegion = 256;             // list entries per wave before they are joined
constexpr int kMaxShift = 21;            // bins of the maxima: four per octave,
constexpr int kMaxBins = 64;             // 16 octaves (the last bin: everything below)
constexpr int kTopShift = 20;            // radix selection: the bits from here up,
constexpr int kBins = 512;               // weights down to 2^-64 (c0 >= 2^-40)
constexpr uint32_t kOne = 0x3f800000u;   // weight 1, the largest

// LDS slot of list entry j: one gap after every 16 entries, so that the lanes
// of the list wave, each reading a run of consecutive entries, hit different
// banks.
__device__ __forceinline__ int cand_slot(int j) { return j + (j >> 4); }
constexpr int kCandSlots = kMaxCand + kMaxCand / 16;

struct RowShared {
  unsigned long long hist[kBins]; // mass per bin, 2^-44
  unsigned maxhist[kMaxBins];     // mass of the runs' maxima per bin, 2^-15
  float bw[kRowWaves * kRegion];  // one list region per wave, in index order
  int bi[kRowWaves * kRegion];
  float cw[kCandSlots];           // candidate list, index order
  int ci[kCandSlots];             // their vocabulary indices
  float seg[kMaxEPT * kRowWaves]; // per (wave, slab) sums for whole-row index-order scans
  float scr[64];                  // list wave: the threshold bin's entries
  float rmax[kRowWaves];
  float rsum[kRowWaves];
  float red[kRowWaves];
  int ired[kRowWaves];
  int wcnt[kRowWaves];            // per-wave list counts
  float bcast[4];
  int ibcast[4];
};

// A row's exp weights are formed in several places (the distribution's
// parameters, then draws and probabilities recomputed from the logits); they
// must agree bitwise, so the product and the difference are rounded on their
// own and never contracted into an FMA.
__device__ __forceinline__ float scaled_logit(float l, float inv_temp) {
#pragma clang fp contract(off)
  return l * inv_temp;
}
__device__ __forceinline__ float weight_of(float scaled, float m) {
#pragma clang fp contract(off)
  return fast_exp2((scaled - m) * kLog2e);
}

// Block-wide reductions in a fixed order (every thread gets the result).
__device__ __forceinline__ float block_sum(float v, RowShared& sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh.red[w] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kRowWaves; ++i) s += sh.red[i];
  __syncthreads();
  return s;
}
__device__ __forceinline__ int block_count(int v, RowShared& sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh.ired[w] = v;
  __syncthreads();
  int s = 0;
#pragma unroll
  for (int i = 0; i < kRowWaves; ++i) s += sh.ired[i];
  __syncthreads();
  return s;
}
// The waves' results, one per lane of each 16-lane row, combined in a fixed
// order. Used with an LDS array of its own each time, so one barrier suffices.
static_assert(kRowWaves == 16, "one DPP row holds the waves' results");
__device__ __forceinline__ float block_max_once(float v, float* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return wave_max(red[threadIdx.x & 15]);
}
__device__ __forceinline__ float block_sum_once(float v, float* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return row16_sum(red[threadIdx.x & 15]);
}

// Argmax with the lowest index on ties.
__device__ __forceinline__ void block_argmax(float& val, int& idx, RowShared& sh) {
  wave_argmax(val, idx);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sh.red[w] = val;
    sh.ired[w] = idx;
  }
  __syncthreads();
  val = sh.red[0];
  idx = sh.ired[0];
#pragma unroll
  for (int i = 1; i < kRowWaves; ++i)
    if (argmax_better(sh.red[i], sh.ired[i], val, idx)) {
      val = sh.red[i];
      idx = sh.ired[i];
    }
  __syncthreads();
}

// Vocabulary index of the thread's element i.
template <int EPT>
__device__ __forceinline__ int elem_v(int i) {
  return (int)(threadIdx.x >> 6) * (64 * EPT) + 64 * i + (int)(threadIdx.x & 63);
}

// Number of the thread's elements inside the row: element i exists iff
// i < elems_in_row (a compare with a constant, so no per-element index needs
// to stay live).
template <int EPT>
__device__ __forceinline__ int elems_in_row(int V) {
  const int v0 = elem_v<EPT>(0);
  return V > v0 ? (V - v0 + 63) >> 6 : 0;
}

// The thread's EPT logits of a row, x[i] = row[elem_v(i)], as buffer loads
// over the row's V * 4 bytes: one per-lane offset, the slab as a scalar
// offset, and indices past the row read 0 from the hardware range check, so
// every load is unconditional and all of them are in flight together.
// Callers mask v >= V themselves.
template <int EPT>
__device__ __forceinline__ void load_row(const float* row, int V, float* x) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc((void*)row, (short)0, V * 4, 0x00020000);
  const int base = elem_v<EPT>(0) * 4;
#pragma unroll
  for (int i = 0; i < EPT; ++i)
    x[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, base, 256 * i, 0));
}

__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Smallest index whose cumulative weight in index order exceeds `target`,
// over the whole row; weight(i) gives the thread's i-th weight. Returns -1 if
// the total does not exceed it.
template <int EPT, class Wt>
__device__ __forceinline__ int index_order_draw(Wt weight, float target, RowShared& sh) {
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  // per (slab, wave) sums
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const float s = wave_sum(weight(i));
    if (lane == 0) sh.seg[wave * EPT + i] = s;
  }
  __syncthreads();
  // wave 0 scans the 16 EPT segment sums in index order (each lane owns a run of them)
  if (wave == 0) {
    constexpr int NSEG = EPT * kRowWaves;
    constexpr int PER = NSEG / 64;
    float run = 0.f;
#pragma unroll
    for (int q = 0; q < PER; ++q) run += sh.seg[lane * PER + q];
    const float incl = wave_incl_scan(run);
    float before = incl - run;
    int found = -1;
    float found_before = 0.f;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int sidx = lane * PER + q;
      const float s = sh.seg[sidx];
      if (found < 0 && s > 0.f && before + s > target) {
        found = sidx;
        found_before = before;
      }
      before += s;
    }
    // the first lane (in index order) that found its segment wins
    const unsigned long long m = __ballot(found >= 0);
    if (lane == 0) sh.ibcast[0] = -1;
    if (m && lane == __builtin_ctzll(m)) {
      sh.ibcast[0] = found;
      sh.bcast[0] = found_before;
    }
  }
  __syncthreads();
  const int sidx = sh.ibcast[0];
  const float base = sh.bcast[0];
  __syncthreads();
  if (sidx < 0) return -1;
  const int swave = sidx / EPT;
  const int slab = sidx % EPT;
  // inside the segment: the owning wave scans its 64 lanes
  if (wave == swave) {
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < EPT; ++i)
      if (i == slab) x = weight(i);
    const float incl = wave_incl_scan(x);
    const unsigned long long m = __ballot(x > 0.f && base + incl > target);
    int pick;
    if (m) {
      pick = __builtin_ctzll(m);
    } else {  // rounding: take the last positive weight of the segment
      const unsigned long long pos = __ballot(x > 0.f);
      pick = pos ? 63 - __builtin_clzll(pos) : 0;
    }
    if (lane == 0) sh.ibcast[1] = swave * (64 * EPT) + slab * 64 + pick;
  }
  __syncthreads();
  const int v = sh.ibcast[1];
  __syncthreads();
  return v;
}

__device__ __forceinline__ bool kept_w(float e, int v, const RowDist& d) {
  return e > d.theta || (e == d.theta && e > 0.f && v <= d.tie_cut);
}

// Keeps the compiler from carrying compares of the thread's elements (a mask of
// two scalar registers each) from one pass over them to the next: it would
// spill them.
template <int EPT>
__device__ __forceinline__ void pass_fence(float* w) {
#pragma unroll
  for (int i = 0; i < EPT; ++i) asm volatile("" : "+v"(w[i]));
}

// Writes the row elements of bit patterns >= lo (lo > 0, no negative elements)
// to the LDS list in index order, at cand_slot(position), and returns how many
// there are. Index order is (wave, slab, lane): each wave writes its elements to
// its own region, then moves them behind those of the waves before it. Where
// the total exceeds kMaxCand or a wave's number its region, nothing is moved
// and a number above kMaxCand is returned.
template <int EPT>
__device__ __forceinline__ int compact_row(float* w, uint32_t lo, RowShared& sh) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  pass_fence<EPT>(w);
  int pos0 = 0;  // wave-uniform
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const bool f = __float_as_uint(w[i]) >= lo;
    const unsigned long long b = __ballot(f);
    if (b == 0) continue;  // most slabs hold no entry
    if (f) {
      const int pos = pos0 + lanes_below(b);
      if (pos < kRegion) {
        sh.bw[wave * kRegion + pos] = w[i];
        sh.bi[wave * kRegion + pos] = elem_v<EPT>(i);
      }
    }
    pos0 += __builtin_popcountll(b);
  }
  if (lane == 0) sh.wcnt[wave] = pos0;
  __syncthreads();
  const int cnt = sh.wcnt[lane & (kRowWaves - 1)];  // the 16 counts, in every lane row
  const int incl = row16_incl_scan(cnt);
  const int total = lane_read(incl, kRowWaves - 1);
  if (total > kMaxCand || __ballot(cnt > kRegion) != 0) return kMaxCand + 1;
  const int at = wave == 0 ? 0 : lane_read(incl, wave - 1);
  for (int j = lane; j < pos0; j += 64) {
    sh.cw[cand_slot(at + j)] = sh.bw[wave * kRegion + j];
    sh.ci[cand_slot(at + j)] = sh.bi[wave * kRegion + j];
  }
  __syncthreads();
  return total;
}

// ---- list wave (wave 0, all lanes active): lane l holds entries [l RUN, (l + 1) RUN)

template <int RUN>
__device__ __forceinline__ void load_run(const RowShared& sh, int n, float (&w)[RUN]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < RUN; ++q) {
    const int j = lane * RUN + q;
    w[q] = j < n ? sh.cw[cand_slot(j)] : 0.f;
  }
}

template <int RUN>
__device__ __forceinline__ int run_index(const RowShared& sh, int q) {
  return sh.ci[cand_slot((int)(threadIdx.x & 63) * RUN + q)];
}

// Position in the list of the first entry (index order) whose cumulative
// weight exceeds `target`; the last positive entry when rounding leaves the
// target at or above the sum; 0 when every weight is 0, which the callers rule
// out (a row that keeps no token has no list to draw from).
template <int RUN>
__device__ __forceinline__ int run_draw(const float (&kw)[RUN], float target) {
  const int lane = threadIdx.x & 63;
  float run = 0.f;
#pragma unroll
  for (int q = 0; q < RUN; ++q) run += kw[q];
  const float incl = wave_incl_scan(run);
  const unsigned long long hit = __ballot(run > 0.f && incl > target);
  const unsigned long long pos = __ballot(run > 0.f);
  if (!pos) return 0;
  const int L = hit ? __builtin_ctzll(hit) : 63 - __builtin_clzll(pos);
  int j = 0;
  if (lane == L) {
    float acc = incl - run;
    int first = -1, last = 0;
#pragma unroll
    for (int q = 0; q < RUN; ++q) {
      if (kw[q] > 0.f) {
        acc += kw[q];
        last = q;
        if (first < 0 && acc > target) first = q;
      }
    }
    j = lane * RUN + (first >= 0 ? first : last);
  }
  return __builtin_amdgcn_readlane(j, L);
}

// Theta from the list (list wave; n entries): the largest value whose mass
// reaches P, which lies in [lo, hi) (bit patterns). Four-way steps (three
// probes, three independent reductions; the probed sets are nested and summed
// in the same order, so the computed masses are ordered like the exact ones)
// until at most 64 entries lie in the bracket. The mass at or above hi is then
// fixed, those entries move to one per lane (through `scr`), and each lane
// takes the mass at or above its own entry: the largest entry whose mass
// reaches P is theta, with no further search.
template <int RUN>
__device__ __forceinline__ float list_theta(const float (&w)[RUN], uint32_t lo, uint32_t hi,
                                            float P, float* scr) {
  const int lane = threadIdx.x & 63;
  int n2;
  for (;;) {
    int inside = 0;
#pragma unroll
    for (int q = 0; q < RUN; ++q) {
      const uint32_t b = __float_as_uint(w[q]);
      inside += b >= lo && b < hi ? 1 : 0;
    }
    n2 = wave_sum(inside);
    if (RUN == 1 || n2 <= 64 || hi - lo <= 3) break;
    const uint32_t st = (hi - lo) >> 2;
    const uint32_t m1 = lo + st, m2 = m1 + st, m3 = m2 + st;
    float p1 = 0.f, p2 = 0.f, p3 = 0.f;
#pragma unroll
    for (int q = 0; q < RUN; ++q) {
      const uint32_t b = __float_as_uint(w[q]);
      p1 += b >= m1 ? w[q] : 0.f;
      p2 += b >= m2 ? w[q] : 0.f;
      p3 += b >= m3 ? w[q] : 0.f;
    }
    const int g1 = __builtin_amdgcn_readfirstlane(wave_sum(p1) >= P ? 1 : 0);
    const int g2 = __builtin_amdgcn_readfirstlane(wave_sum(p2) >= P ? 1 : 0);
    const int g3 = __builtin_amdgcn_readfirstlane(wave_sum(p3) >= P ? 1 : 0);
    if (g3) {
      lo = m3;
    } else if (g2) {
      lo = m2;
      hi = m3;
    } else if (g1) {
      lo = m1;
      hi = m2;
    } else {
      hi = m1;
    }
  }
  if (n2 == 0) return __uint_as_float(lo);  // rounding: the entries at or above hi are kept
  if (n2 > 64) {  // three or fewer bit patterns with more than 64 entries (ties): one probe each
    for (uint32_t b = hi - 1; b > lo; --b) {
      float p = 0.f;
#pragma unroll
      for (int q = 0; q < RUN; ++q) p += __float_as_uint(w[q]) >= b ? w[q] : 0.f;
      if (__builtin_amdgcn_readfirstlane(wave_sum(p) >= P ? 1 : 0)) return __uint_as_float(b);
    }
    return __uint_as_float(lo);
  }
  float base = 0.f;
  int cnt = 0;
#pragma unroll
  for (int q = 0; q < RUN; ++q) {
    const uint32_t b = __float_as_uint(w[q]);
    base += b >= hi ? w[q] : 0.f;
    cnt += (b >= lo && b < hi) ? 1 : 0;
  }
  const float B = wave_sum(base);
  int pos = wave_incl_scan(cnt) - cnt;
#pragma unroll
  for (int q = 0; q < RUN; ++q) {
    const uint32_t b = __float_as_uint(w[q]);
    if (b >= lo && b < hi) scr[pos++] = w[q];
  }
  const float x = lane < n2 ? scr[lane] : 0.f;
  float part[4] = {B, 0.f, 0.f, 0.f};  // (entries n2 .. 63 are 0 and add nothing)
  for (int k = 0; k < n2; k += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float y = lane_read(x, k + q);
      part[q] += y >= x ? y : 0.f;
    }
  }
  const float mass = (part[0] + part[1]) + (part[2] + part[3]);
  // (the smallest entry's mass reaches P up to rounding; it is taken if none does)
  const float smallest = -wave_max(lane < n2 ? -x : -INFINITY);
  const float best = wave_max(lane < n2 && mass >= P ? x : 0.f);
  return best > 0.f ? best : smallest;
}

// Completes a row's distribution from its list (list wave; theta in [lo, hi)): theta, the
// tie cut and the kept mass. `kw` receives the kept weights of the lane's run.
template <int RUN>
__device__ __forceinline__ void run_dist(RowShared& sh, int n, uint32_t lo, uint32_t hi, float P,
                                         int V, RowDist& d, float (&kw)[RUN]) {
  const int lane = threadIdx.x & 63;
  float w[RUN];
  load_run<RUN>(sh, n, w);
  const float th = list_theta<RUN>(w, lo, hi, P, sh.scr);
  d.theta = th;
  float above = 0.f;
  int ties = 0;
#pragma unroll
  for (int q = 0; q < RUN; ++q) {
    above += w[q] > th ? w[q] : 0.f;
    ties += w[q] == th ? 1 : 0;  // th > 0, so padding zeros never tie
  }
  const float mass_above = wave_sum(above);
  const int n_tie = wave_sum(ties);
  int k = n_tie;
  if (n_tie > 1) {
    k = (int)ceilf((P - mass_above) / th);
    k = k < 1 ? 1 : (k > n_tie ? n_tie : k);
  }
  d.tie_cut = V;
  if (k < n_tie) {  // vocabulary index of the k-th tied entry (the list is in index order)
    const int incl = wave_incl_scan(ties);
    const int L = __builtin_ctzll(__ballot(incl >= k));
    int cut = 0;
    if (lane == L) {
      int seen = incl - ties;
#pragma unroll
      for (int q = 0; q < RUN; ++q)
        if (w[q] == th && ++seen == k) cut = run_index<RUN>(sh, q);
    }
    d.tie_cut = __builtin_amdgcn_readlane(cut, L);
  }
  float kp = 0.f;
#pragma unroll
  for (int q = 0; q < RUN; ++q) {
    kw[q] = w[q] > th || (w[q] == th && run_index<RUN>(sh, q) <= d.tie_cut) ? w[q] : 0.f;
    kp += kw[q];
  }
  d.kept = wave_sum(kp);
}

__device__ __forceinline__ unsigned long long fixed_mass(float e) {
  return (unsigned long long)(e * 17592186044416.f);  // 2^44; a row's sum stays below 2^60
}

// The first bin, from bin 0 on, at which `above` plus the masses up to it reach
// P (2^-44 units); `above` becomes the mass before that bin. -1 if none does.
// Every wave runs it on its own.
template <int NB>
__device__ __forceinline__ int pick_bin(const unsigned long long* hist, double P, double& above) {
  constexpr int PER = NB / 64;
  const int lane = threadIdx.x & 63;
  double h[PER];
  double run = 0.0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    h[q] = (double)hist[lane * PER + q];
    run += h[q];
  }
  const double incl = wave_incl_scan(run);
  const unsigned long long hit = __ballot(above + incl >= P);
  if (!hit) return -1;
  const int L = __builtin_ctzll(hit);
  double before = above + incl - run;
  int bin = PER - 1;
  bool found = false;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (!found) {
      if (q == PER - 1 || before + h[q] >= P) {
        bin = q;
        found = true;
      } else {
        before += h[q];
      }
    }
  }
  above = lane_read(before, L);
  return L * PER + __builtin_amdgcn_readlane(bin, L);
}

// Loads a row and computes its sampling distribution. `e` receives the
// thread's exp weights exp(l / T - max) (0 beyond V). With a nucleus that fits
// the list, the weights of bit patterns >= `lo` are left there and their number
// is returned: then only m and total are set in d, and the list wave completes
// it (run_dist; theta lies in [lo, hi)). Otherwise the whole distribution is in
// d for every thread and -1 is returned.
template <int EPT>
__device__ __forceinline__ int row_dist(const float* row, int V, float inv_temp, float top_p,
                                        float* e, RowShared& sh, RowDist& d, uint32_t& lo,
                                        uint32_t& hi, float& P) {
  constexpr int kRun = EPT / kGroups;
  load_row<EPT>(row, V, e);
  if (threadIdx.x < kMaxBins) sh.maxhist[threadIdx.x] = 0;
  const int nv = elems_in_row<EPT>(V);
  float mx[kGroups];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    mx[g] = -INFINITY;
#pragma unroll
    for (int i = g * kRun; i < (g + 1) * kRun; ++i) {
      e[i] = i < nv ? scaled_logit(e[i], inv_temp) : -INFINITY;
      mx[g] = fmaxf(mx[g], e[i]);
    }
  }
  d.m = block_max_once(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])), sh.rmax);
  const float m = d.m == -INFINITY ? 0.f : d.m;  // a row of -inf: every weight 0
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    e[i] = weight_of(e[i], m);
    s += e[i];
  }
  const bool nucleus = top_p < 1.f;
  if (nucleus) {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      const float w = weight_of(mx[g], m);  // the run's largest weight
      const int bin = (int)(kOne >> kMaxShift) - (int)(__float_as_uint(w) >> kMaxShift);
      if (bin >= 0 && bin < kMaxBins - 1) atomicAdd(&sh.maxhist[bin], (unsigned)(w * 32768.f));
    }
  }
  d.total = block_sum_once(s, sh.rsum);
  d.theta = 0.f;
  d.tie_cut = V;
  d.kept = d.total;
  if (!nucleus) return -1;
  P = top_p * d.total;
  lo = 0;
  hi = kOne + 1;  // nothing is above 1
  {
    // rounded down, the masses never overstate the maxima's
    const unsigned incl = wave_incl_scan((int)sh.maxhist[threadIdx.x & 63]);
    const unsigned long long hit = __ballot((float)incl >= P * 32768.f * 1.000001f);
    if (hit && d.total > 0.f) {
      const uint32_t c = ((kOne >> kMaxShift) - (uint32_t)__builtin_ctzll(hit)) << kMaxShift;
      const int n = compact_row<EPT>(e, c, sh);
      if (n <= kMaxCand) {
        lo = c;
        return n;
      }
    }
  }
  // radix selection over all weights >= c0 (at most 1)
  __syncthreads();
  for (int b = threadIdx.x; b < kBins; b += kRowThreads) sh.hist[b] = 0;
  __syncthreads();
  const float c0 = (1.f - top_p) * d.total / (float)V;
  pass_fence<EPT>(e);
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const bool in = e[i] >= c0 && e[i] > 0.f;
    if (__ballot(in) == 0) continue;
    if (in) {
      const int bin = (int)(kOne >> kTopShift) - (int)(__float_as_uint(e[i]) >> kTopShift);
      atomicAdd(&sh.hist[bin < kBins ? bin : kBins - 1], fixed_mass(e[i]));
    }
  }
  __syncthreads();
  const double Pd = (double)P * 17592186044416.0;
  double above = 0.0;
  const int bin = pick_bin<kBins>(sh.hist, Pd, above);
  if (bin >= 0 && bin < kBins - 1 && d.total > 0.f) {
    lo = ((kOne >> kTopShift) - (uint32_t)bin) << kTopShift;
    if (bin > 0) hi = lo + (1u << kTopShift);
    const int n = compact_row<EPT>(e, lo, sh);
    if (n <= kMaxCand) return n;
    // the nucleus overflows the list: the bin's remaining bits, 8 + 8 + 4 at a time
#pragma unroll 1
    for (int shift = kTopShift; shift > 0;) {
      const int bits = shift >= 8 ? 8 : shift;
      const int sh2 = shift - bits;
      __syncthreads();  // the previous level's histogram has been read
      if (threadIdx.x < 256) sh.hist[threadIdx.x] = 0;
      __syncthreads();
      pass_fence<EPT>(e);
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const uint32_t b = __float_as_uint(e[i]);
        const bool in = b >= lo && b < hi;
        if (__ballot(in) == 0) continue;
        if (in) atomicAdd(&sh.hist[((1 << bits) - 1) - (int)((b - lo) >> sh2)], fixed_mass(e[i]));
      }
      __syncthreads();
      const int k = pick_bin<256>(sh.hist, Pd, above);
      // (the masses of the level add up to the bin's, so some digit reaches P)
      lo += (uint32_t)(((1 << bits) - 1) - (k < 0 ? (1 << bits) - 1 : k)) << sh2;
      hi = lo + (1u << sh2);
      shift = sh2;
    }
  } else {
    // no weight (or NaN), or rounding left the histogram's mass below P (top_p
    // within an ulp of 1): the largest bit pattern b with sum(e >= b) >= P;
    // sum(e >= 0) = total does
    while (hi - lo > 1) {
      const uint32_t mid = lo + (hi - lo) / 2;
      float part = 0.f;
#pragma unroll
      for (int i = 0; i < EPT; ++i) part += __float_as_uint(e[i]) >= mid ? e[i] : 0.f;
      if (block_sum(part, sh) >= P)
        lo = mid;
      else
        hi = mid;
    }
  }
  d.theta = __uint_as_float(lo);
  float above_f = 0.f;
  int ties = 0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    above_f += e[i] > d.theta ? e[i] : 0.f;
    ties += (e[i] == d.theta && e[i] > 0.f) ? 1 : 0;
  }
  const float mass_above = block_sum(above_f, sh);
  const int n_tie = block_count(ties, sh);
  int k = n_tie;
  if (n_tie > 1 && d.theta > 0.f) {
    k = (int)ceilf((P - mass_above) / d.theta);
    k = k < 1 ? 1 : (k > n_tie ? n_tie : k);
  }
  // index of the k-th tied token (counts are exact in fp32 up to 2^24)
  const float th = d.theta;
  d.tie_cut = k >= n_tie ? V
                         : index_order_draw<EPT>(
                               [&](int i) { return (e[i] == th && e[i] > 0.f) ? 1.f : 0.f; },
                               (float)k - 0.5f, sh);
  float kp = 0.f;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int v = elem_v<EPT>(i);
    kp += kept_w(e[i], v, d) ? e[i] : 0.f;
  }
  d.kept = block_sum(kp, sh);
  return -1;
}

// Whole-row draw from a row's distribution with uniform u (weights in `e`,
// parameters in d); `e` is overwritten with the kept weights.
template <int EPT>
__device__ __forceinline__ int row_draw(float* e, const RowDist& d, float u, RowShared& sh) {
  int last = -1;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int v = elem_v<EPT>(i);
    e[i] = kept_w(e[i], v, d) ? e[i] : 0.f;
    if (e[i] > 0.f) last = v;
  }
  int v = index_order_draw<EPT>([&](int i) { return e[i]; }, u * d.kept, sh);
  if (v < 0) {  // rounding pushed the target past the total: the last kept index
    float lv = (float)last;
    int li = last;
    block_argmax(lv, li, sh);
    v = li;
  }
  return v;
}

template <int EPT>
__device__ __forceinline__ int row_argmax(const float* row, int V, RowShared& sh) {
  float x[EPT];
  load_row<EPT>(row, V, x);
  const int nv = elems_in_row<EPT>(V);
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    if (i < nv && x[i] > best) {  // the index increases with i: strict > keeps the lowest
      best = x[i];
      bi = i;
    }
  }
  bi = bi == 0x7fffffff ? bi : elem_v<EPT>(0) + 64 * bi;
  block_argmax(best, bi, sh);
  return bi == 0x7fffffff ? -1 : bi;  // no logit above -inf: no token
}

// The distribution from the list (list wave), then (with u >= 0) a draw;
// returns the drawn token (or -1 without a draw).
template <int RUN>
__device__ __forceinline__ int list_finish_run(RowShared& sh, int n, uint32_t lo, uint32_t hi,
                                               float P, int V, float u, RowDist& d) {
  float kw[RUN];
  run_dist<RUN>(sh, n, lo, hi, P, V, d, kw);
  if (u < 0.f) return -1;
  const int j = run_draw<RUN>(kw, u * d.kept);
  return sh.ci[cand_slot(j)];
}
// One, 4 or 16 entries per lane.
__device__ __forceinline__ int list_finish(RowShared& sh, int n, uint32_t lo, uint32_t hi, float P,
                                           int V, float u, RowDist& d) {
  return n <= 64           ? list_finish_run<1>(sh, n, lo, hi, P, V, u, d)
         : n <= kSmallCand ? list_finish_run<4>(sh, n, lo, hi, P, V, u, d)
                           : list_finish_run<kRunMax>(sh, n, lo, hi, P, V, u, d);
}

template <int EPT>
__global__ __launch_bounds__(kRowThreads) void sample_kernel(SampleArgs a) {
  __shared__ RowShared sh;
  const int64_t r = blockIdx.x;
  const float* row = a.logits + r * a.V;
  int tok;
  if (a.greedy) {
    tok = row_argmax<EPT>(row, (int)a.V, sh);
  } else {
    float e[EPT];
    RowDist d;
    uint32_t lo = 0, hi = 0;
    float P = 0.f;
    const int n = row_dist<EPT>(row, (int)a.V, a.inv_temp, a.top_p, e, sh, d, lo, hi, P);
    if (n >= 0) {
      if (threadIdx.x >= 64) return;
      tok = list_finish(sh, n, lo, hi, P, (int)a.V, a.u[r], d);
    } else {
      tok = row_draw<EPT>(e, d, a.u[r], sh);
    }
    if (threadIdx.x == 0 && a.params) a.params[r] = d;
  }
  if (threadIdx.x == 0) a.tokens[r] = tok;
}

// Every row's sampling-distribution parameters (rows of several arrays: the
// draft rows, then the verifier rows).
template <int EPT>
__global__ __launch_bounds__(kRowThreads) void row_params_kernel(RowParamArgs a) {
  __shared__ RowShared sh;
  const int64_t r = blockIdx.x;
  const float* row = r < a.rows0 ? a.logits0 + r * a.V : a.logits1 + (r - a.rows0) * a.V;
  float e[EPT];
  RowDist d;
  uint32_t lo = 0, hi = 0;
  float P = 0.f;
  const int n = row_dist<EPT>(row, (int)a.V, a.inv_temp, a.top_p, e, sh, d, lo, hi, P);
  if (n >= 0) {
    if (threadIdx.x >= 64) return;
    list_finish(sh, n, lo, hi, P, (int)a.V, -1.f, d);
  }
  if (threadIdx.x == 0) a.params[r] = d;
}

// Exp weight of logit x under a row's parameters, with row_dist's arithmetic.
__device__ __forceinline__ float exp_weight(float logit, float inv_temp, const RowDist& d) {
  return weight_of(scaled_logit(logit, inv_temp), d.m);
}

// Kept, normalised probability of token v (v < V).
__device__ __forceinline__ float prob_at(const float* row, int v, float inv_temp,
                                         const RowDist& d) {
  const float e = exp_weight(row[v], inv_temp, d);
  return kept_w(e, v, d) ? e / d.kept : 0.f;
}

// Whole-row draw with uniform u from a row's distribution, weights recomputed
// from the logits.
template <int EPT>
__device__ __forceinline__ int draw_kept(const float* row, int V, float it, const RowDist& d,
                                         float u, RowShared& sh) {
  auto w = [&](int i) {
    const int v = elem_v<EPT>(i);
    if (v >= V) return 0.f;
    const float e = exp_weight(row[v], it, d);
    return kept_w(e, v, d) ? e : 0.f;
  };
  int v = index_order_draw<EPT>(w, u * d.kept, sh);
  if (v < 0) {
    int last = -1;
    for (int i = 0; i < EPT; ++i)
      if (w(i) > 0.f) last = elem_v<EPT>(i);
    float lv = (float)last;
    block_argmax(lv, last, sh);
    v = last;
  }
  return v;
}

// Compacts the kept tokens of row p (weights recomputed from the logits) into
// the LDS list; returns their number.
template <int EPT>
__device__ __forceinline__ int compact_kept(const float* prow, int V, float it, const RowDist& dp,
                                            RowShared& sh) {
  float w[EPT];
  load_row<EPT>(prow, V, w);
  const int nv = elems_in_row<EPT>(V);
  const int v0 = elem_v<EPT>(0);
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const float e = exp_weight(w[i], it, dp);
    w[i] = i < nv && kept_w(e, v0 + 64 * i, dp) ? e : 0.f;
  }
  return compact_row<EPT>(w, 1u, sh);  // every positive weight
}

// List wave: a draw from p's kept list (n entries) with uniform u; with a
// draft row qrow (parameters dq), from max(0, p - q), or p itself if that has
// no mass. -1 where p keeps no token (a row with a +inf logit, or of NaN or -inf
// only), as the sampler gives for such a row.
template <int RUN>
__device__ __forceinline__ int list_residual_draw(const RowShared& sh, int n, const RowDist& dp,
                                                  const float* qrow, const RowDist& dq, float it,
                                                  float u) {
  if (n == 0) return -1;
  float w[RUN];
  load_run<RUN>(sh, n, w);
  if (qrow) {
    float r[RUN];
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < RUN; ++q) {
      r[q] = 0.f;
      if (w[q] > 0.f)
        r[q] = fmaxf(w[q] / dp.kept - prob_at(qrow, run_index<RUN>(sh, q), it, dq), 0.f);
      s += r[q];
    }
    const float tot = wave_sum(s);
    if (tot > 0.f) return sh.ci[cand_slot(run_draw<RUN>(r, u * tot))];
  }
  return sh.ci[cand_slot(run_draw<RUN>(w, u * dp.kept))];
}

// Verification: one block per sequence. Rows' parameters come from
// row_params_kernel; weights are recomputed from the logits as needed (the
// rows stay in L2). The draw after a rejection (or after the last draft) runs
// over the verifier row's kept tokens, which hold all of max(0, p - q). Bound by
// latency: 32 us per launch (102 sequences of 6 drafts at V = 49,152) with the
// drafts tested one after the other and two passes over the row for the kept
// tokens, 20 us with the tests side by side and one pass.
template <int EPT, bool GREEDY>
__global__ __launch_bounds__(kRowThreads) void verify_kernel(VerifyArgs a) {
  __shared__ RowShared sh;
  const int64_t b = blockIdx.x;
  const int V = (int)a.V;
  const int G = a.gamma;
  const float it = a.inv_temp;
  int k = 0;
  int next = 0;
  if (GREEDY) {
#pragma nounroll
    for (; k < G; ++k) {
      next = row_argmax<EPT>(a.target_logits + (b * (G + 1) + k) * a.V, V, sh);
      if (next != a.draft_tokens[(int64_t)k * a.batch + b]) break;
    }
  } else {
    // The acceptance tests do not depend on each other: one lane per draft, so
    // that a sequence waits for one chain of loads (token, logits) rather than
    // one per kept draft. Every wave does it for itself.
#pragma nounroll
    for (int k0 = 0; k0 < G; k0 += 64) {
      const int kl = k0 + (int)(threadIdx.x & 63);
      bool rejected = false;
      if (kl < G) {
        const int64_t at = (int64_t)kl * a.batch + b;
        const int x = a.draft_tokens[at];
        const RowDist dq = a.dparams[at];
        const RowDist dp = a.tparams[b * (G + 1) + kl];
        const bool in = x >= 0 && x < V;
        const float qx = in ? prob_at(a.draft_logits + at * a.V, x, it, dq) : 0.f;
        const float px = in ? prob_at(a.target_logits + (b * (G + 1) + kl) * a.V, x, it, dp) : 0.f;
        rejected = !(a.u_accept[at] * qx < px);
      }
      const unsigned long long m = __ballot(rejected);
      k = k0 + (m ? __builtin_ctzll(m) : 64);
      if (m) break;
    }
    k = k < G ? k : G;
  }
  if (!GREEDY && k < G) {
    const float* trow = a.target_logits + (b * (G + 1) + k) * a.V;
    const float* drow = a.draft_logits + ((int64_t)k * a.batch + b) * a.V;
    const RowDist dq = a.dparams[(int64_t)k * a.batch + b];
    const RowDist dp = a.tparams[b * (G + 1) + k];
    // rejected: draw from max(0, p - q)
    const int n = compact_kept<EPT>(trow, V, it, dp, sh);
    if (n <= kMaxCand) {
      if (threadIdx.x >= 64) return;
      next = n <= kSmallCand ? list_residual_draw<4>(sh, n, dp, drow, dq, it, a.u_sample[b])
                             : list_residual_draw<kRunMax>(sh, n, dp, drow, dq, it, a.u_sample[b]);
    } else {
      auto res = [&](int i) {
        const int v = elem_v<EPT>(i);
        if (v >= V) return 0.f;
        return fmaxf(prob_at(trow, v, it, dp) - prob_at(drow, v, it, dq), 0.f);
      };
      float rs = 0.f;
#pragma unroll 4
      for (int i = 0; i < EPT; ++i) rs += res(i);
      const float tot = block_sum(rs, sh);
      if (tot > 0.f) {
        int v = index_order_draw<EPT>(res, a.u_sample[b] * tot, sh);
        if (v < 0) {
          int last = -1;
          for (int i = 0; i < EPT; ++i)
            if (res(i) > 0.f) last = elem_v<EPT>(i);
          float lv = (float)last;
          block_argmax(lv, last, sh);
          v = last;
        }
        next = v;
      } else {
        // no residual mass: the rejected token was impossible under both
        // distributions and they coincide, so the draw is from the verifier's
        next = draw_kept<EPT>(trow, V, it, dp, a.u_sample[b], sh);
      }
    }
  }
  if (k == G) {  // every draft kept: one more token from the verifier
    const float* trow = a.target_logits + (b * (G + 1) + G) * a.V;
    if (GREEDY) {
      next = row_argmax<EPT>(trow, V, sh);
    } else {
      const RowDist dp = a.tparams[b * (G + 1) + G];
      const int n = compact_kept<EPT>(trow, V, it, dp, sh);
      if (n <= kMaxCand) {
        if (threadIdx.x >= 64) return;
        next = n <= kSmallCand ? list_residual_draw<4>(sh, n, dp, nullptr, dp, it, a.u_sample[b])
                           : list_residual_draw<kRunMax>(sh, n, dp, nullptr, dp, it,
                                                         a.u_sample[b]);
      } else {
        next = draw_kept<EPT>(trow, V, it, dp, a.u_sample[b], sh);
      }
    }
  }
  if (threadIdx.x == 0) {
    a.n_accepted[b] = k;
    a.next_token[b] = next;
  }
}

using HeadWide = WideMma<128, 128, 2, 2, 2>;
// 192 vocabulary rows: 80 KB of stages, two blocks fill a CU's LDS
using HeadWide192 = WideMma<192, 128, 2, 2, 2>;
// few rows: a quarter (half) of the token columns, so that three (two) K-tiles
// of the head are in flight ahead: 48 KB of stages, three blocks per CU
using HeadFew = WideMma<64, 32, 2, 1, 4>;
using HeadSome = WideMma<64, 64, 2, 2, 3>;
// 128 columns, vocabularies too small for a 128-row block per CU
using HeadShort = WideMma<64, 128, 2, 2, 3>;
// widths that are not multiples of the 64-wide K-tile
using HeadShortTail = WideMma<64, 128, 2, 2, 3, 128, kLayoutKC, kLayoutKC, true>;
using HeadFewTail = WideMma<64, 32, 2, 1, 4, 128, kLayoutKC, kLayoutKC, true>;
using HeadSomeTail = WideMma<64, 64, 2, 2, 3, 128, kLayoutKC, kLayoutKC, true>;
using HeadWideTail = WideMma<128, 128, 2, 2, 2, 128, kLayoutKC, kLayoutKC, true>;
using HeadWide192Tail = WideMma<192, 128, 2, 2, 2, 128, kLayoutKC, kLayoutKC, true>;
using HeadGenF32 = TileMma<F32, 128, 128, 2, 2>;

}  // namespace

// Tile of the head product (vocabulary rows x token columns).
// - At most 64 rows of hidden states: bound by the head's bytes and by how many
//   of them are in flight, so 64 vocabulary rows and 32 or 64 columns, with
//   three or two K-tiles ahead in each of three blocks per CU. One row at
//   width 4,352, V = 49,152: 84 -> 74 us (5.8 TB/s); 16 rows at width 2,048, V =
//   16,000: 31 -> 16 us; 64 rows at width 4,352: 94 -> 91 us.
// - 128 columns otherwise. Where 128-row tiles would not give every CU a block,
//   64 rows: 102 rows at width 2,048, V = 16,000 (125 blocks) 36 -> 22 us, V =
//   32,000 (250 blocks) 41.6 -> 39.7; at 313 blocks 27.9 -> 30.0, so not there.
// - From four such token tiles on (the verifier's rows) 192 vocabulary rows: at
//   102 x 7 rows and V = 49,152 that makes 1,536 blocks, three full rounds of two
//   blocks per CU, where 128-row tiles make 2,304 (four and a half).
void head_tile(bool wide, int64_t T, int64_t V, int* rows, int* cols) {
  *cols = !wide || T > 64 ? 128 : T > 32 ? 64 : 32;
  const int64_t blocks = ((T + 127) / 128) * ((V + 127) / 128);  // of 128 x 128
  *rows = !wide ? 128 : T <= 64 || blocks < 256 ? 64 : T > 3 * 128 ? 192 : 128;
}
int row_elems_per_thread(int64_t V) {
  for (int e : {16, 32, 48, 64})
    if (V <= (int64_t)e * kRowThreads) return e;
  return 0;
}

template <class Mma, typename E>
static void launch_head_t(const HeadArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((head_logits_kernel<Mma, E>), dim3((unsigned)a.n_tt * (unsigned)a.n_vt),
                     dim3(Mma::NT), 0, stream, a);
}

hipError_t launch_head_logits(const HeadArgs& a, bool f32, hipStream_t stream) {
  int rows, cols;
  head_tile(!f32, a.T, a.V, &rows, &cols);
  if (a.n_vt != (int)((a.V + rows - 1) / rows) || a.n_tt != (int)((a.T + cols - 1) / cols))
    return hipErrorInvalidValue;
  const bool tail = a.d % 64 != 0;
  if (f32)
    launch_head_t<HeadGenF32, F32>(a, stream);
  else if (cols == 32)
    tail ? launch_head_t<HeadFewTail, Bf16>(a, stream) : launch_head_t<HeadFew, Bf16>(a, stream);
  else if (cols == 64)
    tail ? launch_head_t<HeadSomeTail, Bf16>(a, stream) : launch_head_t<HeadSome, Bf16>(a, stream);
  else if (rows == 64)
    tail ? launch_head_t<HeadShortTail, Bf16>(a, stream) : launch_head_t<HeadShort, Bf16>(a, stream);
  else if (rows == 192)
    tail ? launch_head_t<HeadWide192Tail, Bf16>(a, stream) : launch_head_t<HeadWide192, Bf16>(a, stream);
  else
    tail ? launch_head_t<HeadWideTail, Bf16>(a, stream) : launch_head_t<HeadWide, Bf16>(a, stream);
  return hipGetLastError();
}

hipError_t launch_sample(const SampleArgs& a, int ept, hipStream_t stream) {
  const dim3 grid((unsigned)a.rows);
  switch (ept) {
    case 16: hipLaunchKernelGGL(sample_kernel<16>, grid, dim3(kRowThreads), 0, stream, a); break;
    case 32: hipLaunchKernelGGL(sample_kernel<32>, grid, dim3(kRowThreads), 0, stream, a); break;
    case 48: hipLaunchKernelGGL(sample_kernel<48>, grid, dim3(kRowThreads), 0, stream, a); break;
    case 64: hipLaunchKernelGGL(sample_kernel<64>, grid, dim3(kRowThreads), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_row_params(const RowParamArgs& a, int ept, hipStream_t stream) {
  const dim3 grid((unsigned)(a.rows0 + a.rows1));
  switch (ept) {
    case 16: hipLaunchKernelGGL(row_params_kernel<16>, grid, dim3(kRowThreads), 0, stream, a); break;
    case 32: hipLaunchKernelGGL(row_params_kernel<32>, grid, dim3(kRowThreads), 0, stream, a); break;
    case 48: hipLaunchKernelGGL(row_params_kernel<48>, grid, dim3(kRowThreads), 0, stream, a); break;
    case 64: hipLaunchKernelGGL(row_params_kernel<64>, grid, dim3(kRowThreads), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int EPT>
static void launch_verify_ept(const VerifyArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)a.batch);
  if (a.greedy)
    hipLaunchKernelGGL((verify_kernel<EPT, true>), grid, dim3(kRowThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((verify_kernel<EPT, false>), grid, dim3(kRowThreads), 0, stream, a);
}

hipError_t launch_verify(const VerifyArgs& a, int ept, hipStream_t stream) {
  switch (ept) {
    case 16: launch_verify_ept<16>(a, stream); break;
    case 32: launch_verify_ept<32>(a, stream); break;
    case 48: launch_verify_ept<48>(a, stream); break;
    case 64: launch_verify_ept<64>(a, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mls
