// The two backward products of the LM head (the head is linear, paper
// section 2, "Modeling"), both products for every sub-model in one grouped launch:
//   grad_W_i[chunk] = G_i^T h_i
//   grad_h_i       += G_i W_i[chunk]
// The bf16 and fp32 kernels read the slab G [t][v], h [t][d] and the head [v][d]
// as they are stored; the general bf16 kernel is an NT tile product whose
// transposed operands come from the transpose kernel below.
#include "mls_core.h"
#include "mls_device.h"
#include "mls_launch.h"

namespace mls {

namespace {

// One output element: fp32 C (overwritten or accumulated) or bf16 Cb (see GemmGroup).
__device__ __forceinline__ void store_out(const GemmGroup& g, int64_t idx, float v) {
  if (g.Cb) {
    if (g.Cpart) v += g.Cpart[idx];
    if (g.accumulate) v += __uint_as_float((uint32_t)g.Cb[idx] << 16);
    g.Cb[idx] = to_storage<Bf16>(v);
  } else {
    float* c = g.C + idx;
    *c = g.accumulate ? *c + v : v;
  }
}

// General bf16 path (operands of 4 GiB and more): pre-transposed operands.
__global__ __launch_bounds__(kThreads, 2) void gemm_nt_kernel(GemmArgs a) {
  using E = Bf16;
  using Mma = TileMma<E, kGemmBM, kGemmBN, 2, 2>;
  constexpr int FM = Mma::FM;
  constexpr int FN = Mma::FN;
  __shared__ __attribute__((aligned(16))) char smem[Mma::kSmemBytes];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % 2;
  const int wn = wave / 2;
  const int b = blockIdx.x;
  int gi = 0;
  for (int k = 1; k < a.ngroups; ++k)
    if (b >= a.g[k].tile_begin) gi = k;
  const GemmGroup& g = a.g[gi];
  const int local = b - g.tile_begin;
  const int tm = local % g.tiles_m;
  const int tn = local / g.tiles_m;
  const int64_t m0 = (int64_t)tm * kGemmBM;
  const int64_t n0 = (int64_t)tn * kGemmBN;

  Mma mma;
  mma.run(static_cast<const char*>(g.A), g.lda * E::kBytes, m0, g.rows,
          static_cast<const char*>(g.B), g.ldb * E::kBytes, n0, g.cols, g.K * E::kBytes, smem,
          tid);

#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const int64_t n = n0 + Mma::col_of(wn, fn, lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = m0 + Mma::row_of(wm, fm, r, lane);
        if (m < g.rows && n < g.cols) store_out(g, m * g.ldc + n, mma.acc[fm][fn][r]);
      }
    }
}

// fp32 path: the slab, the head chunk and h are read in their stored layouts.
// v_mfma_f32_32x32x2_f32 takes one fp32 of A and of B per lane, A[m = l % 32][k
// = l / 32], so a K-tile kept in LDS as [k][m] rows feeds it with plain 4-byte
// reads of consecutive lanes: an M-contiguous operand (the head chunk, h, and
// the slab for grad_W) is stored as it is loaded and only the K-contiguous one
// (the slab for grad_h) is transposed on its way into LDS, so neither transposed
// copies in memory nor a second slab layout are needed. Four waves: a 2 x 2
// grid of 32 x 32 tiles (KS = 1), or, for launches with too few tiles to fill
// the chip, one 32 x 32 tile whose K-tiles the waves take a quarter each of
// (KS = 4; the four sums are added in wave order, so results are reproducible).
// At T = 256, widths 128 / 256, V = 4,096 (30 blocks of 128 x 128 before) a
// chunk's products take 20 us instead of 90, and the transposed copies' 9 us go.
template <int BM, int BN, int BK>
struct F32Tile {
  static constexpr int LDA = BM + 2;  // row length: transposed 4-byte stores hit distinct banks
  static constexpr int LDB = BN + 2;
  float a[BK * LDA];
  float b[BK * LDB];
};

// 16-byte chunks of a K-tile [k0, k0 + BK) x [m0, m0 + ROWS) of an operand held
// by one thread: KC [m][k] (rows: m extent, K: k extent), MC [k][m] (rows: k
// extent, K: m extent). Chunks past either extent are 0.
template <int ROWS, int BK, bool MC>
struct F32Loader {
  static constexpr int kChunks = ROWS * BK / 4 / kThreads;
  static constexpr int kPer = MC ? ROWS / 4 : BK / 4;  // chunks per stored row
  float4 r[kChunks];
  __device__ __forceinline__ void load(const float* __restrict__ base, int64_t ld, int64_t m0,
                                       int64_t m_ext, int64_t k0, int64_t k_ext, int tid) {
#pragma unroll
    for (int j = 0; j < kChunks; ++j) {
      const int ci = tid + kThreads * j;
      const int64_t row = (MC ? k0 : m0) + ci / kPer;
      const int64_t col = (MC ? m0 : k0) + ci % kPer * 4;
      const bool in = row < (MC ? k_ext : m_ext) && col < (MC ? m_ext : k_ext);
      r[j] = in ? *reinterpret_cast<const float4*>(base + row * ld + col)
                : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  template <int LD>
  __device__ __forceinline__ void store(float* lds, int tid) const {
#pragma unroll
    for (int j = 0; j < kChunks; ++j) {
      const int ci = tid + kThreads * j;
      const int row = ci / kPer;
      const int col = ci % kPer * 4;
      const float v[4] = {r[j].x, r[j].y, r[j].z, r[j].w};
      if (MC) {
        *reinterpret_cast<float2*>(lds + row * LD + col) = make_float2(v[0], v[1]);
        *reinterpret_cast<float2*>(lds + row * LD + col + 2) = make_float2(v[2], v[3]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) lds[(col + q) * LD + row] = v[q];
      }
    }
  }
};

template <int BM, int BN, int KS, bool AMC>
__device__ __forceinline__ void f32_tile(const GemmGroup& g, int tm, int tn, char* smem, int tid) {
  constexpr int BK = 32 * KS;
  using Tile = F32Tile<BM, BN, BK>;
  Tile* stage = reinterpret_cast<Tile*>(smem);
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = KS > 1 ? 0 : wave & 1;
  const int wn = KS > 1 ? 0 : wave >> 1;
  const int kw = KS > 1 ? wave * 32 : 0;  // the wave's part of a K-tile
  const int64_t m0 = (int64_t)tm * BM;
  const int64_t n0 = (int64_t)tn * BN;
  const int64_t mext = g.ldc_rows, next = g.ldc, K = g.K;
  const float* A = static_cast<const float*>(g.A);
  const float* B = static_cast<const float*>(g.B);
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  F32Loader<BM, BK, AMC> la;
  F32Loader<BN, BK, true> lb;
  const int64_t nk = (K + BK - 1) / BK;
  la.load(A, g.lda, m0, mext, 0, K, tid);
  lb.load(B, g.ldb, n0, next, 0, K, tid);
  la.template store<Tile::LDA>(stage[0].a, tid);
  lb.template store<Tile::LDB>(stage[0].b, tid);
  __syncthreads();
  const int ml = wm * 32 + (lane & 31);
  const int nl = wn * 32 + (lane & 31);
  for (int64_t kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    if (more) {
      la.load(A, g.lda, m0, mext, (kt + 1) * BK, K, tid);
      lb.load(B, g.ldb, n0, next, (kt + 1) * BK, K, tid);
    }
    const Tile& t = stage[kt & 1];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int k = kw + 2 * s + (lane >> 5);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(t.a[k * Tile::LDA + ml], t.b[k * Tile::LDB + nl],
                                                 acc, 0, 0, 0);
    }
    if (more) {
      Tile& nx = stage[(kt + 1) & 1];
      la.template store<Tile::LDA>(nx.a, tid);
      lb.template store<Tile::LDB>(nx.b, tid);
    }
    __syncthreads();
  }
  if (KS > 1) {  // the waves' sums, through LDS
    float* part = reinterpret_cast<float*>(smem);
    if (wave > 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) part[((wave - 1) * 16 + r) * 64 + lane] = acc[r];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < KS - 1; ++w)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += part[(w * 16 + r) * 64 + lane];
  }
  const int64_t n = n0 + nl;
  if (n >= next) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t m = m0 + wm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (m < mext) store_out(g, m * g.ldc + n, acc[r]);
  }
}

template <int BM, int BN, int KS>
__global__ __launch_bounds__(kThreads) void gemm_f32_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[2 * sizeof(F32Tile<BM, BN, 32 * KS>)];
  const int b = blockIdx.x;
  int gi = 0;
  for (int k = 1; k < a.ngroups; ++k)
    if (b >= a.g[k].tile_begin) gi = k;
  const GemmGroup& g = a.g[gi];
  const int local = b - g.tile_begin;
  const int tn = local % g.tiles_n;
  const int tm = local / g.tiles_n;
  if (g.kind == 0)
    f32_tile<BM, BN, KS, false>(g, tm, tn, smem, threadIdx.x);
  else
    f32_tile<BM, BN, KS, true>(g, tm, tn, smem, threadIdx.x);
}

// bf16 path: 256 x 256 tiles, 8 waves (2 per SIMD) of 128 x 64, direct-to-LDS
// loads, five stages of 32-wide K (all 160 KB of LDS; see run_pipelined). The
// head chunk (grad_h) and the slab and h (grad_W) are read in their stored
// layouts through transposing LDS reads, so no operand is ever transposed in
// memory.
constexpr int kWideBM = 256;
constexpr int kWideBN = 256;
using WideGemmH = WideMma<kWideBM, kWideBN, 2, 4, 5, 64, kLayoutKC, kLayoutMC>;
using WideGemmW = WideMma<kWideBM, kWideBN, 2, 4, 5, 64, kLayoutMC, kLayoutMC>;
static_assert(kFusedBM % WideGemmH::BK == 0,
              "the K-tile holding a chunk's last row lies in a tile that the logit-gradient kernel writes");

// Loads and stores of one wave's part of an output tile through buffer
// descriptors over the tile's existing rows (rows past them read as 0 and are
// not written). Element (row, col) of the tile is at byte offset
// (row * ldc + col) * size; coff[fn] is the lane's part for column block fn,
// (its first row) * ldc + its column, or kNoCol for a column past the output
// (widths are multiples of 8), which the descriptor's range check then drops.
// 32-column blocks wholly past the output are skipped by a uniform branch
// (ok[fn]). INSIDE (all of the tile's rows
// exist): the (fm, r) part of the row goes into the scalar offset; otherwise
// every element gets its own vector offset, which the descriptor checks. Each
// kind of load is one loop with no branch inside, so a wave's loads are all in
// flight together.
// Cache policy of the fp32 output stores and of the reads of an fp32 output
// into the accumulators: non-temporal ("nt"), as each such element is touched
// once per launch. With the stores the headline step's GEMMs and the forward
// that follows them ran 0.01-0.02 ms faster each (7.76 -> 7.71 ms per step
// together with the forward's non-temporal slab stores); the reads took the
// GEMMs from 4.43-4.45 to 4.41-4.42 ms per step.
constexpr int kStoreNT = 2;
// In bytes (x 2 or x 4) kNoCol and any row offset added to it (256 rows of at
// most 2^20 columns) lie past a tile's rows (at most 2^30 bytes) and below 2^32.
constexpr uint32_t kNoCol = 0x20000000u;

template <class Mma, bool INSIDE>
struct TileIo {
  static constexpr int FM = Mma::FM;
  static constexpr int FN = Mma::FN;
  typedef f32x16_t Acc[FM][FN];

  __device__ __forceinline__ static int rrow(int fm, int r) { return fm * 32 + 8 * (r >> 2) + (r & 3); }
  __device__ __forceinline__ static uint32_t voff(const uint32_t* coff, int ldc, int fm, int fn,
                                                  int r, int size) {
    if (INSIDE) return coff[fn] * (uint32_t)size;
    return (coff[fn] + (uint32_t)(rrow(fm, r) * ldc)) * (uint32_t)size;
  }
  __device__ __forceinline__ static int soff(int ldc, int fm, int r, int size) {
    return INSIDE ? rrow(fm, r) * ldc * size : 0;
  }
  __device__ __forceinline__ static float ld32(__amdgpu_buffer_rsrc_t rs, const uint32_t* coff,
                                               int ldc, int fm, int fn, int r) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                         rs, voff(coff, ldc, fm, fn, r, 4), soff(ldc, fm, r, 4),
                                         kStoreNT));
  }
  __device__ __forceinline__ static float ld16(__amdgpu_buffer_rsrc_t rs, const uint32_t* coff,
                                               int ldc, int fm, int fn, int r) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(
                               rs, voff(coff, ldc, fm, fn, r, 2), soff(ldc, fm, r, 2), 0)
                           << 16);
  }

  // acc = Cpart (if part) + old output (if acc_old; bf16 when out16); blocks
  // past the output are left as they are (never stored)
  __device__ __forceinline__ static void init(Acc& acc, __amdgpu_buffer_rsrc_t rc,
                                              __amdgpu_buffer_rsrc_t rp, const uint32_t* coff,
                                              const bool* ok, int ldc, bool part, bool acc_old,
                                              bool out16) {
    if (part) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        if (ok[fn]) {
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fm][fn][r] = ld32(rp, coff, ldc, fm, fn, r);
        }
      if (acc_old) {  // and the old bf16 output: one column block at a time
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          if (!ok[fn]) continue;
          float old[FM][16];
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) old[fm][r] = ld16(rc, coff, ldc, fm, fn, r);
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fm][fn][r] += old[fm][r];
        }
      }
    } else if (out16) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        if (ok[fn]) {
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fm][fn][r] = ld16(rc, coff, ldc, fm, fn, r);
        }
    } else {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        if (ok[fn]) {
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fm][fn][r] = ld32(rc, coff, ldc, fm, fn, r);
        }
    }
  }

  __device__ __forceinline__ static void store(const Acc& acc, __amdgpu_buffer_rsrc_t rc,
                                               const uint32_t* coff, const bool* ok, int ldc,
                                               bool out16) {
    if (out16) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        if (!ok[fn]) continue;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            __builtin_amdgcn_raw_buffer_store_b16(to_storage<Bf16>(acc[fm][fn][r]), rc,
                                                  voff(coff, ldc, fm, fn, r, 2), soff(ldc, fm, r, 2), 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        if (!ok[fn]) continue;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[fm][fn][r]), rc,
                                                  voff(coff, ldc, fm, fn, r, 4), soff(ldc, fm, r, 4),
                                                  kStoreNT);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
};

// Tile (tm, tn) of group g, over its K part `part_k` (kind 0 groups in parts).
template <class Mma>
__device__ __forceinline__ void wide_tile(const GemmGroup& g, int tm, int tn, int part_k,
                                          int64_t mext, int64_t next, char* smem, int tid) {
  constexpr int FM = Mma::FM;
  constexpr int FN = Mma::FN;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % Mma::kWGM;
  const int wn = wave / Mma::kWGM;
  const int64_t m0 = (int64_t)tm * Mma::kBM;
  const int64_t n0 = (int64_t)tn * Mma::kBN;
  // Output through buffer descriptors over the tile's rows [m0, m0 + BM) that
  // exist (rows past mext fall outside them: their loads return 0 and their
  // stores are dropped), so each element's address is a 32-bit offset.
  const int64_t rows = mext - m0 < Mma::kBM ? mext - m0 : Mma::kBM;
  const bool out16 = g.Cb != nullptr;
  const int64_t k0 = part_k * g.ksplit;
  const int64_t K = g.splits > 1 && g.K - k0 > g.ksplit ? g.ksplit : g.K - k0;
  float* const C = g.C + part_k * g.csplit;
  const __amdgpu_buffer_rsrc_t rc =
      out16 ? uniform_rsrc(reinterpret_cast<const char*>(g.Cb + m0 * g.ldc), (int)(rows * g.ldc * 2))
            : uniform_rsrc(reinterpret_cast<const char*>(C + m0 * g.ldc), (int)(rows * g.ldc * 4));
  const bool part = out16 && g.Cpart;
  const __amdgpu_buffer_rsrc_t rp = uniform_rsrc(
      reinterpret_cast<const char*>(part ? g.Cpart + m0 * g.ldc : g.C), part ? (int)(rows * g.ldc * 4) : 0);
  const bool acc_old = g.accumulate != 0;
  const int ldc = (int)g.ldc;

  uint32_t coff[FN];
  bool ok[FN];
  const int wnu = __builtin_amdgcn_readfirstlane(wn);
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int col = (int)n0 + Mma::col_of(wn, fn, lane);
    coff[fn] = col < next ? (uint32_t)(Mma::row_of(wm, 0, 0, lane) * ldc + col) : kNoCol;
    ok[fn] = n0 + wnu * Mma::WTN + fn * 32 < next;  // the whole 32-column block (wave-uniform)
  }
  const bool inside = m0 + Mma::kBM <= mext;

  // A read-modify-write output (accumulate, or the fp32 partial sums of
  // earlier chunks) is read straight into the accumulators before the K loop,
  // so the product is added to it there and the epilogue only stores; the
  // reads' latency overlaps the first K-tile's loads.
  Mma mma;
  mma.run_pipelined(static_cast<const char*>(g.A) + k0 * 2, g.lda * 2, m0, g.rows,
               static_cast<const char*>(g.B) + k0 * g.ldb * 2, g.ldb * 2, n0, g.cols - k0, K * 2,
               smem, tid, [&]() {
                 if (!part && !acc_old)
                   mma.zero();
                 else if (inside)
                   TileIo<Mma, true>::init(mma.acc, rc, rp, coff, ok, ldc, part, acc_old, out16);
                 else
                   TileIo<Mma, false>::init(mma.acc, rc, rp, coff, ok, ldc, part, acc_old, out16);
               });
  if (inside)
    TileIo<Mma, true>::store(mma.acc, rc, coff, ok, ldc, out16);
  else
    TileIo<Mma, false>::store(mma.acc, rc, coff, ok, ldc, out16);
}

template <class MmaH, class MmaW>
__global__ __launch_bounds__(MmaH::NT, 1) void gemm_wide_kernel(GemmArgs a, int nb) {
  static_assert(MmaH::kSmemBytes == MmaW::kSmemBytes && MmaH::NT == MmaW::NT, "one footprint");
  __shared__ __attribute__((aligned(16))) char smem[MmaH::kSmemBytes];
  const int b = xcd_remap_phased(blockIdx.x, nb, a.phase_tiles);
  int gi = 0;
  for (int k = 1; k < a.ngroups; ++k)
    if (b >= a.g[k].tile_begin) gi = k;
  const GemmGroup& g = a.g[gi];
  int local = b - g.tile_begin;
  int part = 0;  // K part
  if (g.splits > 1) {
    part = local / (g.tiles_m * g.tiles_n);
    local -= part * g.tiles_m * g.tiles_n;
  }
  int tm, tn;
  if (g.group_m > 0) {
    tile_coords(local, g.tiles_m, g.tiles_n, g.group_m, tm, tn);
  } else {
    tn = local % g.tiles_n;
    tm = local / g.tiles_n;
  }
  // output extents: rows of C (grad_h: tokens; grad_W: chunk vocabulary rows) and
  // its columns (the width)
  const int64_t mext = g.ldc_rows;
  const int64_t next = g.ldc;
  if (g.kind == 0)
    wide_tile<MmaH>(g, tm, tn, part, mext, next, smem, threadIdx.x);
  else
    wide_tile<MmaW>(g, tm, tn, 0, mext, next, smem, threadIdx.x);
}

// Adds the K parts of grad_h (fixed order, so results are reproducible).
__global__ __launch_bounds__(kThreads) void split_sum_kernel(SplitSumArgs a) {
  const int i = blockIdx.y;
  if (!a.out[i]) return;
  const int64_t n = a.n[i];
  const float* part = a.part[i];
  for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * kThreads) {
    float v = part[k];
#pragma unroll 4
    for (int s = 1; s < a.splits; ++s) v += part[s * n + k];
    if (a.out16) {
      uint16_t* o = static_cast<uint16_t*>(a.out[i]) + k;
      if (a.accumulate) v += __uint_as_float((uint32_t)*o << 16);
      *o = to_storage<Bf16>(v);
    } else {
      float* o = static_cast<float*>(a.out[i]) + k;
      *o = a.accumulate ? *o + v : v;
    }
  }
}

__global__ __launch_bounds__(kThreads) void transpose_kernel(TransposeArgs a) {
  using S = uint16_t;
  const TransposeJob& j = a.j[blockIdx.z];
  const int64_t rb = (int64_t)blockIdx.x * 64;
  const int64_t cb = (int64_t)blockIdx.y * 64;
  if (rb >= j.out_rows || cb >= j.cols) return;
  __shared__ S tile[64][65];
  const int tx = threadIdx.x & 63;
  const int ty = threadIdx.x >> 6;
  const S* src = static_cast<const S*>(j.src);
  S* dst = static_cast<S*>(j.dst);
  for (int rr = ty; rr < 64; rr += 4) {
    const int64_t r = rb + rr;
    const int64_t c = cb + tx;
    S v = S(0);
    if (r < j.out_rows && c < j.cols && j.r0 + r < j.src_rows) v = src[(j.r0 + r) * j.ld_src + c];
    tile[rr][tx] = v;
  }
  __syncthreads();
  for (int cc = ty; cc < 64; cc += 4) {
    const int64_t c = cb + cc;
    const int64_t r = rb + tx;
    if (c < j.cols && r < j.out_rows) dst[c * j.ld_dst + r] = tile[tx][cc];
  }
}

}  // namespace

int gemm_tile_rows(bool wide) { return wide ? kWideBM : kGemmBM; }
int gemm_tile_cols(bool wide) { return wide ? kWideBN : kGemmBN; }
int gemm_wide_k_tile() { return WideGemmH::BK; }

hipError_t launch_gemm_wide(const GemmArgs& a, int total_tiles, hipStream_t stream) {
  if (total_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((gemm_wide_kernel<WideGemmH, WideGemmW>), dim3(total_tiles),
                     dim3(WideGemmH::NT), 0, stream, a, total_tiles);
  return hipGetLastError();
}

hipError_t launch_split_sum(const SplitSumArgs& a, hipStream_t stream) {
  int64_t n = 0;
  for (int i = 0; i < a.M; ++i) n = a.n[i] > n ? a.n[i] : n;
  const int64_t blocks = (n + kThreads - 1) / kThreads;
  const dim3 grid((unsigned)(blocks < 2048 ? blocks : 2048), (unsigned)a.M);
  hipLaunchKernelGGL(split_sum_kernel, grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmArgs& a, int tile, int total_tiles, hipStream_t stream) {
  if (total_tiles <= 0) return hipSuccess;
  if (tile == 64)
    hipLaunchKernelGGL((gemm_f32_kernel<64, 64, 1>), dim3(total_tiles), dim3(kThreads), 0, stream, a);
  else if (tile == 32)
    hipLaunchKernelGGL((gemm_f32_kernel<32, 32, 4>), dim3(total_tiles), dim3(kThreads), 0, stream, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_gemm_nt(const GemmArgs& a, int total_tiles, hipStream_t stream) {
  if (total_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(gemm_nt_kernel, dim3(total_tiles), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_transpose(const TransposeArgs& a, int64_t max_out_rows, int64_t max_cols,
                            hipStream_t stream) {
  if (a.njobs <= 0) return hipSuccess;
  dim3 grid((unsigned)((max_out_rows + 63) / 64), (unsigned)((max_cols + 63) / 64),
            (unsigned)a.njobs);
  hipLaunchKernelGGL(transpose_kernel, grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace mls
