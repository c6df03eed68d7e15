// Wide-tile bf16 MFMA main loop with direct global->LDS loads (gfx950).
//
// Same product as TileMma (C[m][n] = sum_k A[m][k] B[n][k], both operands
// row-major with K contiguous, output layout of v_mfma_f32_32x32x16_bf16) for
// tiles of up to 256 x 256 and any number of waves. Differences:
//  - operands are moved from global memory straight into LDS with
//    buffer_load_dwordx4 ... lds (16 bytes per lane, no register staging);
//    each lane fetches the global chunk that belongs in its LDS slot under the
//    XOR swizzle of lds_off(), so fragment reads stay conflict-free. A buffer
//    descriptor covers the block's operand panel, so per-lane offsets are
//    32-bit, fixed for the whole K loop (the K position is a scalar offset),
//    and rows past the end of the operand read as zero;
//  - STAGES K-tiles of RB bytes (64 or 32 bf16) are in flight; a K-tile is consumed after an
//    explicit vmcnt wait and a plain s_barrier (no memory fence, so younger
//    loads stay in flight across the barrier);
//  - K of an MC operand is a multiple of a K-tile; K of KC operands too unless
//    KTAIL is set, which takes any multiple of 8: the last K-tile's lanes past
//    the row end get an offset outside the panel and read zero. The operand
//    row stride is at least K, a panel below 4 GiB (2 GiB with KTAIL).
#pragma once

#include "mls_device.h"

namespace mls {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

// Buffer descriptor of a block-uniform base and byte count. The inputs pass
// through readfirstlane so the descriptor lives in scalar registers: values
// the compiler derived with vector instructions (tile coordinates from integer
// division) would otherwise leave it in vector registers, and every buffer
// load through it would then be wrapped in a loop over distinct descriptors.
__device__ __forceinline__ char* uniform_ptr(const char* base) {
  const uint64_t v = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<char*>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const char* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(base), (short)0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ void block_barrier() { __builtin_amdgcn_s_barrier(); }

// Barrier after which other waves may overwrite LDS this wave has read: the
// wave's own LDS reads are drained first (s_barrier itself waits for nothing,
// and direct-to-LDS loads issued by other waves after the barrier reach LDS
// through the vector memory path, unordered with respect to reads still queued).
__device__ __forceinline__ void stage_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
}

// Blocks are dispatched round-robin over the 8 XCDs of the chip; this gives
// each XCD a contiguous range of logical tile indices (a bijection on
// [0, nb)), so tiles that share operand panels share one L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int q = nb / 8;
  const int r = nb % 8;
  const int x = b % 8;
  return x * q + (x < r ? x : r) + b / 8;
}

// Like xcd_remap for a launch whose first n1 tiles cost more than the rest:
// every XCD gets an even share of each phase, as one contiguous range per
// phase. Requires every XCD's share of phase 1 to fit in its block count
// (the host passes n1 = 0, i.e. plain xcd_remap, otherwise).
__device__ __forceinline__ int xcd_remap_phased(int b, int nb, int n1) {
  if (n1 <= 0 || n1 >= nb) return xcd_remap(b, nb);
  const int x = b % 8;
  const int i = b / 8;
  const int q = n1 / 8;
  const int r = n1 % 8;
  const int q1 = q + (x < r ? 1 : 0);
  if (i < q1) return x * q + (x < r ? x : r) + i;
  int start2 = 0;
  for (int y = 0; y < x; ++y) start2 += (nb - y + 7) / 8 - (q + (y < r ? 1 : 0));
  return n1 + start2 + (i - q1);
}

// Logical tile index -> (vocabulary tile, token tile). Tiles are taken in
// groups of `group_v` vocabulary tiles; inside a group the vocabulary tile
// varies fastest, so the blocks resident on one XCD at a time cover a
// rectangle of about group_v vocabulary tiles x (32 / group_v) token tiles
// and both operand panels are re-read from L2 rather than from memory.
__device__ __forceinline__ void tile_coords(int bl, int n_vt, int n_tt, int group_v, int& vt,
                                            int& tt) {
  const int per_group = group_v * n_tt;
  const int g = bl / per_group;
  const int first = g * group_v;
  const int gsz = (n_vt - first) < group_v ? (n_vt - first) : group_v;
  const int in = bl - g * per_group;
  vt = first + in % gsz;
  tt = in / gsz;
}

// LDS placement for tiles whose rows hold RB bytes of K (RB = 128 or 64):
// 16-byte chunk c of row `row` lives at chunk position c ^ swz(row). For
// 128-byte rows, rows r..r+7 and r, r+8 differ; for 64-byte rows (4 chunks)
// the XOR is ((row >> 1) & 3) ^ (3 * bit3(row)), which is a bijection over 16
// aligned rows sharing row % 4 and over 8 aligned rows sharing row % 2, so
// fragment reads are conflict-free for 8- and 16-lane read phases alike.
template <int RB>
__device__ __forceinline__ int swz_chunk(int row, int c) {
  if (RB == 128) return c ^ (row & 7) ^ ((row >> 3) & 1);
  return c ^ ((row >> 1) & 3) ^ (((row >> 3) & 1) * 3);
}

template <int RB>
__device__ __forceinline__ uint4 lds_read16_rb(const char* base, int row, int c) {
  return *reinterpret_cast<const uint4*>(base + row * RB + (swz_chunk<RB>(row, c) << 4));
}

// Operand layouts: KC = row-major [m][k] (K contiguous, the MFMA's natural
// operand order); MC = row-major [k][m] (M contiguous). An MC tile is staged
// in LDS as stored (K-tile rows of BM*2 bytes) and its fragments are read with
// ds_read_b64_tr_b16, which hands lane i of each 16-lane group column m0+i of
// four consecutive rows. Two such reads give the 8 consecutive K values of
// one MFMA operand. Chunks of a staged row are XOR-swizzled with 4*(k % 4):
// the 32 lanes served together read 64 contiguous bytes from each of four
// rows, and the swizzle puts those four 64-byte pieces in distinct banks.
enum { kLayoutKC = 0, kLayoutMC = 1 };

typedef short v4s_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int mc_chunk(int krow, int c) { return c ^ ((krow & 3) << 2); }

__device__ __forceinline__ uint2 lds_read_tr8(const char* p) {
  const v4s_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4s_t*)((__attribute__((address_space(3))) char*)p));
  return __builtin_bit_cast(uint2, v);
}

template <int BM, int BN, int WGM, int WGN, int STAGES, int RB = 128, int ALAY = kLayoutKC,
          int BLAY = kLayoutKC, bool KTAIL = false>
struct WideMma {
  static constexpr int kBM = BM;
  static constexpr int kBN = BN;
  static constexpr int kWGM = WGM;
  static constexpr int kWGN = WGN;
  static constexpr int NW = WGM * WGN;
  static constexpr int NT = NW * 64;
  static constexpr int WTM = BM / WGM;
  static constexpr int WTN = BN / WGN;
  static constexpr int FM = WTM / 32;
  static constexpr int FN = WTN / 32;
  static constexpr int CPR = RB / 16;     // 16-byte chunks per LDS row (KC layout)
  static constexpr int KSTEPS = RB / 32;  // MFMA K-steps (16 bf16) per K-tile
  static constexpr int BK = RB / 2;       // K values per K-tile
  static constexpr int kStageBytes = (BM + BN) * RB;
  static constexpr int kSmemBytes = STAGES * kStageBytes;
  static constexpr int LA = BM * CPR / NT;  // load instructions per thread per K-tile, A
  static constexpr int LB = BN * CPR / NT;
  static constexpr int kLoadsPerTile = LA + LB;
  static_assert(RB == 128 || RB == 64, "LDS rows of 64 or 128 bytes");
  static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile must split evenly over the waves");
  static_assert(STAGES >= 2 && STAGES <= 5, "2..5 stages");
  static_assert(kLoadsPerTile * (STAGES - 1) < 64, "vmcnt range");
  static_assert(!KTAIL || (RB == 128 && ALAY == kLayoutKC && BLAY == kLayoutKC),
                "K tails: K-contiguous operands");

  f32x16_t acc[FM][FN];

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[fm][fn][r] = 0.0f;
  }

  // Per-lane byte offsets (inside the operand panel) of the L chunks this lane
  // moves for a ROWS x 128-byte tile; fixed for the whole K loop.
  template <int L>
  __device__ __forceinline__ static void panel_offsets(int64_t ld_bytes, int wave, int lane,
                                                       uint32_t* off) {
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const int slot = (j * NW + wave) * 64 + lane;
      const int row = slot / CPR;
      const int c = swz_chunk<RB>(row, slot % CPR);  // the XOR is an involution
      off[j] = (uint32_t)(row * ld_bytes) + (uint32_t)(c << 4);
    }
  }

  // MC operand: per-lane offsets of its chunks inside a K-tile of BK rows of
  // ROWS*2 bytes (relative to the tile's first row and the block's column m0).
  template <int ROWS, int L>
  __device__ __forceinline__ static void panel_offsets_mc(int64_t ld_bytes, int wave, int lane,
                                                          uint32_t* off) {
    constexpr int CPM = ROWS / 8;  // chunks per staged row
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const int slot = (j * NW + wave) * 64 + lane;
      const int krow = slot / CPM;
      const int c = mc_chunk(krow, slot % CPM);
      off[j] = (uint32_t)(krow * ld_bytes) + (uint32_t)(c << 4);
    }
  }

  // bytes of the rows [row0, row0 + rows) that exist
  __device__ __forceinline__ static int64_t panel_bytes(int64_t ld_bytes, int64_t row0,
                                                        int64_t nrows, int rows) {
    int64_t avail = nrows - row0;
    avail = avail < rows ? avail : rows;
    return (avail > 0 ? avail : 0) * ld_bytes;
  }
  __device__ __forceinline__ static __amdgpu_buffer_rsrc_t panel_rsrc(const char* base,
                                                                      int64_t ld_bytes,
                                                                      int64_t row0, int64_t nrows,
                                                                      int rows) {
    return uniform_rsrc(base + row0 * ld_bytes, (int)panel_bytes(ld_bytes, row0, nrows, rows));
  }

  // Enqueue the direct loads of one KC operand tile at byte `sofs` of its rows
  // (a scalar offset, which is not range-checked: every lane's address stays
  // inside its row).
  template <int L>
  __device__ __forceinline__ static void issue_operand(__amdgpu_buffer_rsrc_t rsrc,
                                                       const uint32_t* off, int sofs, char* lds,
                                                       int wave) {
#pragma unroll
    for (int j = 0; j < L; ++j) {
      char* dst = lds + (j * NW + wave) * 64 * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t*)dst, 16, off[j], sofs, 0, 0);
    }
  }

  // As issue_operand for the K-tile at byte `sofs` of a KC operand whose rows
  // hold `kbytes` bytes of K: chunks past them read as zero (their offset is
  // moved outside the panel, which the descriptor's range check turns into 0).
  template <int L>
  __device__ __forceinline__ static void issue_operand_tail(__amdgpu_buffer_rsrc_t rsrc,
                                                            const uint32_t* off, int sofs,
                                                            int kbytes, char* lds, int wave,
                                                            int lane) {
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const int slot = (j * NW + wave) * 64 + lane;
      const int cb = swz_chunk<RB>(slot / CPR, slot % CPR) << 4;  // byte of the chunk in its K-tile
      char* dst = lds + (j * NW + wave) * 64 * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t*)dst, 16,
                                               sofs + cb < kbytes ? off[j] : 0x80000000u, sofs, 0,
                                               0);
    }
  }

  // Issues load j (0 .. LA + LB - 1) of one K-tile into stage `st`; ka / kb are
  // the tile's K positions: a KC operand's scalar offset (see issue_operand), an
  // MC operand's row offset, added to the lane's (so it is range-checked).
  __device__ __forceinline__ static void issue_one(int j, __amdgpu_buffer_rsrc_t ra,
                                                   __amdgpu_buffer_rsrc_t rb, const uint32_t* offa,
                                                   const uint32_t* offb, uint32_t ka, uint32_t kb,
                                                   char* st, int wave) {
    if (j < LA) {
      char* dst = st + (j * NW + wave) * 64 * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)dst, 16,
                                               offa[j] + (ALAY == kLayoutKC ? 0u : ka),
                                               ALAY == kLayoutKC ? (int)ka : 0, 0, 0);
    } else {
      const int jb = j - LA;
      char* dst = st + BM * RB + (jb * NW + wave) * 64 * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_t*)dst, 16,
                                               offb[jb] + (BLAY == kLayoutKC ? 0u : kb),
                                               BLAY == kLayoutKC ? (int)kb : 0, 0, 0);
    }
  }

  // One MFMA operand fragment of an MC tile: row block `r0` (32 rows), K-step kk.
  template <int ROWS>
  __device__ __forceinline__ static uint4 mc_frag(const char* base, int r0, int kk, int lane) {
    constexpr int RBYTES = ROWS * 2;
    const int g = lane >> 4;
    const int j = lane & 15;
    const int m = r0 + (g & 1) * 16 + 4 * (j & 3);
    const int k = kk * 16 + (g >> 1) * 8 + (j >> 2);
    const int c = m >> 3;
    const int in = (m & 7) * 2;
    const uint2 lo = lds_read_tr8(base + k * RBYTES + (mc_chunk(k, c) << 4) + in);
    const uint2 hi = lds_read_tr8(base + (k + 4) * RBYTES + (mc_chunk(k + 4, c) << 4) + in);
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
  }

  __device__ __forceinline__ void load_frags(const char* sA, const char* sB, int kk, int lane,
                                             int wm, int wn, uint4* a, uint4* b) {
    const int c = 2 * kk + (lane >> 5);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
      a[fm] = lds_read16_rb<RB>(sA + wm * WTM * RB, fm * 32 + (lane & 31), c);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
      b[fn] = lds_read16_rb<RB>(sB + wn * WTN * RB, fn * 32 + (lane & 31), c);
  }

  __device__ __forceinline__ void compute_stage(const char* sA, const char* sB, int lane, int wm,
                                                int wn) {
    constexpr int kMfma = FM * FN;
    constexpr int kReads = FM + FN;
    constexpr int kPer = kMfma / kReads > 0 ? kMfma / kReads : 1;  // MFMAs per read
    uint4 a[2][FM], b[2][FN];
    load_frags(sA, sB, 0, lane, wm, wn, a[0], b[0]);
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      __builtin_amdgcn_sched_barrier(0);
      if (kk < KSTEPS - 1) load_frags(sA, sB, kk + 1, lane, wm, wn, a[(kk + 1) & 1], b[(kk + 1) & 1]);
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) mma_step<Bf16>(acc[fm][fn], a[kk & 1][fm], b[kk & 1][fn]);
      if (kk < KSTEPS - 1) {
#pragma unroll
        for (int q = 0; q < kReads; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, kPer, 0);  // MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // DS read
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // acc = A[a_row0 : +BM, :K] * B[b_row0 : +BN, :K]^T with K = kbytes / 2, both
  // operands K-contiguous; a_rows / b_rows: rows of the stored operand matrix
  // (rows beyond it read as zero).
  // On return every wave has passed a barrier after its last LDS read, so the
  // LDS stages may be reused.
  __device__ __forceinline__ void run(const char* __restrict__ A, int64_t lda_bytes,
                                      int64_t a_row0, int64_t a_rows,
                                      const char* __restrict__ B, int64_t ldb_bytes,
                                      int64_t b_row0, int64_t b_rows, int64_t kbytes,
                                      char* smem, int tid) {
    static_assert(ALAY == kLayoutKC && BLAY == kLayoutKC, "K-contiguous operands");
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave % WGM;
    const int wn = wave / WGM;
    zero();
    const int nk = KTAIL ? (int)((kbytes + RB - 1) / RB) : (int)(kbytes / RB);
    const __amdgpu_buffer_rsrc_t ra = panel_rsrc(A, lda_bytes, a_row0, a_rows, BM);
    const __amdgpu_buffer_rsrc_t rb = panel_rsrc(B, ldb_bytes, b_row0, b_rows, BN);
    uint32_t offa[LA], offb[LB];
    panel_offsets<LA>(lda_bytes, wave, lane, offa);
    panel_offsets<LB>(ldb_bytes, wave, lane, offb);
    auto issue = [&](int kt) {
      char* st = smem + (kt % STAGES) * kStageBytes;
      if (KTAIL && (kt + 1) * RB > kbytes) {
        issue_operand_tail<LA>(ra, offa, kt * RB, (int)kbytes, st, wave, lane);
        issue_operand_tail<LB>(rb, offb, kt * RB, (int)kbytes, st + BM * RB, wave, lane);
      } else {
        issue_operand<LA>(ra, offa, kt * RB, st, wave);
        issue_operand<LB>(rb, offb, kt * RB, st + BM * RB, wave);
      }
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < nk) issue(s);
    for (int kt = 0; kt < nk; ++kt) {
      // tiles issued after kt that may stay in flight
      const int ahead = (nk - 1 - kt) < (STAGES - 2) ? (nk - 1 - kt) : (STAGES - 2);
      if (STAGES >= 4 && ahead >= 2) {
        wait_vmcnt<(STAGES >= 4 ? 2 : 0) * kLoadsPerTile>();
      } else if (STAGES >= 3 && ahead >= 1) {
        wait_vmcnt<(STAGES >= 3 ? 1 : 0) * kLoadsPerTile>();
      } else {
        wait_vmcnt<0>();
      }
      // stage (kt - 1) % STAGES is refilled below: every wave's reads of it must
      // have completed
      stage_barrier();
      if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1);
      const char* stage = smem + (kt % STAGES) * kStageBytes;
      compute_stage(stage, stage + BM * RB, lane, wm, wn);
    }
    stage_barrier();
  }

  // Fragment f (0 .. FM - 1: A, then B) of K-step kk.
  __device__ __forceinline__ static uint4 frag(const char* st, int f, int kk, int lane, int wm,
                                               int wn) {
    const char* sB = st + BM * RB;
    const int c = 2 * kk + (lane >> 5);
    if (f < FM) {
      if (ALAY == kLayoutKC) return lds_read16_rb<RB>(st + wm * WTM * RB, f * 32 + (lane & 31), c);
      return mc_frag<BM>(st, wm * WTM + f * 32, kk, lane);
    }
    if (BLAY == kLayoutKC) return lds_read16_rb<RB>(sB + wn * WTN * RB, (f - FM) * 32 + (lane & 31), c);
    return mc_frag<BN>(sB, wn * WTN + (f - FM) * 32, kk, lane);
  }

  // One K-step of run_pipelined(): its MFMAs on the fragments (a, b), with one
  // fragment of the next K-step read (rd(f)) behind each of the first FM + FN and
  // one K-tile load (ld(j)) behind each of the last ones, in exactly this order:
  // left to itself the scheduler puts the reads and loads in one run, in which
  // the matrix core idles.
  template <class Rd, class Ld>
  __device__ __forceinline__ void k_step(const uint4* a, const uint4* b, Rd&& rd, Ld&& ld) {
    constexpr int kMfma = FM * FN;
    constexpr int kFrags = FM + FN;
    static_assert(kMfma >= kFrags && kMfma >= kLoadsPerTile, "a slot for every read and load");
#pragma unroll
    for (int m = 0; m < kMfma; ++m) {
      mma_step<Bf16>(acc[m / FN][m % FN], a[m / FN], b[m % FN]);
      if (m < kFrags) rd(m < FN ? FM + m : m - FN);  // B's first: the next K-step's first MFMAs need all of them
      if (m >= kMfma - kLoadsPerTile) ld(m - (kMfma - kLoadsPerTile));
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // The product for any operand layout, with the accumulators set by init() (it
  // runs before any K-tile load is issued, so loads it issues are older than the
  // first K-tile's and complete with it). For an MC operand a_rows / b_rows is
  // the K extent that exists and a_row0 / b_row0 the first column.
  //
  // A K-tile holds two K-steps, and nothing is waited for that was not issued a
  // K-step or more before. The barrier that publishes K-tile kt + 1 stands
  // between the K-steps of tile kt: past it, the second one runs on fragments
  // already in registers while the first fragments of tile kt + 1 are read, and
  // the loads of tile kt + STAGES go to the stage of tile kt, whose reads every
  // wave has drained, so the matrix core has work on both sides of the barrier
  // and STAGES - 1 K-tiles stay in flight. Against two stages of 64-wide K, whose
  // first fragments are read after the barrier, the 256 x 256 gradient GEMM with
  // five stages of 32-wide K takes 4.31 instead of 4.44 ms per headline step, timed
  // in turn (1.18 PFLOP/s; 4.2 to 4.5 ms by card and under a profiler), and 4
  // stages the same. What was left on the card where it took 4.22: without its
  // loads the loop took 3.5 ms, without its fragment reads no less, and with every
  // tile on the same panels (all loads hit L2) 4.02, at a clock near 1.8 GHz.
  template <class Init>
  __device__ __forceinline__ void run_pipelined(const char* __restrict__ A, int64_t lda_bytes,
                                                int64_t a_row0, int64_t a_rows,
                                                const char* __restrict__ B, int64_t ldb_bytes,
                                                int64_t b_row0, int64_t b_rows, int64_t kbytes,
                                                char* smem, int tid, Init&& init) {
    static_assert(KSTEPS == 2 && !KTAIL && STAGES == 5, "K-tiles of two K-steps, five stages");
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM;
    const int wn = wave / WGM;
    init();
    const int nk = (int)(kbytes / RB);
    // KC operands: panel of BM (BN) rows. MC operands: panel of BM (BN) columns
    // over the stored rows; reads past them return 0. Tiles past the last are loaded like the others,
    // through descriptors of length 0 (they read as zero, touch no memory and
    // keep the number of loads in flight, and with it the wait below, the same).
    const int64_t sza = ALAY == kLayoutKC ? panel_bytes(lda_bytes, a_row0, a_rows, BM)
                                          : a_rows * lda_bytes - a_row0 * 2;
    const int64_t szb = BLAY == kLayoutKC ? panel_bytes(ldb_bytes, b_row0, b_rows, BN)
                                          : b_rows * ldb_bytes - b_row0 * 2;
    const int bytes_a = __builtin_amdgcn_readfirstlane((int)(sza > 0 ? sza : 0));
    const int bytes_b = __builtin_amdgcn_readfirstlane((int)(szb > 0 ? szb : 0));
    char* const pa = uniform_ptr(A + (ALAY == kLayoutKC ? a_row0 * lda_bytes : a_row0 * 2));
    char* const pb = uniform_ptr(B + (BLAY == kLayoutKC ? b_row0 * ldb_bytes : b_row0 * 2));
    uint32_t offa[LA], offb[LB];
    if (ALAY == kLayoutKC)
      panel_offsets<LA>(lda_bytes, wave, lane, offa);
    else
      panel_offsets_mc<BM, LA>(lda_bytes, wave, lane, offa);
    if (BLAY == kLayoutKC)
      panel_offsets<LB>(ldb_bytes, wave, lane, offb);
    else
      panel_offsets_mc<BN, LB>(ldb_bytes, wave, lane, offb);
    const uint32_t stepa = ALAY == kLayoutKC ? (uint32_t)RB : (uint32_t)(BK * lda_bytes);
    const uint32_t stepb = BLAY == kLayoutKC ? (uint32_t)RB : (uint32_t)(BK * ldb_bytes);
    auto rd = [&](int f, int slot, int kk, uint4* a, uint4* b) {
      const uint4 v = frag(smem + slot * kStageBytes, f, kk, lane, wm, wn);
      if (f < FM)
        a[f] = v;
      else
        b[f - FM] = v;
    };
    auto ld = [&](int j, int kt, int slot) {
      const bool in = kt < nk;
      issue_one((j + LA) % kLoadsPerTile,
                __builtin_amdgcn_make_buffer_rsrc(pa, (short)0, in ? bytes_a : 0, 0x00020000),
                __builtin_amdgcn_make_buffer_rsrc(pb, (short)0, in ? bytes_b : 0, 0x00020000), offa,
                offb, kt * stepa, kt * stepb, smem + slot * kStageBytes, wave);
    };
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
#pragma unroll
      for (int j = 0; j < kLoadsPerTile; ++j) ld(j, s, s);
    wait_vmcnt<(STAGES - 1) * kLoadsPerTile>();
    stage_barrier();
    uint4 a0[FM], b0[FN], a1[FM], b1[FN];
#pragma unroll
    for (int f = 0; f < FM + FN; ++f) rd(f, 0, 0, a0, b0);
    int slot = 0;
#pragma unroll 1
    for (int kt = 0; kt < nk; ++kt) {
      const int next = slot == STAGES - 1 ? 0 : slot + 1;
      __builtin_amdgcn_sched_barrier(0);
      k_step(a0, b0, [&](int f) { rd(f, slot, 1, a1, b1); }, [](int) {});
      wait_vmcnt<(STAGES - 2) * kLoadsPerTile>();
      stage_barrier();
      __builtin_amdgcn_sched_barrier(0);
      // (past the last tile: fragments of a stage of zeros, which nothing uses)
      k_step(a1, b1, [&](int f) { rd(f, next, 0, a0, b0); },
             [&](int j) { ld(j, kt + STAGES, slot); });
      slot = next;
    }
    wait_vmcnt<0>();
    stage_barrier();
  }

  __device__ __forceinline__ static int row_of(int wm, int fm, int r, int lane) {
    return wm * WTM + fm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  }
  __device__ __forceinline__ static int col_of(int wn, int fn, int lane) {
    return wn * WTN + fn * 32 + (lane & 31);
  }
};

}  // namespace mls
