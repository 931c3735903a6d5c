// GEMM kernel fed by direct global-to-LDS loads (global_load_lds_dwordx4: no
// staging registers, no LDS store instructions), for every operand layout,
// tile size and element type the launcher (gemm.hip) picks from.
//
// Workgroup: four waves, 2 x 2, each owning a (BM/2) x (BN/2) block of 16x16
// MFMA tiles.  k runs in tiles of 32 through a ring of four LDS stages:
// iteration t waits until tile t+1 has landed, synchronises once, issues the
// loads of tile t+4 into the stage of tile t (whose fragments every wave
// holds by then), and reads the fragments of tile t+1 between the MFMAs of
// tile t (fragment registers are double-buffered), so one barrier covers a
// k tile and a load has three iterations to land.
//
// LDS layouts.  A direct load writes 1 KB per wave contiguously, so the
// XOR swizzles that keep the fragment reads free of bank conflicts are
// applied to the global address each lane loads:
//   k-contiguous operand: [rows][32 k]; the 16-byte chunk c of row r sits at
//     c ^ ((r >> 1) & 3) (bf16, 4 chunks) or c ^ (r & 7) (fp32, 8 chunks);
//     fragments by ds_read_b128.
//   other operand: panels of PANEL rows, each [32 k][PANEL rows].  bf16:
//     fragments by two ds_read_b64_tr_b16, each transposing a 4 (k) x 16
//     (rows) block across 16 lanes; one LDS cycle serves the k rows K0..K0+3
//     and K0+8..K0+11, which the swizzle puts on distinct banks: chunk c of
//     k row k at c ^ (2 (k & 3) + 8 ((k >> 3) & 1)) for rows of 16 chunks or
//     more, c ^ (2 ((k >> 1) & 1) + 4 ((k >> 3) & 1)) for rows of 8.  fp32:
//     fragments by ds_read_b32, chunk c at c ^ (4 ((k >> 3) & 3)) (16 chunks)
//     or c ^ (4 ((k >> 3) & 1)) (8 chunks).
// Rows past the operand are clamped to its last valid row (or chunk of rows):
// they only reach output rows or columns that are never stored.  k past the
// end reads 16 bytes of zeros instead, in both operands, so any k whose
// chunks are whole works; the loop runs whole groups of four k tiles, then the
// one to three that are left.
#pragma once

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace atom {
namespace dl {

constexpr int BK = 32, NT = 256, STAGES = 4;

// What direct loads read for k past the end.
static __device__ __attribute__((aligned(16))) uint32_t zero_chunk[4];

// One operand tile: R rows (m of A, n of B) x 32 k in a stage.
template <typename T, bool KC, int R>
struct Operand {
  static constexpr int E = 16 / sizeof(T);                      // elements per chunk
  static constexpr int RL = R < 64 ? R : (R + 63) / 64 * 64;    // rows loaded
  static constexpr int BYTES = RL * BK * static_cast<int>(sizeof(T));
  static constexpr int LPT = BYTES / (NT * 16);                 // loads per thread
  static constexpr int PANEL = sizeof(T) == 2 ? (RL % 256 == 0 ? 256 : RL % 128 == 0 ? 128 : 64) : (RL % 64 == 0 ? 64 : 32);
  static constexpr int CPR = KC ? BK / E : PANEL / E;           // chunks per LDS row
  static_assert(BYTES % (NT * 16) == 0 && RL % PANEL == 0, "tile split");

  static __device__ __forceinline__ int swz(int r) {
    if constexpr (KC) return sizeof(T) == 2 ? (r >> 1) & 3 : r & 7;
    else if constexpr (sizeof(T) == 2) return PANEL >= 128 ? 2 * (r & 3) + 8 * ((r >> 3) & 1) : 2 * ((r >> 1) & 1) + 4 * ((r >> 3) & 1);
    else return PANEL == 64 ? 4 * ((r >> 3) & 3) : 4 * ((r >> 3) & 1);
  }

  // Source of this thread's chunk q * NT + tid of a tile.
  struct Src {
    const T* p;     // address for k tile 0
    int64_t kstep;  // elements to advance per k tile
    int k;          // first k of the chunk inside a tile
    __device__ void init(const T* X, int64_t ld, int r0, int Rlim, int id) {
      if constexpr (KC) {
        const int r = id / CPR, c = (id % CPR) ^ swz(r);
        p = X + static_cast<int64_t>(min(r0 + r, Rlim - 1)) * ld + c * E;
        kstep = BK;
        k = c * E;
      } else {
        const int panel = id / (CPR * BK), kk = id / CPR % BK, c = (id % CPR) ^ swz(kk);
        p = X + static_cast<int64_t>(kk) * ld + min(r0 + panel * PANEL + c * E, Rlim - E);
        kstep = static_cast<int64_t>(BK) * ld;
        k = kk;
      }
    }
    // TAIL: a tile may reach past k, where the chunk reads zeros
    template <bool TAIL>
    __device__ __forceinline__ void load(uint8_t* stage, int kt, int K, int group) const {
      const void* s = p + kt * kstep;
      if constexpr (TAIL) s = kt * BK + k < K ? s : static_cast<const void*>(zero_chunk);
      lds_dma16(s, __builtin_amdgcn_readfirstlane(lds_offset(stage) + group * 1024));
    }
  };

  // Byte offsets inside a stage of this lane's fragment of tile rows
  // row0..row0+15; loop-invariant.
  struct Off {
    uint32_t o[KC ? (sizeof(T) == 2 ? 1 : 2) : (sizeof(T) == 2 ? 2 : 1)];
    __device__ void init(int row0, int lane) {
      const int r = lane & 15, g = lane >> 4;
      if constexpr (KC) {
        const int row = row0 + r;
        if constexpr (sizeof(T) == 2) {
          o[0] = row * 64 + 16 * (g ^ swz(row));
        } else {
          o[0] = row * 128 + 16 * ((2 * g) ^ swz(row));
          o[1] = row * 128 + 16 * ((2 * g + 1) ^ swz(row));
        }
      } else if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = 8 * g + 4 * h + (r >> 2);
          const int m = row0 + 4 * (r & 3);
          o[h] = (m / PANEL) * (PANEL * BK * 2) + k * (PANEL * 2) + 16 * ((m % PANEL >> 3) ^ swz(k)) + 8 * (r & 1);
        }
      } else {
        const int m = row0 + r;
        o[0] = (m / PANEL) * (PANEL * BK * 4) + 8 * g * (PANEL * 4) + 16 * ((m % PANEL >> 2) ^ swz(8 * g)) + 4 * (m & 3);
      }
    }
  };

  static __device__ __forceinline__ void frag(Frag<T>& f, const uint8_t* st, const Off& fo) {
    if constexpr (sizeof(T) == 2) {
      if constexpr (KC) {
        f.v = *reinterpret_cast<const uint4*>(st + fo.o[0]);
      } else {
        const uint2 lo = ds_read_tr8(st + fo.o[0]), hi = ds_read_tr8(st + fo.o[1]);
        f.v = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
    } else if constexpr (KC) {
      f.lo = *reinterpret_cast<const float4*>(st + fo.o[0]);
      f.hi = *reinterpret_cast<const float4*>(st + fo.o[1]);
    } else {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float*>(st + fo.o[0] + j * (PANEL * 4));
      f.lo = make_float4(v[0], v[1], v[2], v[3]);
      f.hi = make_float4(v[4], v[5], v[6], v[7]);
    }
  }
};

// Barrier after this wave's LDS reads have completed; the wait is the
// builtin so that the compiler knows those fragment registers are ready.
__device__ __forceinline__ void barrier_after_reads() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt unconstrained
  asm volatile("s_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// acc += a b with the accumulator pinned to its AGPRs.  The accumulator
// registers of a 128-row wave (192 or 256) sit in the AGPR file; left to itself
// the register allocator splits them between AGPRs and VGPRs and copies them around every
// MFMA.  Issued in program order (volatile); the kernel supplies the wait
// states between the accumulators' other writes and reads and these MFMAs.
__device__ __forceinline__ void mfma_agpr(f32x4_t& acc, const Frag<bf16_t>& a, const Frag<bf16_t>& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
               : "+a"(acc)
               : "v"(__builtin_bit_cast(bf16x8_t, a.v)), "v"(__builtin_bit_cast(bf16x8_t, b.v)));
}

template <int EPI>
constexpr bool epi_reads_elem() {
  return EPI == EPI_ACC_F32 || EPI == EPI_BIAS_RESID || EPI == EPI_GELU_BWD;
}
template <int EPI>
constexpr bool epi_has_bias() {
  return EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESID;
}

template <typename T>
__device__ __forceinline__ void unpack4(const T* p, float* v) {
  if constexpr (sizeof(T) == 2) {
    const uint2 w = *reinterpret_cast<const uint2*>(p);
    v[0] = bf2f(w.x & 0xffff); v[1] = bf2f(w.x >> 16); v[2] = bf2f(w.y & 0xffff); v[3] = bf2f(w.y >> 16);
  } else {
    const float4 w = *reinterpret_cast<const float4*>(p);
    v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
  }
}
template <typename T>
__device__ __forceinline__ void pack4(T* p, const float* v) {
  if constexpr (sizeof(T) == 2)
    *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
  else
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// Workgroups a CU holds: one of the 256-row tiles (their LDS and, with one
// wave per SIMD, the AGPR accumulators), else what four stages leave room for.
template <typename T, int BM, int BN>
constexpr int occupancy() {
  if (BM == 256) return 1;
  constexpr int lds = STAGES * (BM + BN) * BK * static_cast<int>(sizeof(T));
  return lds > 80 * 1024 ? 1 : lds > 53 * 1024 ? 2 : lds > 40 * 1024 ? 3 : 4;
}

// TAIL: k is not a multiple of 128, so one to three k tiles may follow the last
// whole group of four, the last tile may reach past k, and every load tests its
// chunk (three vector instructions: 3-4 % at 4096x12288x4096, so whole groups
// take the copy without).
template <typename T, bool AKC, bool BKC, int EPI, int BM, int BN, bool TAIL>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(occupancy<T, BM, BN>(), occupancy<T, BM, BN>())))
gemm_dl_kernel(GemmArgs g) {
  using OA = Operand<T, AKC, BM>;
  using OB = Operand<T, BKC, BN>;
  constexpr bool PIN = BM == 256;  // accumulators in AGPRs, one wave per SIMD
  constexpr int TM = BM / 32, TN = BN / 32;
  static_assert(TM >= TN, "fragment rows");
  constexpr int LT = OA::LPT + OB::LPT;  // loads per thread and k tile
  // epilogue staging: RB rows of a wave's block at a time, PITCH floats per row
  constexpr int RB = TM * 16 < 32 ? TM * 16 : 32, PITCH = TN * 16 + 4;
  constexpr int LDS = std::max(STAGES * (OA::BYTES + OB::BYTES), 4 * RB * PITCH * 4);
  __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wm = w >> 1, wn = w & 1;

  // Work item order: consecutive workgroups go round-robin over the 8 XCDs,
  // so each XCD takes a contiguous range of items (its tiles share operand
  // panels through its L2); items are the tiles of the first k range, then of
  // the next; tiles go in groups of 8 row tiles sweeping the columns.
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int tiles = tiles_m * tiles_n, total = static_cast<int>(gridDim.x);
  const int xcd = blockIdx.x & 7, rem = total & 7;
  int pid = xcd * (total >> 3) + min(xcd, rem) + (blockIdx.x >> 3);
  const int split = pid / tiles;
  pid -= split * tiles;
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int first_m = (pid / per_group) * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  const int pid_m = first_m + (pid % per_group) % gsize;
  const int pid_n = (pid % per_group) / gsize;
  const int m0 = pid_m * BM, n0 = pid_n * BN;

  typename OA::Src sra[OA::LPT];
  typename OB::Src srb[OB::LPT];
#pragma unroll
  for (int q = 0; q < OA::LPT; ++q) sra[q].init(static_cast<const T*>(g.A), g.lda, m0, g.M, q * NT + tid);
#pragma unroll
  for (int q = 0; q < OB::LPT; ++q) srb[q].init(static_cast<const T*>(g.B), g.ldb, n0, g.N, q * NT + tid);
  // k tiles of this workgroup: kquads groups of four per split, the rest in
  // the last one (the launcher leaves none empty).  With TAIL the last group
  // may be short: only the tiles that hold k are loaded and multiplied
  // (4096x8192x576: 49.0 us with a whole last group, 47.0; 8192x8192x352: 81, 78).
  const int quads = (g.K + 4 * BK - 1) / (4 * BK);
  const int kbase = split * g.kquads * 4;
  const int nk4 = min(g.kquads, quads - split * g.kquads) * 4;
  const int nk = TAIL ? min(nk4, (g.K + BK - 1) / BK - kbase) : nk4;
  // Each XCD starts its k loop at its own eighth of the range (the tile's
  // sum is rotated, the same for every launch of the shape).  Workgroups
  // walk k in step, so without it the whole GPU reads the same column range
  // of every row at once; when both operands are k-contiguous, rows of a long
  // k are 32 KB apart and those addresses share their low bits, which crowds
  // a few memory channels (4096x4096x16384: 500 -> 418 us).  The workgroups
  // of one XCD share operand tiles through its L2, so they keep one offset.
  const int koff = (xcd * (nk4 >> 3)) & ~3;
  auto rot = [&](int kt) {
    const int r = kt + koff;
    return kbase + (r >= nk ? r - nk : r);
  };

  f32x4_t acc[TM][TN];
  // fp32: odd k tiles have accumulators of their own, and after 512 k both join
  // the running totals and start again from zero, so a sum has 64 MFMAs
  // of 4 k in a row, and k / 512 totals, instead of k / 4.  Error against 64 bits at k =
  // 8192: 3.0e-7 relative; 1.15e-6 without the totals, 8.1e-7 with the ranges
  // that the register-staged kernel splits such a k into.  (One set of
  // accumulators and totals after every 256 k: as exact, but the chain of
  // MFMAs on one accumulator costs 3-4 % at 32x32.)
  constexpr bool TOTALS = sizeof(T) == 4;
  f32x4_t acc2[TOTALS ? TM : 1][TOTALS ? TN : 1], tot[TOTALS ? TM : 1][TOTALS ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (TOTALS) tot[i][j] = acc2[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (PIN) asm volatile("" : "+a"(acc[i][j]));
    }
  // wait states between the zeroing writes and the first MFMA reading them
  if constexpr (PIN) asm volatile("s_nop 7\n\ts_nop 7");

  typename OA::Off foa[TM];
  typename OB::Off fob[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) foa[i].init(wm * TM * 16 + i * 16, lane);
#pragma unroll
  for (int j = 0; j < TN; ++j) fob[j].init(wn * TN * 16 + j * 16, lane);

  auto stage_a = [&](int s) -> uint8_t* { return lds + s * OA::BYTES; };
  auto stage_b = [&](int s) -> uint8_t* { return lds + STAGES * OA::BYTES + s * OB::BYTES; };
  auto load = [&](int s, int kt, int l) {
    if (l < OA::LPT) sra[l < OA::LPT ? l : 0].template load<TAIL>(stage_a(s), kt, g.K, l * 4 + w);
    else srb[l < OA::LPT ? 0 : l - OA::LPT].template load<TAIL>(stage_b(s), kt, g.K, (l - OA::LPT) * 4 + w);
  };

  Frag<T> fa0[TM], fb0[TN], fa1[TM], fb1[TN];
  // prologue: tiles 0..3 in flight, fragments of tile 0 in set 0.  Loads
  // past the last tile repeat it (into stages nobody reads again), so every
  // iteration has the same loads outstanding; they land before the exit.
#pragma unroll
  for (int s = 0; s < STAGES; ++s) {
    const int kt = rot(TAIL ? min(s, nk - 1) : s);
#pragma unroll
    for (int l = 0; l < LT; ++l) load(s, kt, l);
  }
  wait_loads<3 * LT>();
  barrier_after_reads();
#pragma unroll
  for (int i = 0; i < TM; ++i) OA::frag(fa0[i], stage_a(0), foa[i]);
#pragma unroll
  for (int j = 0; j < TN; ++j) OB::frag(fb0[j], stage_b(0), fob[j]);

  auto body = [&](auto S_, int t, Frag<T>(&ca)[TM], Frag<T>(&cb)[TN], Frag<T>(&na)[TM], Frag<T>(&nb)[TN]) {
    constexpr int S = decltype(S_)::value;
    // tile t+1 has landed for every wave, and every wave has read tile t
    wait_loads<2 * LT>();
    barrier_after_reads();
    const int kt = rot(min(t + 4, nk - 1));
    // per row i: the fragments i of tile t+1 (after the last tile they come
    // from a stale stage and are never used), then the MFMAs of row i of this
    // tile, which hide the reads' latency, with the direct loads of tile t+4
    // spread over the rows, half way through each (3-4 % faster than at the
    // row's start; clustering the loads cost 3-5 %)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      OA::frag(na[i], stage_a((S + 1) & 3), foa[i]);
      if (i < TN) OB::frag(nb[i < TN ? i : 0], stage_b((S + 1) & 3), fob[i < TN ? i : 0]);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (j == TN / 2) {
#pragma unroll
          for (int l = 0; l < LT; ++l)
            if (l * TM / LT == i) load(S, kt, l);
        }
        if constexpr (PIN) mfma_agpr(acc[i][j], cb[j], ca[i]);
        else if constexpr (TOTALS && (S & 1)) mfma16(acc2[i][j], cb[j], ca[i]);
        else mfma16(acc[i][j], cb[j], ca[i]);
      }
    }
  };
  // whole groups of four: no tile is conditional inside the loop
  for (int t = 0; t + 4 <= nk; t += 4) {
    body(std::integral_constant<int, 0>{}, t, fa0, fb0, fa1, fb1);
    body(std::integral_constant<int, 1>{}, t + 1, fa1, fb1, fa0, fb0);
    body(std::integral_constant<int, 2>{}, t + 2, fa0, fb0, fa1, fb1);
    body(std::integral_constant<int, 3>{}, t + 3, fa1, fb1, fa0, fb0);
    if constexpr (TOTALS)
      if ((t & 12) == 12) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            tot[i][j] += acc[i][j] + acc2[i][j];
            acc[i][j] = acc2[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
      }
  }

  if constexpr (TAIL) {
    const int t = nk & ~3;
    if (t < nk) body(std::integral_constant<int, 0>{}, t, fa0, fb0, fa1, fb1);
    if (t + 1 < nk) body(std::integral_constant<int, 1>{}, t + 1, fa1, fb1, fa0, fb0);
    if (t + 2 < nk) body(std::integral_constant<int, 2>{}, t + 2, fa0, fb0, fa1, fb1);
  }

  // every direct load has landed; wait states between the last MFMAs and
  // the reads of their accumulators
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
  if constexpr (PIN) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
  }
  if constexpr (TOTALS) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = tot[i][j] + (acc[i][j] + acc2[i][j]);
  }
  // Epilogue through LDS, RB rows of the wave's block at a time: the
  // accumulators go to a wave-private [RB][BN/2] fp32 staging area, and each
  // lane takes back 4 consecutive columns of one row, so a wave's stores (and
  // the epilogue's reads of bias, residual or saved pre-activations) cover
  // whole rows of the block instead of 32-byte pieces of 16 rows.
  barrier_after_reads();  // every wave is done with the stages
  float* stg = reinterpret_cast<float*>(lds) + w * (RB * PITCH);
  const int row0 = m0 + wm * TM * 16, col0 = n0 + wn * TN * 16;
  // N, ldc and ldaux are multiples of 4 (the launcher checks): a lane's four
  // columns are all inside the matrix or all past it, and every access is one
  // 4-vector.  They are the same columns in every row the lane stores, so the
  // bias is loaded once and the row pointers advance by a fixed stride.  LPR
  // lanes cover a row and a pass RPP rows (a power of two: with 24 or 20
  // lanes per row the rest of the wave idles).
  constexpr int LPR = TN * 4, RPP = LPR > 16 ? 2 : 64 / LPR, NQ = RB / RPP, NB = TM * 16 / RB;
  const int cc = 4 * (lane % LPR), nb = col0 + cc, rsub = lane / LPR;
  const bool col_ok = nb < g.N && rsub < RPP;
  const int rsub0 = LPR * RPP == 64 ? rsub : min(rsub, RPP - 1);
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  if constexpr (epi_has_bias<EPI>())
    if (col_ok) unpack4(static_cast<const T*>(g.bias) + nb, bv);
  // The element operands (C itself, the fp32 residual or the saved
  // pre-activation) are requested ahead of their use: every CU reaches its
  // epilogue at about the same time, so a load issued just before its use
  // waits out a GPU-wide burst.  bf16 operands go out two blocks ahead (two
  // registers per row), fp32 ones one block ahead.
  // Interior blocks take a branch-free copy of the epilogue: with per-row
  // bounds tests the compiler waits for every load in flight at each test,
  // which defeats the loads issued ahead.
  auto epilogue = [&](auto GUARD_, const GemmArgs& ga) {
    constexpr bool GUARD = decltype(GUARD_)::value;
    constexpr int E = EPI;
    constexpr bool F32_OUT = E == EPI_STORE_F32 || E == EPI_ACC_F32 || E == EPI_BIAS_RESID;
    constexpr bool ELEM = epi_reads_elem<E>();
    constexpr bool AUX16 = E == EPI_GELU_BWD && sizeof(T) == 2;
    constexpr int AHEAD = std::min(AUX16 ? 2 : 1, NB - 1);
    using Raw = typename std::conditional<AUX16, uint2, float4>::type;
    Raw xr[NB][NQ];
    // lanes past the rows of a pass (24 lanes per row) load and store nothing
    const bool lane_on = LPR * RPP == 64 || rsub < RPP;
    auto load_block = [&](int h) {
      const int mq = row0 + h * RB + rsub;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (GUARD ? (mq + RPP * q < ga.M && col_ok) : lane_on) {
          if constexpr (E == EPI_GELU_BWD)
            xr[h][q] = *reinterpret_cast<const Raw*>(static_cast<const T*>(ga.aux) +
                                                     static_cast<int64_t>(mq + RPP * q) * ga.ldaux + nb);
          else
            xr[h][q] = *reinterpret_cast<const Raw*>((E == EPI_ACC_F32 ? static_cast<const float*>(ga.C) : ga.resid) +
                                                     static_cast<int64_t>(mq + RPP * q) * ga.ldc + nb);
        }
      }
    };
    if constexpr (ELEM) {
#pragma unroll
      for (int h = 0; h <= AHEAD; ++h) load_block(h);
    }
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      if constexpr (ELEM)
        if (h > 0 && h + AHEAD < NB) load_block(h + AHEAD);
      const int mq = row0 + h * RB + rsub;  // row of q = 0; row q is mq + RPP q
      const int64_t cq = static_cast<int64_t>(mq) * ga.ldc + nb, aq = static_cast<int64_t>(mq) * ga.ldaux + nb;
#pragma unroll
      for (int ii = 0; ii < RB / 16; ++ii)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const f32x4_t& a = acc[h * (RB / 16) + ii][j];
          *reinterpret_cast<float4*>(stg + (ii * 16 + lr) * PITCH + j * 16 + lg * 4) = make_float4(a[0], a[1], a[2], a[3]);
        }
      float4 sv[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        sv[q] = *reinterpret_cast<const float4*>(stg + (RPP * q + rsub0) * PITCH + cc);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (GUARD ? !(mq + RPP * q < ga.M && col_ok) : !lane_on) continue;
        float v[4] = {sv[q].x, sv[q].y, sv[q].z, sv[q].w};
        const int64_t off = cq + RPP * q * ga.ldc;
        float xe[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (AUX16) {
          xe[0] = bf2f(xr[h][q].x & 0xffff); xe[1] = bf2f(xr[h][q].x >> 16);
          xe[2] = bf2f(xr[h][q].y & 0xffff); xe[3] = bf2f(xr[h][q].y >> 16);
        } else if constexpr (ELEM) {
          xe[0] = xr[h][q].x; xe[1] = xr[h][q].y; xe[2] = xr[h][q].z; xe[3] = xr[h][q].w;
        }
        // the arithmetic of epilogue4 (gemm.hip), in the same order
        if constexpr (E == EPI_ACC_F32) {
          for (int r = 0; r < 4; ++r) v[r] += xe[r];
        } else if constexpr (E == EPI_BIAS) {
          for (int r = 0; r < 4; ++r) v[r] += bv[r];
        } else if constexpr (E == EPI_BIAS_GELU) {
          float gv[4];
          for (int r = 0; r < 4; ++r) {
            const float u = to_f<T>(from_f<T>(v[r] + bv[r]));
            v[r] = u;
            gv[r] = gelu_f(u);
          }
          pack4(static_cast<T*>(ga.aux) + aq + RPP * q * ga.ldaux, v);
          for (int r = 0; r < 4; ++r) v[r] = gv[r];
        } else if constexpr (E == EPI_BIAS_RESID) {
          for (int r = 0; r < 4; ++r) v[r] = xe[r] + (v[r] + bv[r]);
        } else if constexpr (E == EPI_GELU_BWD) {
          for (int r = 0; r < 4; ++r) v[r] *= gelu_grad_f(xe[r]);
        }
        if constexpr (E == EPI_STORE_F32) {
          if (g.stream) stream4(static_cast<float*>(ga.C) + off, v);
          else pack4(static_cast<float*>(ga.C) + off, v);
        } else if constexpr (F32_OUT) pack4(static_cast<float*>(ga.C) + off, v);
        else pack4(static_cast<T*>(ga.C) + off, v);
      }
    }
  };
  const bool interior = row0 + TM * 16 <= g.M && col0 + TN * 16 <= g.N;
  if constexpr (EPI == EPI_STORE_F32) {
    // a split over k: the raw fp32 sums go to C[split][M][N] (the workspace),
    // and splitk_reduce adds the splits in order and applies the epilogue
    if (g.splits > 1) g.C = static_cast<float*>(g.C) + static_cast<int64_t>(split) * g.M * g.N;
  }
  if (interior) epilogue(std::false_type{}, g);
  else epilogue(std::true_type{}, g);
}

// Launches one tile configuration; MAIN_ONLY instantiates the layout and
// epilogue combinations of the training step only.  The copy without TAIL
// exists for those in bf16 (fp32 tiles are bound by their MFMAs).
template <typename T, int BM, int BN, bool MAIN_ONLY>
hipError_t launch(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  const dim3 grid(static_cast<unsigned>(tiles * g.splits)), block(NT);
  const bool tail = g.K % (4 * BK) != 0;
#define ATOM_DL(AK, BK_, E)                                                                        \
  case E:                                                                                          \
    if constexpr (sizeof(T) == 2 && gemm_main_combo(AK, BK_, E))                                   \
      if (!tail) {                                                                                 \
        hipLaunchKernelGGL((gemm_dl_kernel<T, AK, BK_, E, BM, BN, false>), grid, block, 0, s, g);  \
        return hipGetLastError();                                                                  \
      }                                                                                            \
    if constexpr (!MAIN_ONLY || gemm_main_combo(AK, BK_, E)) {                                     \
      hipLaunchKernelGGL((gemm_dl_kernel<T, AK, BK_, E, BM, BN, true>), grid, block, 0, s, g);     \
      return hipGetLastError();                                                                    \
    }                                                                                              \
    break;
#define ATOM_DL_LAYOUT(AK, BK_)                                                                    \
  if (akc == AK && bkc == BK_) switch (epi) {                                                      \
      ATOM_DL(AK, BK_, EPI_STORE)                                                                  \
      ATOM_DL(AK, BK_, EPI_STORE_F32)                                                              \
      ATOM_DL(AK, BK_, EPI_ACC_F32)                                                                \
      ATOM_DL(AK, BK_, EPI_BIAS)                                                                   \
      ATOM_DL(AK, BK_, EPI_BIAS_GELU)                                                              \
      ATOM_DL(AK, BK_, EPI_BIAS_RESID)                                                             \
      ATOM_DL(AK, BK_, EPI_GELU_BWD)                                                               \
      default: break;                                                                              \
    }
  ATOM_DL_LAYOUT(true, true)
  ATOM_DL_LAYOUT(true, false)
  ATOM_DL_LAYOUT(false, false)
  ATOM_DL_LAYOUT(false, true)
#undef ATOM_DL_LAYOUT
#undef ATOM_DL
  return hipErrorInvalidValue;
}

}  // namespace dl
}  // namespace atom
