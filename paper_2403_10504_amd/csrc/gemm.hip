// Dense GEMM on CDNA4 matrix cores with fused epilogues.
//
//   C[m][n] (op)= sum_k A(m,k) * B(k,n),   fp32 accumulation.
//
// Operand layouts (both row-major in memory):
//   A_KC: A(m,k) = A[m*lda + k]   (k contiguous)   else A(m,k) = A[k*lda + m]
//   B_KC: B(k,n) = B[n*ldb + k]   (k contiguous)   else B(k,n) = B[k*ldb + n]
// The three products of a linear layer y = x W^T + b with W stored [out][in]:
//   forward   y  = x  W^T : A = x  (KC),          B = W  (KC)
//   data grad dx = dy W   : A = dy (KC),          B = W  (not KC)
//   weight grad dW = dy^T x: A = dy (not KC),      B = x  (not KC)
//
// The direct-load kernel (gemm_dl.h) takes the problems whose 16-byte chunks
// are whole (dl_applies), but for fp32 ones of short k; choose() picks its tile
// and a split over k.  The kernel here is for the rest (k, leading dimensions
// or rows of a not k-contiguous operand that are no multiples of 8 in bf16 or 4
// in fp32, N or ldc no multiples of 4): tiles of 128x128 by four waves or, of
// large bf16 problems, 256x256 by sixteen, a 128-byte k tile (64 bf16 or 32
// fp32) staged through registers and
// double-buffered in LDS with k contiguous (rows padded to 144 bytes to
// spread ds_read_b128 over the banks; operands that are not k-contiguous in
// memory are transposed while being written to LDS).  A split over k writes
// fp32 partials that a second kernel sums in split order before the epilogue,
// so the result does not depend on scheduling.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace atom {
namespace {

constexpr int ROW_BYTES = 128, PITCH_BYTES = 144;

// Workgroup tile of BS x BS computed by W x W waves, each owning a 64 x 64
// block of 16x16 MFMA tiles.
template <int BS_>
struct Cfg {
  static constexpr int BS = BS_, W = BS / 64, NT = 64 * W * W;
};
using Small = Cfg<128>;
using Big = Cfg<256>;
constexpr int TM = 4, TN = 4;

template <typename T>
struct Tile {
  static constexpr int BK = ROW_BYTES / sizeof(T);    // k per tile
  static constexpr int PITCH = PITCH_BYTES / sizeof(T);
  static constexpr int KV = 16 / sizeof(T);           // elements per 16 bytes
  static constexpr int PAIR = 4 / sizeof(T);          // elements per dword
  static constexpr int NSLICE = BK / 32;
};

// Stages an R-row x BK tile of one operand (rows = m for A, n for B) with NT
// threads.  Registers hold the next tile while the current one is consumed.
template <typename T, bool KC, int R, int NT>
struct Loader {
  using TL = Tile<T>;
  static constexpr int DW = R * ROW_BYTES / 4 / NT;   // dwords per thread
  static constexpr int UPK = R / TL::PAIR;            // !KC: dword units per k row
  static constexpr int UPT = 8 * UPK / NT;            // !KC: units per thread
  static constexpr int NOFF = KC ? DW / 4 : UPT;
  uint32_t r[DW];
  uint32_t off[NOFF];  // byte offsets of this thread's loads inside a full tile

  // Offsets for load_fast (leading dimension ld, elements).
  __device__ void init(int64_t ld, int tid) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < NOFF; ++i) {
        const int c = tid + NT * i;
        off[i] = static_cast<uint32_t>(((c >> 3) * ld + (c & 7) * TL::KV) * sizeof(T));
      }
    } else {
#pragma unroll
      for (int i = 0; i < NOFF; ++i) {
        const int u = tid + NT * i;
        off[i] = static_cast<uint32_t>(((u / UPK) * TL::KV * ld + (u % UPK) * TL::PAIR) * sizeof(T));
      }
    }
  }

  // Unguarded load of a tile that lies wholly inside the operand (rows
  // r0..r0+R-1 and k0..k0+BK-1): one uniform base pointer and the 32-bit
  // per-thread offsets from init.
  __device__ void load_fast(const T* __restrict__ X, int64_t ld, int r0, int k0) {
    if constexpr (KC) {
      const char* base = reinterpret_cast<const char*>(X + static_cast<int64_t>(r0) * ld + k0);
#pragma unroll
      for (int i = 0; i < NOFF; ++i) {
        const uint4 v = *reinterpret_cast<const uint4*>(base + off[i]);
        r[4 * i + 0] = v.x;
        r[4 * i + 1] = v.y;
        r[4 * i + 2] = v.z;
        r[4 * i + 3] = v.w;
      }
    } else {
      const char* base = reinterpret_cast<const char*>(X + static_cast<int64_t>(k0) * ld + r0);
      const uint32_t step = static_cast<uint32_t>(ld * sizeof(T));
#pragma unroll
      for (int i = 0; i < NOFF; ++i)
#pragma unroll
        for (int j = 0; j < TL::KV; ++j) r[i * TL::KV + j] = *reinterpret_cast<const uint32_t*>(base + off[i] + j * step);
    }
  }

  // KC: rows are contiguous along k, R rows x 8 chunks of 16 bytes.
  // !KC: memory is [k][row]; a unit is KV consecutive k rows x PAIR rows.
  __device__ void load(const T* __restrict__ X, int64_t ld, int Rlim, int K, int r0, int k0, int tid) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < DW / 4; ++i) {
        const int c = tid + NT * i;
        const int row = c >> 3, kc = c & 7;
        const int gr = r0 + row, gk = k0 + kc * TL::KV;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (gr < Rlim && gk < K) v = *reinterpret_cast<const uint4*>(X + static_cast<int64_t>(gr) * ld + gk);
        r[4 * i + 0] = v.x;
        r[4 * i + 1] = v.y;
        r[4 * i + 2] = v.z;
        r[4 * i + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < UPT; ++i) {
        const int u = tid + NT * i;
        const int kb = u / UPK, rc = u % UPK;
        const int gr = r0 + rc * TL::PAIR;
#pragma unroll
        for (int j = 0; j < TL::KV; ++j) {
          const int gk = k0 + kb * TL::KV + j;
          uint32_t v = 0;
          if (gr < Rlim && gk < K) v = *reinterpret_cast<const uint32_t*>(X + static_cast<int64_t>(gk) * ld + gr);
          r[i * TL::KV + j] = v;
        }
      }
    }
  }

  __device__ void store(T* __restrict__ S, int tid) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < DW / 4; ++i) {
        const int c = tid + NT * i;
        const int row = c >> 3, kc = c & 7;
        *reinterpret_cast<uint4*>(S + row * TL::PITCH + kc * TL::KV) =
            make_uint4(r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < UPT; ++i) {
        const int u = tid + NT * i;
        const int kb = u / UPK, rc = u % UPK;
        const uint32_t* d = r + i * TL::KV;
        if constexpr (sizeof(T) == 2) {
          // d[j] packs (row 2rc, row 2rc+1) at k = 8kb + j; transpose to two
          // 16-byte rows of 8 consecutive k.
          uint4 lo, hi;
          lo.x = (d[0] & 0xffffu) | (d[1] << 16); hi.x = (d[0] >> 16) | (d[1] & 0xffff0000u);
          lo.y = (d[2] & 0xffffu) | (d[3] << 16); hi.y = (d[2] >> 16) | (d[3] & 0xffff0000u);
          lo.z = (d[4] & 0xffffu) | (d[5] << 16); hi.z = (d[4] >> 16) | (d[5] & 0xffff0000u);
          lo.w = (d[6] & 0xffffu) | (d[7] << 16); hi.w = (d[6] >> 16) | (d[7] & 0xffff0000u);
          *reinterpret_cast<uint4*>(S + (2 * rc) * TL::PITCH + kb * 8) = lo;
          *reinterpret_cast<uint4*>(S + (2 * rc + 1) * TL::PITCH + kb * 8) = hi;
        } else {
          *reinterpret_cast<uint4*>(S + rc * TL::PITCH + kb * 4) = make_uint4(d[0], d[1], d[2], d[3]);
        }
      }
    }
  }
};

template <typename T>
__device__ __forceinline__ void store4(T* p, const float* v, bool vec, int nvalid) {
  if (vec) {
    if constexpr (sizeof(T) == 2) {
      uint2 w;
      w.x = pack_bf16(v[0], v[1]);
      w.y = pack_bf16(v[2], v[3]);
      *reinterpret_cast<uint2*>(p) = w;
    } else {
      *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    }
  } else {
    for (int r = 0; r < nvalid; ++r) p[r] = from_f<T>(v[r]);
  }
}

template <typename T>
__device__ __forceinline__ void load4(const T* p, float* v, bool vec, int nvalid) {
  if (vec) {
    if constexpr (sizeof(T) == 2) {
      uint2 w = *reinterpret_cast<const uint2*>(p);
      v[0] = bf2f(w.x & 0xffff); v[1] = bf2f(w.x >> 16); v[2] = bf2f(w.y & 0xffff); v[3] = bf2f(w.y >> 16);
    } else {
      float4 w = *reinterpret_cast<const float4*>(p);
      v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
    }
  } else {
    for (int r = 0; r < 4; ++r) v[r] = r < nvalid ? to_f<T>(p[r]) : 0.f;
  }
}

// Epilogue of one 4-wide output fragment: v[r] = C[m][nb + r] before the op.
template <typename T, int EPI>
__device__ __forceinline__ void epilogue4(const GemmArgs& g, int m, int nb, float* v, bool ld_vec) {
  const int nvalid = min(4, g.N - nb);
  const bool vec = ld_vec && nvalid == 4;
  const int64_t off = static_cast<int64_t>(m) * g.ldc + nb;
  if constexpr (EPI == EPI_STORE) {
    store4<T>(static_cast<T*>(g.C) + off, v, vec, nvalid);
  } else if constexpr (EPI == EPI_STORE_F32) {
    store4<float>(static_cast<float*>(g.C) + off, v, vec, nvalid);
  } else if constexpr (EPI == EPI_ACC_F32) {
    float o[4];
    load4<float>(static_cast<const float*>(g.C) + off, o, vec, nvalid);
    for (int r = 0; r < 4; ++r) v[r] += o[r];
    store4<float>(static_cast<float*>(g.C) + off, v, vec, nvalid);
  } else if constexpr (EPI == EPI_BIAS) {
    float b[4];
    load4<T>(static_cast<const T*>(g.bias) + nb, b, nvalid == 4, nvalid);
    for (int r = 0; r < 4; ++r) v[r] += b[r];
    store4<T>(static_cast<T*>(g.C) + off, v, vec, nvalid);
  } else if constexpr (EPI == EPI_BIAS_GELU) {
    float b[4], gv[4];
    load4<T>(static_cast<const T*>(g.bias) + nb, b, nvalid == 4, nvalid);
    for (int r = 0; r < 4; ++r) {
      // g = GELU(u) of the stored (rounded) u, so the backward sees the same u.
      const float u = to_f<T>(from_f<T>(v[r] + b[r]));
      v[r] = u;
      gv[r] = gelu_f(u);
    }
    const int64_t aoff = static_cast<int64_t>(m) * g.ldaux + nb;
    store4<T>(static_cast<T*>(g.aux) + aoff, v, vec && (g.ldaux & 3) == 0, nvalid);
    store4<T>(static_cast<T*>(g.C) + off, gv, vec, nvalid);
  } else if constexpr (EPI == EPI_BIAS_RESID) {
    float b[4], x[4];
    load4<T>(static_cast<const T*>(g.bias) + nb, b, nvalid == 4, nvalid);
    load4<float>(g.resid + off, x, vec, nvalid);
    for (int r = 0; r < 4; ++r) v[r] = x[r] + (v[r] + b[r]);
    store4<float>(static_cast<float*>(g.C) + off, v, vec, nvalid);
  } else if constexpr (EPI == EPI_GELU_BWD) {
    float u[4];
    const int64_t aoff = static_cast<int64_t>(m) * g.ldaux + nb;
    load4<T>(static_cast<const T*>(g.aux) + aoff, u, vec && (g.ldaux & 3) == 0, nvalid);
    for (int r = 0; r < 4; ++r) v[r] *= gelu_grad_f(u[r]);
    store4<T>(static_cast<T*>(g.C) + off, v, vec, nvalid);
  }
}

// One output tile per workgroup (blockIdx.x), one k range per split
// (blockIdx.y).  With splits > 1 the raw fp32 sums go to the workspace
// ws[split][M][N] and splitk_reduce applies the epilogue.
template <typename T, bool AKC, bool BKC, int EPI, class CF>
__global__ void __launch_bounds__(CF::NT) gemm_kernel(GemmArgs g) {
  using TL = Tile<T>;
  constexpr int BM = CF::BS, BN = CF::BS, NT = CF::NT;
  __shared__ __attribute__((aligned(16))) T As[2][BM * TL::PITCH];
  __shared__ __attribute__((aligned(16))) T Bs[2][BN * TL::PITCH];

  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wm = w / CF::W, wn = w % CF::W;

  // Tile order: XCD-aware remap (consecutive ids go round-robin over the 8
  // XCDs, so give each XCD a contiguous range), then groups of 8 row-tiles
  // sweeping the columns.
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int total = tiles_m * tiles_n;
  int pid = blockIdx.x;
  if ((total & 7) == 0) pid = (pid & 7) * (total >> 3) + (pid >> 3);
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int first_m = (pid / per_group) * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  const int pid_m = first_m + (pid % per_group) % gsize;
  const int pid_n = (pid % per_group) / gsize;
  const int m0 = pid_m * BM, n0 = pid_n * BN;

  const T* __restrict__ A = static_cast<const T*>(g.A);
  const T* __restrict__ B = static_cast<const T*>(g.B);

  const int nk_all = (g.K + TL::BK - 1) / TL::BK;
  const int per_split = (nk_all + gridDim.y - 1) / gridDim.y;
  const int kt0 = blockIdx.y * per_split;
  const int kt1 = min(nk_all, kt0 + per_split);

  Loader<T, AKC, BM, NT> la;
  Loader<T, BKC, BN, NT> lb;
  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // operands that are not k-contiguous load tiles wholly inside the operand
  // without bounds checks (measured: no gain for k-contiguous ones)
  const bool kfull = g.K % TL::BK == 0;
  const bool afast = !AKC && kfull && m0 + BM <= g.M, bfast = !BKC && kfull && n0 + BN <= g.N;
  la.init(g.lda, tid);
  lb.init(g.ldb, tid);
  auto load_a = [&](int k0) {
    if (afast) la.load_fast(A, g.lda, m0, k0);
    else la.load(A, g.lda, g.M, g.K, m0, k0, tid);
  };
  auto load_b = [&](int k0) {
    if (bfast) lb.load_fast(B, g.ldb, n0, k0);
    else lb.load(B, g.ldb, g.N, g.K, n0, k0, tid);
  };
  if (kt0 < kt1) {
    load_a(kt0 * TL::BK);
    load_b(kt0 * TL::BK);
    la.store(As[0], tid);
    lb.store(Bs[0], tid);
  }
  __syncthreads();

  for (int kt = kt0; kt < kt1; ++kt) {
    const int cur = (kt - kt0) & 1;
    const bool more = kt + 1 < kt1;
    if (more) {
      load_a((kt + 1) * TL::BK);
      load_b((kt + 1) * TL::BK);
    }
    const T* as = As[cur] + (wm * TM * 16 + lr) * TL::PITCH + lg * 8;
    const T* bs = Bs[cur] + (wn * TN * 16 + lr) * TL::PITCH + lg * 8;
#pragma unroll
    for (int s = 0; s < TL::NSLICE; ++s) {
      Frag<T> fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) frag_load(fa[i], as + i * 16 * TL::PITCH + s * 32);
#pragma unroll
      for (int j = 0; j < TN; ++j) frag_load(fb[j], bs + j * 16 * TL::PITCH + s * 32);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) mfma16(acc[i][j], fb[j], fa[i]);
    }
    if (more) {
      la.store(As[cur ^ 1], tid);
      lb.store(Bs[cur ^ 1], tid);
    }
    __syncthreads();
  }

  // acc[i][j][r] = C[m][nb + r]
  if (gridDim.y > 1) {
    float* ws = g.ws + static_cast<int64_t>(blockIdx.y) * g.M * g.N;
    const bool vec_ws = (g.N & 3) == 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + (wm * TM + i) * 16 + lr;
      if (m >= g.M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int nb = n0 + (wn * TN + j) * 16 + lg * 4;
        if (nb >= g.N) continue;
        const int nvalid = min(4, g.N - nb);
        float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
        store4<float>(ws + static_cast<int64_t>(m) * g.N + nb, v, vec_ws && nvalid == 4, nvalid);
      }
    }
    return;
  }
  const bool ld_vec = (g.ldc & 3) == 0;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + (wm * TM + i) * 16 + lr;
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int nb = n0 + (wn * TN + j) * 16 + lg * 4;
      if (nb >= g.N) continue;
      float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      epilogue4<T, EPI>(g, m, nb, v, ld_vec);
    }
  }
}

// Sum of the split partials in split order, then the epilogue.
template <typename T, int EPI>
__global__ void __launch_bounds__(256) splitk_reduce(GemmArgs g, int splits) {
  const int64_t MN = static_cast<int64_t>(g.M) * g.N;
  const int64_t q = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (q >= MN) return;
  const int m = static_cast<int>(q / g.N);
  const int nb = static_cast<int>(q % g.N);
  if ((g.N & 3) == 0) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < splits; ++s) {
      const float4 p = *reinterpret_cast<const float4*>(g.ws + s * MN + q);
      v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
    }
    epilogue4<T, EPI>(g, m, nb, v, (g.ldc & 3) == 0);
  } else {
    for (int e = 0; e < 4 && q + e < MN; ++e) {
      const int mm = static_cast<int>((q + e) / g.N), nn = static_cast<int>((q + e) % g.N);
      float v[4] = {0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < splits; ++s) v[0] += g.ws[s * MN + q + e];
      GemmArgs g1 = g;
      g1.N = nn + 1;  // one valid column at nn
      epilogue4<T, EPI>(g1, mm, nn, v, false);
    }
  }
}

// Output tiles of bs x bs.
int tiles_of(const GemmArgs& g, int bs) { return ((g.M + bs - 1) / bs) * ((g.N + bs - 1) / bs); }

template <typename T>
hipError_t launch_reduce(const GemmArgs& g, int epi, int splits, hipStream_t s) {
  const int64_t MN = static_cast<int64_t>(g.M) * g.N;
  dim3 rgrid(static_cast<unsigned>((MN + 1023) / 1024)), rblock(256);
  switch (epi) {
#define ATOM_CASE(E) \
  case E: hipLaunchKernelGGL((splitk_reduce<T, E>), rgrid, rblock, 0, s, g, splits); break;
    ATOM_CASE(EPI_STORE)
    ATOM_CASE(EPI_STORE_F32)
    ATOM_CASE(EPI_ACC_F32)
    ATOM_CASE(EPI_BIAS)
    ATOM_CASE(EPI_BIAS_GELU)
    ATOM_CASE(EPI_BIAS_RESID)
    ATOM_CASE(EPI_GELU_BWD)
#undef ATOM_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, bool AKC, bool BKC, class CF>
hipError_t launch_cfg(const GemmArgs& g, int epi, int splits, hipStream_t s) {
  dim3 grid(tiles_of(g, CF::BS), splits), block(CF::NT);
  switch (epi) {
#define ATOM_CASE(E) \
  case E: hipLaunchKernelGGL((gemm_kernel<T, AKC, BKC, E, CF>), grid, block, 0, s, g); break;
    ATOM_CASE(EPI_STORE)
    ATOM_CASE(EPI_STORE_F32)
    ATOM_CASE(EPI_ACC_F32)
    ATOM_CASE(EPI_BIAS)
    ATOM_CASE(EPI_BIAS_GELU)
    ATOM_CASE(EPI_BIAS_RESID)
    ATOM_CASE(EPI_GELU_BWD)
#undef ATOM_CASE
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits == 1) return e;
  return launch_reduce<T>(g, epi, splits, s);
}

// The direct-load kernel (gemm_dl.h) takes problems whose 16-byte chunks are
// whole: k, leading dimensions and the row count of an operand that is not
// k-contiguous multiples of a chunk, and output rows (and the saved
// pre-activation's) of whole 4-vectors.
bool dl_applies(const GemmArgs& g, int esz, bool akc, bool bkc, int epi) {
  const int e = 16 / esz;
  const bool aux = epi == EPI_BIAS_GELU || epi == EPI_GELU_BWD;
  return g.K > 0 && g.K % e == 0 && g.lda % e == 0 && g.ldb % e == 0 && (akc || g.M % e == 0) && (bkc || g.N % e == 0) &&
         g.N % 4 == 0 && g.ldc % 4 == 0 && (!aux || g.ldaux % 4 == 0);
}

// What a problem runs as: the direct-load kernel's tile and its split over k,
// or (staged) the register-staged kernel's.
struct Choice {
  int bm, bn, splits;
  bool staged;
};

// Tile configurations with the times the choice rests on, in us: a CU's time
// for one k tile (32) of one workgroup, for a workgroup's start and its
// epilogue (to the element type; epi: what fp32 stores, fp32 read and written,
// GELU forward and GELU backward take more), and once per call.  Fitted to
// 18686 problems in bf16 and 11450 in fp32 (sizes 64 to 16384, every layout
// and epilogue) x every tile and split that fits, on one machine, for the
// smallest loss against the best of them, above all where a single 256x256 or
// register-staged 128x128 tile would win: 0.8 and 0.5 % on average (with no
// epilogue terms 2 and 1.8 %, short k lost most: 14824x12136x384 187 us in
// 256x256 tiles, 234 in 128x128).  What they say: big tiles read the least per
// FLOP, 192 or 128 columns where 256 divide N badly (16384x768x3072: 78 -> 75
// us; 2048x5120x15360: 310 -> 273; 1000x8192x2048: 54 -> 40), 128x128 and 64x64
// where there are too few big tiles for 256 CUs (1000x2048x8192: 157 -> 61, 44
// split in two; 520x768x3072: 65 -> 17).
struct TileCfg {
  int bm, bn, occ;  // occ: workgroups a CU holds
  double ktile, fixed, epi[4], call;
};
constexpr TileCfg BF16_TILES[] = {{256, 256, 1, 0.604, 8.93, {3.26, 10.96, 7.39, 18.10}, 0.70},
                                  {256, 192, 1, 0.486, 7.82, {1.66, 7.20, 8.13, 13.97}, 1.89},
                                  {256, 128, 1, 0.412, 5.52, {1.34, 5.36, 4.31, 6.24}, 0.80},
                                  {128, 128, 2, 0.249, 1.74, {0.63, 2.11, 1.82, 2.08}, 2.10},
                                  {64, 64, 4, 0.131, 0.437, {0.255, 0.358, 0.373, 0.371}, 1.58}};
// fp32: the matrix cores bound both direct-load tiles (512 and 128 MFMAs of 32
// cycles per k tile); 64x64 is 5-10 % faster where it fills the chip.  The
// register-staged 128x128 tile up to 256 k, where stores and starts dominate
// (5020x1524x136: 44 -> 30 us; from there on it loses, and its one set of
// accumulators sums more than 64 MFMAs in a row).
constexpr TileCfg F32_TILES[] = {{64, 64, 2, 0.554, 1.138, {0.034, 0.195, 0.316, 0.443}, 2.93},
                                 {32, 32, 4, 0.157, 0.353, {0.023, 0.048, 0.08, 0.169}, 2.90}};
constexpr TileCfg F32_STAGED = {128, 128, 2, 2.258, 3.0, {-0.13, 3.88, 4.12, 6.15}, 5.12};
constexpr int STAGED_MAX_K = 256;
// A split over k: the second kernel's launch, every partial written and read
// once, its epilogue as above, and per range.
struct SplitCost {
  double fixed, per_partial, epi[3], range;
};
constexpr SplitCost BF16_SPLIT = {2.86, 0.661e-6, {0.694e-6, 1.491e-6, 1.041e-6}, 0.315};
constexpr SplitCost F32_SPLIT = {2.1, 0.257e-6, {1.404e-6, 1.689e-6, 3.692e-6}, 0.0};
constexpr int MAX_SPLITS = 16, CUS = 256;

// Ranges of k that an fp32 result of bf16 operands is at least the sum of, so
// that its rounding error stays that of 256-row tiles split until 192
// workgroups run, or of 128-row tiles split into ranges of 1024 k (a sum takes
// k / 32 MFMAs in a row: 1.5e-7 relative at 512 k and 3.1e-7 at 2560).  Other
// results round to bf16, 1.7e-3.
int min_ranges(const GemmArgs& g, int esz, int epi) {
  if (esz != 2 || !g.ws || (epi != EPI_STORE_F32 && epi != EPI_ACC_F32)) return 1;
  const int t256 = tiles_of(g, 256), t128 = tiles_of(g, 128);
  if (t256 >= 192) return 1;
  const int64_t held = static_cast<int64_t>(g.ws_bytes) / (static_cast<int64_t>(g.M) * g.N * 4);
  const int most = static_cast<int>(std::min<int64_t>(held, MAX_SPLITS));
  int n = 1;
  const bool whole = (g.M | g.N) % 8 == 0;
  while (whole && 2 * n <= most && t256 * n < 192 && g.K % (256 * n) == 0) n *= 2;
  if (n > 1 && t256 * n >= 96) return n;
  if (t128 >= 2 * CUS || g.K < 2048) return 1;
  return std::max(1, std::min({(2 * CUS + t128 - 1) / t128, g.K / 1024, most}));
}

// The configuration and split count with the smallest predicted time.
Choice choose(const GemmArgs& g, int esz, bool akc, bool bkc, int epi) {
  const int quads = (g.K + 127) / 128, least = min_ranges(g, esz, epi);
  const double mn = static_cast<double>(g.M) * g.N;
  const SplitCost& sc = esz == 2 ? BF16_SPLIT : F32_SPLIT;
  // index into epi[], -1: to the element type
  const int e = epi == EPI_STORE_F32 ? 0 : epi == EPI_ACC_F32 || epi == EPI_BIAS_RESID ? 1 : epi == EPI_BIAS_GELU ? 2
              : epi == EPI_GELU_BWD ? 3 : -1;
  Choice best{0, 0, 1, false};
  double best_t = 0.0;
  auto consider = [&](const TileCfg& c, bool staged) {
    if (c.bm == 256 && c.bn < 256 && !gemm_main_combo(akc, bkc, epi)) return;
    const int64_t tiles = static_cast<int64_t>((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn);
    for (int want = 1; want <= (staged ? 1 : MAX_SPLITS); ++want) {
      const int per = (quads + want - 1) / want, splits = (quads + per - 1) / per;
      if (splits != want) continue;
      if (want > 1 && (!g.ws || mn * want * 4 > static_cast<double>(g.ws_bytes))) break;
      // two groups of 128 k per range at least, and no more ranges than fill the chip twice
      if (want > least && want > 1 && (per < 2 || tiles * want > 2 * CUS * c.occ)) break;
      // the most workgroups a CU gets
      const double share = static_cast<double>((tiles * want + CUS - 1) / CUS);
      const int ktiles = want > 1 ? 4 * per : (g.K + 31) / 32, ke = want > 1 ? 0 : e;
      double t = share * (ktiles * c.ktile + c.fixed + (ke >= 0 ? c.epi[ke] : 0.0)) + c.call;
      if (want > 1)
        t += sc.fixed + mn * (sc.per_partial * want + (e > 0 ? sc.epi[e - 1] : 0.0)) + sc.range * want;
      if (want < least) t += 1e9;  // only where nothing reaches the ranges asked for
      if (best.bm == 0 || t < best_t) {
        best = Choice{c.bm, c.bn, want, staged};
        best_t = t;
      }
    }
  };
  if (esz == 2) {
    for (const auto& c : BF16_TILES) consider(c, false);
  } else {
    for (const auto& c : F32_TILES) consider(c, false);
    if (g.K <= STAGED_MAX_K) consider(F32_STAGED, true);
  }
  return best;
}

// The register-staged kernel's choice: 128x128 tiles, split over k where those
// leave the CUs idle and k is long, limited by the workspace; in bf16 256x256
// tiles from one per CU on while a round of them (one per CU) takes less than
// the rounds of 128x128 tiles (two per CU) it stands for.  A round takes 1.85
// times as long at small k, towards 1.9, 1.45 and 1.27 times at large k with
// two, one and no k-contiguous operand (transposing into LDS costs the 128x128
// tile most).  1792 problems with t256 >= 256: 3428x8096x896 neither
// k-contiguous 113 -> 79 us, 4096x50258x4096 both 2279 -> 1912; 15699x7318x128
// 260 in 256x256, 248 in 128x128.
Choice choose_staged(const GemmArgs& g, int esz, bool akc, bool bkc) {
  const int t256 = tiles_of(g, 256), tiles = tiles_of(g, 128);
  if (esz == 2 && t256 >= CUS) {
    const double far = akc && bkc ? 1.9 : akc || bkc ? 1.45 : 1.27;
    const double ratio = far + (1.85 - far) * 256 / (g.K + 256);
    if ((t256 + CUS - 1) / CUS * ratio < (tiles + 2 * CUS - 1) / (2 * CUS)) return Choice{256, 256, 1, true};
  }
  const int bk = ROW_BYTES / esz, nk = (g.K + bk - 1) / bk;
  int splits = 1;
  if (g.ws && tiles < 2 * CUS && nk >= 32) {
    splits = std::min((2 * CUS + tiles - 1) / tiles, nk / 16);
    const int64_t per = static_cast<int64_t>(g.M) * g.N * 4;
    splits = static_cast<int>(std::min<int64_t>(splits, static_cast<int64_t>(g.ws_bytes / per)));
    splits = std::max(1, std::min(splits, 16));
  }
  return Choice{128, 128, splits, true};
}

Choice choice_of(const GemmArgs& g, int esz, bool akc, bool bkc, int epi) {
  return dl_applies(g, esz, akc, bkc, epi) ? choose(g, esz, akc, bkc, epi) : choose_staged(g, esz, akc, bkc);
}

// Whether the direct-load kernel stores an fp32 result past the caches: it
// overflows them (STREAM_BYTES; logits of a head chunk), and its rows are whole
// 128-byte lines.  Other rows share lines with their neighbours, which cached
// stores merge (fp32 12400 x 5496 with k = 128: 65 us cached, 84 streamed;
// 10144 x 9056: 86 and 84).
bool stream_result(const GemmArgs& g, int epi, int splits) {
  return epi == EPI_STORE_F32 && splits == 1 && g.ldc % 32 == 0 && static_cast<int64_t>(g.M) * g.N * 4 > STREAM_BYTES;
}

template <typename T>
hipError_t launch_dl(GemmArgs g, const Choice& c, bool akc, bool bkc, int epi, hipStream_t s) {
  const int quads = (g.K + 127) / 128;
  g.kquads = (quads + c.splits - 1) / c.splits;
  g.splits = (quads + g.kquads - 1) / g.kquads;  // none empty
  g.stream = stream_result(g, epi, g.splits);
  GemmArgs k = g;
  const int kepi = g.splits > 1 ? EPI_STORE_F32 : epi;
  if (g.splits > 1) {
    k.C = g.ws;
    k.ldc = g.N;
  }
  hipError_t e;
  if constexpr (sizeof(T) == 4)
    e = c.bm == 64 ? gemm_dl_f32_64(k, akc, bkc, kepi, s) : gemm_dl_f32_32(k, akc, bkc, kepi, s);
  else
    e = c.bm == 64    ? gemm_dl_64(k, akc, bkc, kepi, s)
        : c.bm == 128 ? gemm_dl_128(k, akc, bkc, kepi, s)
        : c.bn == 128 ? gemm_dl_256x128(k, akc, bkc, kepi, s)
        : c.bn == 192 ? gemm_dl_192(k, akc, bkc, kepi, s)
                      : gemm_dl_256(k, akc, bkc, kepi, s);
  if (e != hipSuccess || g.splits == 1) return e;
  return launch_reduce<T>(g, epi, g.splits, s);
}

template <typename T, bool AKC, bool BKC>
hipError_t launch_t(const GemmArgs& g, int epi, hipStream_t s) {
  const Choice c = choice_of(g, sizeof(T), AKC, BKC, epi);
  if (!c.staged) return launch_dl<T>(g, c, AKC, BKC, epi, s);
  if constexpr (sizeof(T) == 2)
    if (c.bm == 256) return launch_cfg<T, AKC, BKC, Big>(g, epi, 1, s);
  return launch_cfg<T, AKC, BKC, Small>(g, epi, c.splits, s);
}

}  // namespace

// Shape and alignment rules checked before launch (bounds inside the kernel
// rely on them): K a multiple of 8 (bf16) or 4 (fp32), so a 16-byte k chunk
// is either wholly inside or wholly outside; a k-contiguous operand needs a
// leading dimension that keeps 16-byte chunks aligned; a bf16 operand that is
// not k-contiguous is read as dwords of two rows, so it needs an even row
// count and an even leading dimension; all pointers 16-byte aligned.
hipError_t gemm_check(const GemmArgs& g, int dtype, bool akc, bool bkc) {
  const int kv = dtype == DT_BF16 ? 8 : 4;
  if (g.M < 0 || g.N < 0 || g.K < 0) return hipErrorInvalidValue;
  if (g.K % kv) return hipErrorInvalidValue;
  if (akc ? g.lda % kv : (dtype == DT_BF16 && ((g.lda | g.M) & 1))) return hipErrorInvalidValue;
  if (bkc ? g.ldb % kv : (dtype == DT_BF16 && ((g.ldb | g.N) & 1))) return hipErrorInvalidValue;
  if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B) | reinterpret_cast<uintptr_t>(g.C)) & 15)
    return hipErrorInvalidValue;
  if (akc ? g.lda < g.K : g.lda < g.M) return hipErrorInvalidValue;
  if (bkc ? g.ldb < g.K : g.ldb < g.N) return hipErrorInvalidValue;
  if (g.ldc < g.N) return hipErrorInvalidValue;
  return hipSuccess;
}

hipError_t gemm(const GemmArgs& g, int dtype, bool akc, bool bkc, int epi, hipStream_t s) {
  hipError_t e = gemm_check(g, dtype, akc, bkc);
  if (e != hipSuccess) return e;
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if (dtype == DT_BF16) {
    if (akc && bkc) return launch_t<bf16_t, true, true>(g, epi, s);
    if (akc && !bkc) return launch_t<bf16_t, true, false>(g, epi, s);
    if (!akc && !bkc) return launch_t<bf16_t, false, false>(g, epi, s);
    return launch_t<bf16_t, false, true>(g, epi, s);
  }
  if (akc && bkc) return launch_t<float, true, true>(g, epi, s);
  if (akc && !bkc) return launch_t<float, true, false>(g, epi, s);
  if (!akc && !bkc) return launch_t<float, false, false>(g, epi, s);
  return launch_t<float, false, true>(g, epi, s);
}

}  // namespace atom

// What a product with contiguous operands and rows runs as (tests).
extern "C" void atom_gemm_choice(int dtype, int akc, int bkc, int epi, int M, int N, int K, uint64_t ws_bytes,
                                 int* out) {
  using namespace atom;
  GemmArgs g{};
  g.M = M, g.N = N, g.K = K;
  g.lda = akc ? K : M, g.ldb = bkc ? K : N, g.ldc = g.ldaux = N;
  float some;
  g.ws = ws_bytes ? &some : nullptr;
  g.ws_bytes = ws_bytes;
  const Choice c = choice_of(g, dtype == DT_BF16 ? 2 : 4, akc != 0, bkc != 0, epi);
  out[0] = c.staged, out[1] = c.bm, out[2] = c.bn, out[3] = c.splits;
  out[4] = !c.staged && stream_result(g, epi, c.splits);
}
