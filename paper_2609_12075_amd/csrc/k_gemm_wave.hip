// Projection kernels whose wavefronts split K: for products of few output
// tiles (the action stage at small batch, the fp32 models).
//
// A block owns a tile of 16 TN weight rows x 16 TM activation rows, and each
// of its NW waves computes the whole tile over its own part of K: K is cut
// into chunks of 128 bytes per row, and chunk c belongs to wave c % NW. The
// waves' partial tiles are added in LDS in a fixed order and the epilogue
// runs once per output. What the epilogue reads (bias, old residual, row
// table, RoPE angles) is loaded ahead of the operands, so that its memory
// round trip runs beside theirs. No K ranges over blocks and so no second
// launch: with one output tile per CU such a product is bound by one or two
// memory round trips plus the launch, not by the matrix pipe.
#include <algorithm>
#include <type_traits>

#include "gemm_epi.h"
#include "gemm_kernels.h"

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// acc += W A^T over 64 bytes of K per row: a lane's 16 bytes of a row are the
// elements (lane / 16) E .. + E - 1 (E per 16 bytes), for both operands. In
// fp32 the four 16 x 16 x 4 instructions take element e of every lane each
// (any assignment of K to instructions is the same sum as long as both
// operands share it).
template <typename T>
__device__ __forceinline__ f32x4 mma16(u32x4 w, u32x4 x, f32x4 acc) {
  if constexpr (sizeof(T) == 2) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
  } else {
    const f32x4 wf = __builtin_bit_cast(f32x4, w), xf = __builtin_bit_cast(f32x4, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], xf[e], acc, 0, 0, 0);
    return acc;
  }
}

// s0 + s1 += the squares of a fragment's 16 bytes
template <typename T>
__device__ __forceinline__ void sumsq16(u32x4 v, float& s0, float& s1) {
  if constexpr (sizeof(T) == 2) {
    sumsq8(__builtin_bit_cast(bf16x8, v), s0, s1);
  } else {
    const f32x4 f = __builtin_bit_cast(f32x4, v);
    s0 = fmaf(f[2], f[2], fmaf(f[0], f[0], s0));
    s1 = fmaf(f[3], f[3], fmaf(f[1], f[1], s1));
  }
}

// The end both kernels share: the waves' partial tiles (lane holds rows n =
// 16 i + 4 (lane / 16) + e of column m = 16 j + lane % 16) are added in LDS
// and the epilogue runs; `red` holds a plane of the tile per wave. The caller
// has loaded the epilogue's operands (epi) for this thread's rows ms (valid
// where ok) when `fin` is set. RMS: rsq[wave][row] receives the waves' sums of
// squares. The barrier is met by every thread of the block.
template <int TN, int TM, int NW>
struct Tile {
  static constexpr int BN = 16 * TN, BM = 16 * TM, NT = 64 * NW;
  static constexpr int LDC = BN + (BN > 16 ? 4 : 0), PLANE = BM * LDC;      // floats
  static constexpr int CPT = BN / 4, RS = NT / CPT, NIT = (BM + RS - 1) / RS;
};

template <int TN, int TM, int NW, int MODE, int RMS>
__device__ __forceinline__ void finish_tile(const GemmArgs& a, f32x4 (&acc)[TN][TM], float (&rs)[TM], float* red, float* rsq,
                                            const EpiRows<MODE, Tile<TN, TM, NW>::NIT>& epi,
                                            const int (&ms)[Tile<TN, TM, NW>::NIT], const bool (&ok)[Tile<TN, TM, NW>::NIT],
                                            bool fin, int m0, int n0, int wave) {
  using G = Tile<TN, TM, NW>;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
  const int nc = (tid % G::CPT) * 4, r0 = tid / G::CPT;
  if constexpr (RMS) {
    // every activation element of the block's rows was read by exactly one
    // lane: add the four lanes of a row here, the waves in wave order below
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      rs[j] += __shfl_xor(rs[j], 16);
      rs[j] += __shfl_xor(rs[j], 32);
      if (lane < 16) rsq[wave * G::BM + j * 16 + lr] = rs[j];
    }
  }
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
      *reinterpret_cast<f32x4*>(red + wave * G::PLANE + (j * 16 + lr) * G::LDC + i * 16 + lq * 4) = acc[i][j];
  __syncthreads();
  auto row_sum = [&](int mr, int nn) {
    f32x4 t = *reinterpret_cast<const f32x4*>(red + mr * G::LDC + nn);
#pragma unroll
    for (int z = 1; z < NW; ++z) t += *reinterpret_cast<const f32x4*>(red + z * G::PLANE + mr * G::LDC + nn);
    if constexpr (RMS) {
      float s = rsq[mr];
#pragma unroll
      for (int z = 1; z < NW; ++z) s += rsq[z * G::BM + mr];
      t = row_scale(t, rsqrtf(s / (float)a.rms_in + a.rms_eps));
    }
    return t;
  };
  if (a.epi_vec) {
    if (!fin) return;
    f32x4 t[G::NIT];
#pragma unroll
    for (int it = 0; it < G::NIT; ++it) t[it] = ok[it] ? row_sum(r0 + it * G::RS, nc) : f32x4{0.f, 0.f, 0.f, 0.f};
    epi.finish(a, t, ms, ok, n0 + nc);
    return;
  }
#pragma unroll 1
  for (int c = tid; c < G::BM * G::CPT; c += G::NT) {
    const int mr = c / G::CPT, nn = (c % G::CPT) * 4;
    const f32x4 t = row_sum(mr, nn);
    float v[4] = {t[0], t[1], t[2], t[3]};
    epilogue4<MODE>(a, m0 + mr, n0 + nn, v);
  }
}

// The end of a tile that one wave computes alone: the epilogue runs from the
// accumulators, four columns of TM rows at a time.
template <int TN, int TM, int MODE, int RMS>
__device__ __forceinline__ void finish_alone(const GemmArgs& a, f32x4 (&acc)[TN][TM], float (&rs)[TM], int m0, int n0) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
  int ms[TM];
  bool ok[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    ms[j] = m0 + 16 * j + lr;
    ok[j] = ms[j] < a.M;
    if constexpr (RMS) {
      // (the four lanes of a row hold its squares between them)
      rs[j] += __shfl_xor(rs[j], 16);
      rs[j] += __shfl_xor(rs[j], 32);
      const float sc = rsqrtf(rs[j] / (float)a.rms_in + a.rms_eps);
#pragma unroll
      for (int i = 0; i < TN; ++i) acc[i][j] = row_scale(acc[i][j], sc);
    }
  }
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    const int n = n0 + 16 * i + 4 * lq;
    if (n >= a.N) continue;
    if (a.epi_vec) {
      epi_rows<MODE, TM>(a, acc[i], ms, ok, n);
      continue;
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      epilogue4<MODE>(a, ms[j], n, v);
    }
  }
}

// The rows of this thread in the vector epilogue; true when it has any.
template <int TN, int TM, int NW>
__device__ __forceinline__ bool my_rows(const GemmArgs& a, int m0, int n0, int (&ms)[Tile<TN, TM, NW>::NIT],
                                        bool (&ok)[Tile<TN, TM, NW>::NIT]) {
  using G = Tile<TN, TM, NW>;
  const int nc = (threadIdx.x % G::CPT) * 4, r0 = threadIdx.x / G::CPT;
#pragma unroll
  for (int it = 0; it < G::NIT; ++it) {
    ms[it] = m0 + r0 + it * G::RS;
    ok[it] = r0 + it * G::RS < G::BM && ms[it] < a.M;
  }
  return a.epi_vec && n0 + nc < a.N && ok[0];
}

// ---------------------------------------------------------------- LDS ring per wave
// Each wave moves its chunks global -> LDS with the direct loads into a ring
// of S slots of its own (R = 16 (TN + TM) rows of 128 bytes; one load covers
// 8 whole rows) and waits on its own loads only: the K loop has no barrier.
// The 16-byte chunk c of row r sits in slot c ^ ((r / 2) % 8), which makes
// the 16-row fragment reads conflict-free. Loading the fragments straight
// into registers instead, without LDS, was measured at a quarter of the load
// rate (~16 bytes a clock per CU: the matrix operand layout puts consecutive
// lanes into different rows, so every lane is a cache line of its own):
// 720 x 1920 by 50 rows 5.9 us against 3.8 us.
// RMS: the RMSNorm of the activation rows folded into the product (a.rms_in);
// every lane squares the fragments that it reads.
template <typename T, int TN, int TM, int NW, int S, int MODE, int RMS>
__global__ void __launch_bounds__(64 * NW) gemm_wave_kernel(GemmArgs a) {
  using G = Tile<TN, TM, NW>;
  constexpr int E = 16 / sizeof(T), CK = 8 * E;          // elements per 16 bytes, per chunk
  constexpr int R = G::BN + G::BM, LOADS = R / 8, SLOT = R * 128, RING = NW * S * SLOT;
  static_assert(NW * G::PLANE * 4 <= RING, "the waves' planes must fit the ring");
  static_assert(S == 1 || S == 2, "the waits below know rings of one or two slots");
  // one LDS object: with a second one the compiler waits for every direct
  // load before each fragment read
  __shared__ __attribute__((aligned(1024))) char smem[RING + (RMS ? NW * G::BM * 4 : 0)];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bx, by, bz;
  xcd_remap_grouped(bx, by, bz, 8);
  (void)bz;
  const int m0 = bx * G::BM, n0 = by * G::BN, K = a.K;
  const T* Z = reinterpret_cast<const T*>(a.zeros);

  int ms[G::NIT];
  bool ok[G::NIT];
  const bool fin = my_rows<TN, TM, NW>(a, m0, n0, ms, ok);
  EpiRows<MODE, G::NIT> epi;
  if (fin) epi.load(a, ms, ok, n0 + (tid % G::CPT) * 4);
  __builtin_amdgcn_sched_barrier(0);

  // load j covers rows 8 j .. 8 j + 7 of the ring slot (weight rows, then
  // activation rows): lane l moves slot l % 8 of row 8 j + l / 8. Rows past
  // the operands read their last row (what they compute is not stored).
  const T* src[LOADS];
  int kof[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int r = j * 8 + (lane >> 3);
    kof[j] = ((lane & 7) ^ ((r >> 1) & 7)) * E;
    src[j] = j * 8 < G::BN ? reinterpret_cast<const T*>(a.W) + (long)min(n0 + r, a.N - 1) * a.ldw
                           : reinterpret_cast<const T*>(a.A) + (long)min(m0 + r - G::BN, a.M - 1) * a.lda;
  }
  char* ring = smem + wave * S * SLOT;
  const int nch = (K + CK - 1) / CK;
  const int per = nch > wave ? (nch - wave + NW - 1) / NW : 0;     // this wave's chunks
  auto issue = [&](int i, int sl) {
    const int kb = (wave + i * NW) * CK;
    char* st = ring + sl * SLOT;
    const bool whole = kb + CK <= K;
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      // 16-byte pieces past K are read from the zero buffer
      const void* g = whole || kb + kof[j] < K ? src[j] + kb + kof[j] : Z;
      __builtin_amdgcn_global_load_lds(g, st + j * 1024, 16, 0, 0);
    }
  };

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rs[TM], rs2[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) rs[j] = rs2[j] = 0.f;
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (i < per) issue(i, i);
  const int lr = lane & 15, lq = lane >> 4;
  for (int i = 0; i < per; ++i) {
    // chunk i has landed once only the next chunk's loads are pending
    if (S == 2 && i + 1 < per) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* st = ring + (i % S) * SLOT;
    u32x4 wf[2][TN], af[2][TM];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = q * 4 + lq;
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int r = 16 * t + lr;
        wf[q][t] = *reinterpret_cast<const u32x4*>(st + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        const int r = G::BN + 16 * t + lr;
        af[q][t] = *reinterpret_cast<const u32x4*>(st + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
      }
    }
    // the fragments are in registers: their slot may be loaded again
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (i + S < per) issue(i + S, i % S);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if constexpr (RMS) {
#pragma unroll
        for (int t = 0; t < TM; ++t) sumsq16<T>(af[q][t], rs[t], rs2[t]);
      }
#pragma unroll
      for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int u = 0; u < TM; ++u) acc[t][u] = mma16<T>(wf[q][t], af[q][u], acc[t][u]);
    }
  }
  __syncthreads();                         // every wave is done with its ring
#pragma unroll
  for (int j = 0; j < TM; ++j) rs[j] += rs2[j];
  finish_tile<TN, TM, NW, MODE, RMS>(a, acc, rs, reinterpret_cast<float*>(smem), reinterpret_cast<float*>(smem + RING),
                                         epi, ms, ok, fin, m0, n0, wave);
}

// ---------------------------------------------------------------- rows of any alignment
// The same product with the fragments loaded straight into registers, U
// 64-byte pieces of K in flight per wave: for rows that the direct loads
// cannot take, and fp32 products of many tiles and short K. bf16: operands whose base is not 16-byte aligned (K and the
// strides are multiples of 8). fp32: rows whose length, stride or base is no
// multiple of 16 bytes; the pieces around the end of K are read element by
// element.
template <typename T, int TN, int TM, int NW, int U, int MODE, int RMS>
__global__ void __launch_bounds__(64 * NW) gemm_gather_kernel(GemmArgs a) {
  using G = Tile<TN, TM, NW>;
  constexpr int E = 16 / sizeof(T), CK = 4 * E;
  constexpr bool ALONE = NW == 1;
  __shared__ __attribute__((aligned(16))) float red[ALONE ? 1 : NW * G::PLANE];
  __shared__ float rsq[RMS && !ALONE ? NW * G::BM : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bx, by, bz;
  xcd_remap_grouped(bx, by, bz, 8);
  (void)bz;
  const int m0 = bx * G::BM, n0 = by * G::BN, K = a.K;
  const int lr = lane & 15, lk = (lane >> 4) * E;
  int ms[G::NIT];
  bool ok[G::NIT];
  const bool fin = !ALONE && my_rows<TN, TM, NW>(a, m0, n0, ms, ok);
  EpiRows<MODE, G::NIT> epi;
  if (fin) epi.load(a, ms, ok, n0 + (tid % G::CPT) * 4);
  const T *wrow[TN], *arow[TM];
#pragma unroll
  for (int i = 0; i < TN; ++i) wrow[i] = reinterpret_cast<const T*>(a.W) + (long)min(n0 + i * 16 + lr, a.N - 1) * a.ldw;
#pragma unroll
  for (int j = 0; j < TM; ++j) arow[j] = reinterpret_cast<const T*>(a.A) + (long)min(m0 + j * 16 + lr, a.M - 1) * a.lda;
  // the lane's E elements from k on, zeros past K: all of them inside (WHOLE),
  // all or none (VECTOR; bf16 always), or one by one
  enum Piece { WHOLE, VECTOR, SINGLE };
  struct __attribute__((packed, aligned(sizeof(T)))) P { u32x4 v; };
  auto frag = [&](const T* row, int k, auto how) {
    if constexpr (how() == WHOLE) {
      return reinterpret_cast<const P*>(row + k)->v;
    } else if constexpr (how() == VECTOR) {
      return k < K ? reinterpret_cast<const P*>(row + k)->v : u32x4{0, 0, 0, 0};
    } else {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = k + e < K ? (float)row[k + e] : 0.f;
      return __builtin_bit_cast(u32x4, v);
    }
  };
  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rs[TM], rs2[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) rs[j] = rs2[j] = 0.f;
  const int nch = (K + CK - 1) / CK;
  for (int c0 = wave; c0 < nch; c0 += NW * U) {
    u32x4 wf[U][TN], af[U][TM];
    auto load = [&](auto how) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = (c0 + u * NW) * CK + lk;
#pragma unroll
        for (int i = 0; i < TN; ++i) wf[u][i] = frag(wrow[i], k, how);
#pragma unroll
        for (int j = 0; j < TM; ++j) af[u][j] = frag(arow[j], k, how);
      }
    };
    // (decided for the wave, so that a short K runs through little code)
    if constexpr (sizeof(T) == 2) load(std::integral_constant<int, VECTOR>{});
    else if ((c0 + (U - 1) * NW + 1) * CK <= K) load(std::integral_constant<int, WHOLE>{});
    else if (K % 4 == 0) load(std::integral_constant<int, VECTOR>{});
    else load(std::integral_constant<int, SINGLE>{});
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (RMS) {
#pragma unroll
        for (int j = 0; j < TM; ++j) sumsq16<T>(af[u][j], rs[j], rs2[j]);
      }
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = mma16<T>(wf[u][i], af[u][j], acc[i][j]);
    }
  }
#pragma unroll
  for (int j = 0; j < TM; ++j) rs[j] += rs2[j];
  if constexpr (ALONE) finish_alone<TN, TM, MODE, RMS>(a, acc, rs, m0, n0);
  else finish_tile<TN, TM, NW, MODE, RMS>(a, acc, rs, red, rsq, epi, ms, ok, fin, m0, n0, wave);
}

// ---------------------------------------------------------------- dispatch
bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <int TN, int TM>
dim3 grid_of(const GemmArgs& a) {
  return dim3((a.M + 16 * TM - 1) / (16 * TM), (a.N + 16 * TN - 1) / (16 * TN), 1);
}

template <typename T, int TN, int TM, int NW, int S, int MODE, int RMS>
void go(const GemmArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((gemm_wave_kernel<T, TN, TM, NW, S, MODE, RMS>), (grid_of<TN, TM>(a)), dim3(64 * NW), 0, s, a);
}

template <typename T, int TN, int TM, int NW, int U, int MODE, int RMS>
void go_gather(const GemmArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((gemm_gather_kernel<T, TN, TM, NW, U, MODE, RMS>), (grid_of<TN, TM>(a)), dim3(64 * NW), 0, s, a);
}

template <typename T, int MODE, int RMS>
void launch(const GemmArgs& a, const WavePlan& p, hipStream_t s) {
  if (p.gather) {
    if constexpr (sizeof(T) == 2) {
      go_gather<T, 1, 4, 8, 4, MODE, RMS>(a, s);
    } else {
      if (p.tile == WavePlan::T16x16) go_gather<T, 1, 1, 8, 4, MODE, RMS>(a, s);
      else if (p.tile == WavePlan::T64x64) go_gather<T, 4, 4, 4, 2, MODE, RMS>(a, s);
      else if (p.tile == WavePlan::T64x32) go_gather<T, 4, 2, 1, 1, MODE, RMS>(a, s);
      else if (p.nw == 1) go_gather<T, 2, 2, 1, 2, MODE, RMS>(a, s);
      else go_gather<T, 2, 2, 4, 4, MODE, RMS>(a, s);
    }
    return;
  }
  switch (p.tile) {
    case WavePlan::T16x16: go<T, 1, 1, 8, 2, MODE, RMS>(a, s); break;
    case WavePlan::T32x16: go<T, 2, 1, 4, 2, MODE, RMS>(a, s); break;
    case WavePlan::T32x32: p.slots == 1 ? go<T, 2, 2, 4, 1, MODE, RMS>(a, s) : go<T, 2, 2, 4, 2, MODE, RMS>(a, s); break;
    case WavePlan::T32x64: go<T, 2, 4, 4, 2, MODE, RMS>(a, s); break;
    case WavePlan::T64x64: go<T, 4, 4, 4, 2, MODE, RMS>(a, s); break;
    case WavePlan::T64x32: case WavePlan::T16x64:        // (gather only)
    case WavePlan::NONE: break;
  }
}

template <int MODE>
void launch_mode(const GemmArgs& a, const WavePlan& p, hipStream_t s) {
  const bool f32 = a.w_type == ET_F32;
  if constexpr (MODE != EPI_RESID) {
    if (a.rms_in) {
      if (f32) launch<float, MODE, 1>(a, p, s);
      else launch<bf16, MODE, 1>(a, p, s);
      return;
    }
  }
  if (f32) launch<float, MODE, 0>(a, p, s);
  else launch<bf16, MODE, 0>(a, p, s);
}

}  // namespace

int WavePlan::bn() const { return tile == T16x16 || tile == T16x64 ? 16 : tile == T64x32 || tile == T64x64 ? 64 : 32; }
int WavePlan::bm() const {
  return tile == T16x16 || tile == T32x16 ? 16 : tile == T32x32 || tile == T64x32 ? 32 : 64;
}
int WavePlan::k_step(int w_type) const {
  const int e = w_type == ET_F32 ? 4 : 8;                  // elements of 16 bytes
  return gather ? 4 * e * (tile == T64x32 ? 1 : tile == T64x64 || nw == 1 ? 2 : 4) : 8 * e;
}
int WavePlan::waves() const { return nw ? nw : tile == T16x16 || tile == T16x64 ? 8 : 4; }

// The tile of an fp32 product whose rows the direct loads cannot take. Few
// output tiles: the waves of a block split K, as below. Many: 64 x 64 tiles
// split K while they fit the CUs and K is long; otherwise each wave computes a
// tile alone (there are waves enough, and a short K is no work to share), 32 x
// 32 or, past five waves a CU, 64 x 32 (fewer reads of an operand row).
// Measured (us; tiles by the number of waves that split K):
//   rows x columns x K   16 x 16/8  32 x 32/4  64 x 64/4  32 x 32/1  64 x 32/1
//   512 x 250 x 501          6.8        8.1       16.6       14.7       29.4
//   1024 x 250 x 501        12.5        8.4       16.8       14.9       29.4
//   1024 x 1000 x 65        18.5       12.1        8.6        7.2        9.1
//   1024 x 1000 x 501       31.2       30.3       16.5       16.6       26.9
//   1024 x 1000 x 2047       116         95         46         64        119
//   2048 x 2048 x 65          64         36         26         18         16
//   2048 x 2048 x 1021       200        212        143        132         96
// (the vector unit's kernel that these replaced: 59, 59, 12.8, 59, 275, 18 and
// 196; none of 700 shapes is over 1.2 us slower than it).
// Rows that the direct loads can take go this way too where K is so short that
// filling 128 KiB of ring a CU is most of the time: past 640 tiles of 32 x 32,
// K to 96, past five a CU to 128 (direct loads / this / the vector unit: 1024 x
// 1000 x 64 7.1 / 6.1 / 10.8, x 128 7.5 / 8.0 / 17; 2048 x 2048 x 8 22 / 9 /
// 9, x 64 22 / 16 / 16, x 128 23.1 / 19.4 / 24, x 256 32 / 30 / 42; 8000 x 1000 x
// 128 42 / 36 / 40, x 256 60 / 60 / 75).
static WavePlan gather_plan_f32(const GemmArgs& a) {
  auto blocks = [&](long bn, long bm) { return ((a.N + bn - 1) / bn) * ((a.M + bm - 1) / bm); };
  constexpr long CUS = 256;
  WavePlan p;
  p.gather = true;
  p.slots = 0;
  if (blocks(16, 16) <= 2 * CUS) p.tile = WavePlan::T16x16;
  else if (blocks(32, 32) <= CUS) p.tile = WavePlan::T32x32;
  else if (a.K > 512 && blocks(64, 64) <= CUS) p.tile = WavePlan::T64x64;
  else p.tile = blocks(32, 32) <= 5 * CUS ? WavePlan::T32x32 : WavePlan::T64x32, p.nw = 1;
  return p;
}

WavePlan wave_plan(const GemmArgs& a) {
  WavePlan p;
  const bool f32 = a.w_type == ET_F32;
  const int per16 = f32 ? 4 : 8;               // elements per 16 bytes
  const bool direct = a.zeros && al16(a.A) && al16(a.W) && a.K % per16 == 0 && a.lda % per16 == 0 && a.ldw % per16 == 0;
  auto blocks = [&](long bn, long bm) { return ((a.N + bn - 1) / bn) * ((a.M + bm - 1) / bm); };
  constexpr long CUS = 256;
  const long t32 = blocks(32, 32);
  if (f32 && (!direct || (t32 > 640 && a.K <= (t32 > 5 * CUS ? 128 : 96)))) return gather_plan_f32(a);
  if (!direct) {
    if (a.M <= 64 && a.zeros) p.tile = WavePlan::T16x64, p.gather = true, p.slots = 0;      // (only what no other kernel takes)
    return p;
  }
  const long row_bytes = (long)a.K * 16 / per16;
  // The smallest tile whose blocks leave no CU a second one. Up to 2 KiB of K
  // per row a 32 x 32 tile takes one ring slot (32 KiB of LDS, so that blocks
  // share CUs) and serves up to 640 blocks. Beyond, the staged tiles that
  // share each operand row among more of a block's waves are faster: time over
  // theirs by blocks, K 720 to 1024, stores, GeGLU and folded norms: to 550
  // 0.74-0.85, to 640 0.92-1.04, to 750 0.93-1.05, to 900 1.07-1.12, over 1200
  // 1.13-1.22. 64 x 64 tiles at such K: 0.98-1.11 of the staged ones' time.
  // (A residual product with a row norm behind it is the exception, since its
  // alternative is K ranges and their reduce: 960 x 960 x 960 with the norm
  // 13.7 us there, 12.4 on 32 x 32 and 11.7 on 64 x 64 tiles.) 256 CUs, though
  // the action stage may share them with a VLM stage: planned for 192, a
  // lockstep of the pi0-shaped VLM stage and the SmolVLA-shaped action stage
  // takes as long (2641 and 2645 us), for 128 or 64 longer (2690, 2697).
  // Measured
  // (us, this kernel against the plans used before it, replayed graph): 50
  // rows, 1600 x 720 3.7 / 6.1, 720 x 960 3.3 / 6.0, 3840 x 720 4.1 / 5.6,
  // 720 x 1920 3.8 / 6.6, 2560 x 1024 4.5 / 7.3, 8192 x 1024 6.1 / 9.3,
  // 1024 x 4096 5.4 / 8.1; 400 rows, 720 x 960 4.9 / 7.2, 1024 x 2048 6.5 /
  // 11.1, 1024 x 4096 11.0 / 14.6; past the limits, 400 rows, 2560 x 1024
  // 10.3 / 10.0, 8192 x 1024 20 / 13.8.
  const bool short_k = row_bytes <= 2048;
  p.slots = 2;
  const bool few_rows = a.M <= 64 && a.N >= 1536;
  if (!f32 && a.K > 4096 && !few_rows) return p;      // long K: K ranges over blocks
  if (blocks(16, 16) <= CUS) p.tile = WavePlan::T16x16;
  else if (blocks(32, 16) <= CUS) p.tile = WavePlan::T32x16;
  else if (blocks(32, 32) <= (short_k ? 640 : CUS)) p.tile = WavePlan::T32x32, p.slots = short_k ? 1 : 2;
  else if (!short_k && blocks(32, 64) <= CUS) p.tile = WavePlan::T32x64;
  else if (f32 || (!short_k && blocks(64, 64) <= CUS)) p.tile = WavePlan::T64x64;
  else if (few_rows) p.tile = WavePlan::T32x64;       // (one row of tiles: nothing to share between blocks)
  return p;
}

void launch_gemm_wave(const GemmArgs& a, const WavePlan& p, hipStream_t s) {
  switch (a.mode) {
    case EPI_STORE: launch_mode<EPI_STORE>(a, p, s); break;
    case EPI_RESID: launch_mode<EPI_RESID>(a, p, s); break;
    case EPI_GEGLU: launch_mode<EPI_GEGLU>(a, p, s); break;
    case EPI_QKV: launch_mode<EPI_QKV>(a, p, s); break;
    case EPI_EULER: launch_mode<EPI_EULER>(a, p, s); break;
  }
}
