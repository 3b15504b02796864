// Projection kernels whose wavefronts split K: for products whose output
// tiles are small or few (the fp32 models; the action stage).
//
// A block owns a tile of 16 TN weight rows x 16 TM activation rows, and each
// of its NW waves computes the whole tile over its own part of K: K is cut
// into chunks of 64 bytes per row, chunk c belongs to wave c % NW, and a wave
// loads its fragments straight from global memory into the operand registers
// of the matrix instructions, up to U chunks (all of them, for the action
// stage's short K) in flight at once. No operand passes through LDS and the
// K loop has no barrier: a product costs one or two memory round trips, and
// within a block no operand element is loaded twice. The waves' partial tiles
// are then added in LDS in a fixed order and the epilogue runs once per
// output; what the epilogue reads (bias, old residual, row table, RoPE
// angles) is loaded ahead of the K loop, beside the operands.
#include <algorithm>

#include "gemm_epi.h"
#include "gemm_kernels.h"

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// One 16-byte fragment of a row (E elements from k on), or with VEC false
// (rows whose length, stride or base is not a multiple of 16 bytes) its
// elements one by one, zeros past K.
template <typename T, bool VEC>
__device__ __forceinline__ u32x4 load_frag(const T* row, int k, int K) {
  constexpr int E = 16 / sizeof(T);
  if constexpr (VEC) {
    return *reinterpret_cast<const u32x4*>(row + min(k, K - E));
  } else {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = k + e < K ? (float)row[k + e] : 0.f;
    return __builtin_bit_cast(u32x4, v);
  }
}

// acc += W A^T over one chunk: a lane's 16 bytes of a row are the K elements
// (lane / 16) E .. + E - 1 of the chunk, for both operands. In fp32 the four
// 16 x 16 x 4 instructions take element e of every lane each (any assignment
// of K to instructions is the same sum as long as both operands share it).
template <typename T>
__device__ __forceinline__ f32x4 mma_chunk(u32x4 w, u32x4 x, f32x4 acc) {
  if constexpr (sizeof(T) == 2) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
  } else {
    const f32x4 wf = __builtin_bit_cast(f32x4, w), xf = __builtin_bit_cast(f32x4, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], xf[e], acc, 0, 0, 0);
    return acc;
  }
}

// Planes of the partial tile kept in LDS at once: all NW, or half of them
// (the upper waves hand theirs to the lower ones first) when all would leave
// room for only one block per CU.
constexpr int planes(int nw, int plane_bytes) { return nw * plane_bytes <= 80 * 1024 ? nw : nw / 2; }

// RMS (bf16): the RMSNorm of the activation rows folded into the product
// (a.rms_in): every lane squares the fragments it loads.
template <typename T, int TN, int TM, int NW, int U, int MODE, int RMS, bool VEC>
__global__ void __launch_bounds__(64 * NW) gemm_wave_kernel(GemmArgs a) {
  constexpr int E = 16 / sizeof(T), CK = 4 * E;
  constexpr int BN = 16 * TN, BM = 16 * TM, NT = 64 * NW;
  constexpr int LDC = BN + (BN > 16 ? 4 : 0), PLANE = BM * LDC;
  constexpr int NP = planes(NW, PLANE * 4);
  __shared__ __attribute__((aligned(16))) float red[NP * PLANE];
  __shared__ float rsq[RMS ? NW : 1][RMS ? BM : 1];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bx, by, bz;
  xcd_remap_grouped(bx, by, bz, 8);
  (void)bz;
  const int m0 = bx * BM, n0 = by * BN, K = a.K;
  const T* W = reinterpret_cast<const T*>(a.W);
  const T* A = reinterpret_cast<const T*>(a.A);
  const int lr = lane & 15, lk = (lane >> 4) * E;

  // this lane's fragment rows (clamped into the operands: what a row past
  // the end computes is not stored)
  const T *wrow[TN], *arow[TM];
#pragma unroll
  for (int i = 0; i < TN; ++i) wrow[i] = W + (long)min(n0 + i * 16 + lr, a.N - 1) * a.ldw;
#pragma unroll
  for (int j = 0; j < TM; ++j) arow[j] = A + (long)min(m0 + j * 16 + lr, a.M - 1) * a.lda;

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rs[TM], rs2[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) rs[j] = rs2[j] = 0.f;

  // the epilogue's rows and columns of this thread (vector epilogue)
  constexpr int CPT = BN / 4, RS = NT / CPT, NIT = (BM + RS - 1) / RS;
  const int nc = (tid % CPT) * 4, r0 = tid / CPT;
  int ms[NIT];
  bool ok[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    ms[it] = m0 + r0 + it * RS;
    ok[it] = r0 + it * RS < BM && ms[it] < a.M;
  }
  const bool fin = a.epi_vec && n0 + nc < a.N && ok[0];
  EpiRows<MODE, NIT> epi;

  const int nch = (K + CK - 1) / CK;            // chunks; the last may be short
  const bool tail = VEC && K % CK != 0;
  for (int c0 = wave; c0 < nch; c0 += NW * U) {
    u32x4 wf[U][TN], af[U][TM];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0 + u * NW < nch) {
        const int k = (c0 + u * NW) * CK + lk;
#pragma unroll
        for (int i = 0; i < TN; ++i) wf[u][i] = load_frag<T, VEC>(wrow[i], k, K);
#pragma unroll
        for (int j = 0; j < TM; ++j) af[u][j] = load_frag<T, VEC>(arow[j], k, K);
      }
    }
    if (c0 == wave && fin) epi.load(a, ms, ok, n0 + nc);
    // keep every load of the round ahead of the matrix work
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u * NW;
      if (c < nch) {
        if (tail && c == nch - 1) {
          const bool kok = c * CK + lk < K;
#pragma unroll
          for (int i = 0; i < TN; ++i)
            if (!kok) wf[u][i] = u32x4{0, 0, 0, 0};
#pragma unroll
          for (int j = 0; j < TM; ++j)
            if (!kok) af[u][j] = u32x4{0, 0, 0, 0};
        }
        if constexpr (RMS) {
#pragma unroll
          for (int j = 0; j < TM; ++j) sumsq8(__builtin_bit_cast(bf16x8, af[u][j]), rs[j], rs2[j]);
        }
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j) acc[i][j] = mma_chunk<T>(wf[u][i], af[u][j], acc[i][j]);
      }
    }
  }
  if (wave >= nch && fin) epi.load(a, ms, ok, n0 + nc);   // a wave without a chunk

  // lane holds rows n = 16 i + 4 (lane / 16) + e, column m = 16 j + lane % 16
  auto put = [&](int plane) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
        *reinterpret_cast<f32x4*>(red + plane * PLANE + (j * 16 + lr) * LDC + i * 16 + (lane >> 4) * 4) = acc[i][j];
  };
  if constexpr (RMS) {
    // every activation element of the block's rows was read by exactly one
    // lane: add the four lanes of a row, later the waves in wave order
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      rs[j] += rs2[j];
      rs[j] += __shfl_xor(rs[j], 16);
      rs[j] += __shfl_xor(rs[j], 32);
      if (lane < 16) rsq[wave][j * 16 + lr] = rs[j];
    }
  }
  if constexpr (NP < NW) {
    if (wave >= NP) put(wave - NP);
    __syncthreads();
    if (wave < NP) {
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
          acc[i][j] += *reinterpret_cast<const f32x4*>(red + wave * PLANE + (j * 16 + lr) * LDC + i * 16 + (lane >> 4) * 4);
      put(wave);                                // the plane this wave alone has just read
    }
  } else {
    put(wave);
  }
  __syncthreads();
  auto row_sum = [&](int mr, int nn) {
    f32x4 t = *reinterpret_cast<const f32x4*>(red + mr * LDC + nn);
#pragma unroll
    for (int z = 1; z < NP; ++z) t += *reinterpret_cast<const f32x4*>(red + z * PLANE + mr * LDC + nn);
    if constexpr (RMS) {
      float s = rsq[0][mr];
#pragma unroll
      for (int z = 1; z < NW; ++z) s += rsq[z][mr];
      t = row_scale(t, rsqrtf(s / (float)a.rms_in + a.rms_eps));
    }
    return t;
  };
  if (a.epi_vec) {
    if (!fin) return;
    f32x4 t[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) t[it] = ok[it] ? row_sum(r0 + it * RS, nc) : f32x4{0.f, 0.f, 0.f, 0.f};
    epi.finish(a, t, ms, ok, n0 + nc);
    return;
  }
#pragma unroll 1
  for (int c = tid; c < BM * CPT; c += NT) {
    const int mr = c / CPT, nn = (c % CPT) * 4;
    const f32x4 t = row_sum(mr, nn);
    float v[4] = {t[0], t[1], t[2], t[3]};
    epilogue4<MODE>(a, m0 + mr, n0 + nn, v);
  }
}

template <typename T, int TN, int TM, int NW, int U, int MODE, int RMS, bool VEC>
void launch(const GemmArgs& a, hipStream_t s) {
  dim3 grid((a.M + 16 * TM - 1) / (16 * TM), (a.N + 16 * TN - 1) / (16 * TN), 1);
  hipLaunchKernelGGL((gemm_wave_kernel<T, TN, TM, NW, U, MODE, RMS, VEC>), grid, dim3(64 * NW), 0, s, a);
}

// fp32 tiles: the largest that still gives most CUs a block. 64 x 64 tiles
// are bound by the matrix pipe (an 8-wave block loads 512 bytes and runs
// 8192 multiply-adds per k), smaller ones by the latency of their one or two
// round trips.
template <int MODE>
void launch_f32(const GemmArgs& a, hipStream_t s) {
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  const bool vec = a.K >= 4 && a.K % 4 == 0 && a.lda % 4 == 0 && a.ldw % 4 == 0 && al(a.A) && al(a.W);
  auto blocks = [&](long b) { return ((a.M + b - 1) / b) * ((a.N + b - 1) / b); };
  if (!vec) launch<float, 1, 1, 8, 4, MODE, 0, false>(a, s);
  else if (blocks(64) >= 192) launch<float, 4, 4, 8, 2, MODE, 0, true>(a, s);
  else if (blocks(32) >= 192) launch<float, 2, 2, 8, 4, MODE, 0, true>(a, s);
  else launch<float, 1, 1, 8, 8, MODE, 0, true>(a, s);
}

}  // namespace

void launch_gemm_wave_f32(const GemmArgs& a, hipStream_t s) {
  switch (a.mode) {
    case EPI_STORE: launch_f32<EPI_STORE>(a, s); break;
    case EPI_RESID: launch_f32<EPI_RESID>(a, s); break;
    case EPI_GEGLU: launch_f32<EPI_GEGLU>(a, s); break;
    case EPI_QKV: launch_f32<EPI_QKV>(a, s); break;
    case EPI_EULER: launch_f32<EPI_EULER>(a, s); break;
  }
}
