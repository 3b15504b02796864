// The large-tile projection kernel (the VLM stage's large products).
//
// Block: 256 weight rows x BM = 32 TM activation rows, eight waves in two
// groups of four, one wave of each group per SIMD; group g holds the
// activation rows g BM / 2 .. of the tile, wave w of it the weight rows 64 w ..
// (wave tile 64 x BM / 2). K advances in steps of 64 through two LDS stages
// filled with the direct loads (one block per CU); rows of 128 bytes, chunk c
// of row r in slot c ^ ((r / 2) % 8).
//
// A K-step is two phases: the weight fragments and the first half of the
// activation fragments, then the second half. A phase is a memory part
// (fragment reads into registers, direct loads for a later K-step, waits) and
// a compute part (matrix instructions on registers only), with a barrier
// after each, and group 1 runs one part behind group 0: while one wave of a
// SIMD computes, the other reads, so that the matrix pipe need not wait for
// LDS. The phases fix when a part of a stage was last read, so its next
// contents are requested right after (weights and first half of step kt + 2
// in the second phase of step kt, the second half of step kt + 1 in its first
// phase) and a wave waits for loads that were issued a whole K-step earlier,
// never for the latest (the kernel this one replaces waited for all loads at
// one barrier per K-step, and both waves of a SIMD read fragments at the same
// time: pi0-shaped gate/up at 6528 rows 850 -> 730 us, MLP down 428 -> 366 us,
// gate/up at 26112 rows 2962 -> 2700 us, on one host each).
//
// What bounds it now: without the direct loads in the loop the gate/up takes
// 584 us, without the fragment reads 627 us, with neither 546 us (1.6 PFLOP/s
// with the clock at ~1.7 GHz: the card's power limit); deeper rings (three
// stages of activations), padded rows and other tile orders change nothing.
#include "gemm_epi.h"
#include "gemm_kernels.h"

namespace {

// End of a memory part: all but the `VM` latest direct loads of this wave
// have landed, its fragments are in registers, then the barrier (without a
// fence, which would wait for every load).
#define PART_END(VM) asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory")

template <int MODE, int TM, bool REG>
__global__ void __launch_bounds__(512) gemm_big_kernel(GemmArgs a) {
  constexpr int TN = 4, BN = 256, BM = 32 * TM, HALF = BM / 2, ROWB = 128;
  constexpr int T0 = (TM + 1) / 2, T1 = TM - T0;        // activation subtiles of the two phases
  constexpr int STAGE = (BN + BM) * ROWB;
  constexpr int LDC = BN + 4;
  constexpr int SMEM = REG || 2 * STAGE > HALF * LDC * 4 ? 2 * STAGE : HALF * LDC * 4;
  // direct loads per wave and K-step: weights, first and second activation
  // half (8 rows each; G1 row groups of the second half: when they do not
  // divide among the waves, some are loaded twice, the same bytes to the same
  // place)
  constexpr int LW = 4, L0 = T0 / 2, G1 = T1 * 4, L1 = (G1 + 7) / 8, LF = LW + L0, LS = L1;
  static_assert(T0 % 2 == 0 && T1 > 0, "first half: whole row groups per wave");
  static_assert(!REG || MODE == EPI_GEGLU || MODE == EPI_STORE, "register epilogue: GeGLU or plain store");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn0 = (wave & 3) * 64, wm0 = (wave >> 2) * HALF;
  int bx, by, bz;
  xcd_remap_grouped(bx, by, bz, 4);
  (void)bz;
  const int n_blk = by * BN, m_blk = bx * BM;
  const int K = a.K, nk = (K + 63) / 64;
  const char* W = reinterpret_cast<const char*>(a.W);
  const char* A = reinterpret_cast<const char*>(a.A);
  const char* Z = reinterpret_cast<const char*>(a.zeros);

  // first row of the 8-row group that this wave's j-th load covers; lane l
  // moves slot l % 8 of row l / 8 of it. Rows past the operands read their
  // last row (what they compute is not stored).
  const int lrow = lane >> 3, slot = lane & 7;
  auto row_w = [&](int j) { return (j * 8 + wave) * 8; };
  auto row_0 = [&](int j) {
    const int g = j * 8 + wave;
    return g < T0 * 2 ? g * 8 : HALF + (g - T0 * 2) * 8;
  };
  auto row_1 = [&](int j) {
    const int g0 = j * 8 + wave, g = g0 < G1 ? g0 : g0 - G1;
    return T0 * 16 + (g < T1 * 2 ? g * 8 : HALF + (g - T1 * 2) * 8);
  };
  auto koff = [&](int r) { return (slot ^ (((r + lrow) >> 1) & 7)) * 16; };      // byte of the row's K-step
  long ow[LW], o0[L0], o1[L1];
#pragma unroll
  for (int j = 0; j < LW; ++j) ow[j] = (long)min(n_blk + row_w(j) + lrow, a.N - 1) * a.ldw * 2 + koff(row_w(j));
#pragma unroll
  for (int j = 0; j < L0; ++j) o0[j] = (long)min(m_blk + row_0(j) + lrow, a.M - 1) * a.lda * 2 + koff(row_0(j));
#pragma unroll
  for (int j = 0; j < L1; ++j) o1[j] = (long)min(m_blk + row_1(j) + lrow, a.M - 1) * a.lda * 2 + koff(row_1(j));
  const bool tail = K % 64 != 0;
  auto load = [&](const char* base, long off, int kt, int r, char* dst) {
    const void* g = base + off + kt * 128;
    if (tail && kt == nk - 1 && kt * 128 + koff(r) >= K * 2) g = Z;              // zeros past K
    __builtin_amdgcn_global_load_lds(g, dst, 16, 0, 0);
  };
  auto issue_first = [&](int kt) {       // weights and the first activation half of step kt
    char* st = smem + (kt & 1) * STAGE;
#pragma unroll
    for (int j = 0; j < LW; ++j) load(W, ow[j], kt, row_w(j), st + row_w(j) * ROWB);
#pragma unroll
    for (int j = 0; j < L0; ++j) load(A, o0[j], kt, row_0(j), st + (BN + row_0(j)) * ROWB);
  };
  auto issue_second = [&](int kt) {
    char* st = smem + (kt & 1) * STAGE;
#pragma unroll
    for (int j = 0; j < L1; ++j) load(A, o1[j], kt, row_1(j), st + (BN + row_1(j)) * ROWB);
  };

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int lr = lane & 15, lq = lane >> 4;
  auto frag = [&](const char* st, int r, int q) {
    return *reinterpret_cast<const bf16x8*>(st + r * ROWB + (((q * 4 + lq) ^ ((r >> 1) & 7)) << 4));
  };

  issue_first(0);
  issue_second(0);
  if (nk > 1) {
    issue_first(1);
    PART_END(LF + LS);
  } else {
    PART_END(LS);
  }
  if (wave >= 4) asm volatile("s_barrier" ::: "memory");     // group 1: one part behind
  bf16x8 wf[2][TN], af[2][T0];
  for (int kt = 0; kt < nk; ++kt) {
    const char* st = smem + (kt & 1) * STAGE;
    const char* sa = st + BN * ROWB;
    // first phase
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int i = 0; i < TN; ++i) wf[q][i] = frag(st, wn0 + 16 * i + lr, q);
#pragma unroll
      for (int j = 0; j < T0; ++j) af[q][j] = frag(sa, wm0 + 16 * j + lr, q);
    }
    if (kt + 1 < nk) {
      issue_second(kt + 1);
      PART_END(LF + LS);                 // this step's second half has landed
    } else {
      PART_END(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < T0; ++j)
#pragma unroll
        for (int i = 0; i < TN; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[q][i], af[q][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    // second phase
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < T1; ++j) af[q][j] = frag(sa, wm0 + T0 * 16 + 16 * j + lr, q);
    if (kt + 2 < nk) {
      issue_first(kt + 2);
      PART_END(LF + LS);                 // the next step's weights and first half have landed
    } else {
      PART_END(LS);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < T1; ++j)
#pragma unroll
        for (int i = 0; i < TN; ++i)
          acc[i][T0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[q][i], af[q][j], acc[i][T0 + j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
  }
  if (wave < 4) asm volatile("s_barrier" ::: "memory");      // the groups have met as many barriers
  if constexpr (REG) {
    f32x4 bias[4];
    reg_bias(a, n_blk + wn0, lane, bias);
    reg_epilogue<MODE, TM>(a, acc, bias, n_blk + wn0, m_blk + wm0, lane);
    return;
  }
  // epilogue through LDS, a group's activation rows at a time
  auto Cs = reinterpret_cast<float (*)[LDC]>(smem);
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
    if (wm0 == HALF * h) {
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
          *reinterpret_cast<f32x4*>(&Cs[16 * j + lr][wn0 + 16 * i + lq * 4]) = acc[i][j];
    }
    __syncthreads();
    if (a.epi_vec) {
      tile_epilogue<MODE, BN, HALF, 512, LDC, 1, 4>(a, &Cs[0][0], m_blk + HALF * h, n_blk, tid);
      continue;
    }
#pragma unroll 1
    for (int c = tid; c < HALF * (BN / 4); c += 512) {
      const int mr = c / (BN / 4), nc = (c % (BN / 4)) * 4;
      const f32x4 t = *reinterpret_cast<const f32x4*>(&Cs[mr][nc]);
      float v[4] = {t[0], t[1], t[2], t[3]};
      epilogue4<MODE>(a, m_blk + HALF * h + mr, n_blk + nc, v);
    }
  }
}

template <int MODE, int TM>
void launch_tm(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.M + 32 * TM - 1) / (32 * TM), (a.N + 255) / 256, 1);
  if constexpr (MODE == EPI_GEGLU || MODE == EPI_STORE) {
    if (reg_epi_ok(a)) {
      hipLaunchKernelGGL((gemm_big_kernel<MODE, TM, true>), grid, dim3(512), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_big_kernel<MODE, TM, false>), grid, dim3(512), 0, s, a);
}

template <int MODE>
void launch_mode(const GemmArgs& a, int bm, hipStream_t s) {
  if (bm == 224) launch_tm<MODE, 7>(a, s);
  else launch_tm<MODE, 8>(a, s);
}

}  // namespace

void launch_gemm_big(const GemmArgs& a, int bm, hipStream_t s) {
  VLA_REQUIRE(a.K > 0, "large tiles need K > 0");
  switch (a.mode) {
    case EPI_STORE: launch_mode<EPI_STORE>(a, bm, s); break;
    case EPI_RESID: launch_mode<EPI_RESID>(a, bm, s); break;
    case EPI_GEGLU: launch_mode<EPI_GEGLU>(a, bm, s); break;
    case EPI_QKV: launch_mode<EPI_QKV>(a, bm, s); break;
    case EPI_EULER: launch_mode<EPI_EULER>(a, bm, s); break;
  }
}
