// Launchers of the projection kernels that live in files of their own (the
// dispatch in k_gemm.hip chooses among them). epi_vec must be set.
#pragma once
#include "common.h"

// The kernels whose waves split K (k_gemm_wave.hip): the tile (weight rows x
// activation rows) and ring slots per wave for a product, NONE when another
// kernel serves it better; gather: rows the direct loads cannot take, loaded
// into registers (no slots). Host only.
struct WavePlan {
  enum Tile { NONE, T16x16, T32x16, T32x32, T32x64, T64x64, T64x32, T16x64 } tile = NONE;
  bool gather = false;
  int slots = 2;
  int nw = 0;                      // waves that split K (0: as the tile has it)
  int bn() const;
  int bm() const;
  int k_step(int w_type) const;    // elements of K per chunk, or that a gathering wave has in flight
  int waves() const;
};
WavePlan wave_plan(const GemmArgs& a);
void launch_gemm_wave(const GemmArgs& a, const WavePlan& p, hipStream_t s);

// The large-tile kernel (k_gemm_big.hip): 256 weight rows x bm (256 or 224)
// activation rows per block, bf16, no K ranges.
void launch_gemm_big(const GemmArgs& a, int bm, hipStream_t s);

// Whether the epilogue may run from the accumulators (reg_epilogue): it needs
// bf16 output, whole 16-column groups, 16-byte aligned output rows and bias,
// and for a plain store no row table, row groups or fp32/bf16 copy.
inline bool reg_epi_ok(const GemmArgs& a) {
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (a.out_type != ET_BF16 || a.N % 16 != 0 || a.ldo % 8 != 0 || !al(a.out) || (a.bias && !al(a.bias))) return false;
  if (a.mode == EPI_GEGLU) return true;
  return a.mode == EPI_STORE && !a.tab && a.row_group <= 0 && !a.out2;
}
