// Launchers of the projection kernels that live in files of their own (the
// dispatch in k_gemm.hip chooses among them). epi_vec must be set.
#pragma once
#include "common.h"

// The kernels whose waves split K (k_gemm_wave.hip): the tile (weight rows x
// activation rows) and ring slots per wave for a product, NONE when another
// kernel serves it better. Host only.
struct WavePlan {
  enum Tile { NONE, T16x16, T32x16, T32x32, T32x64, T64x64, GATHER } tile = NONE;
  int slots = 2;
  int bn() const;
  int bm(int w_type) const;
  int waves() const;
};
WavePlan wave_plan(const GemmArgs& a);
void launch_gemm_wave(const GemmArgs& a, const WavePlan& p, hipStream_t s);
