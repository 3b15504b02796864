// Launchers of the projection kernels that live in files of their own (the
// dispatch in k_gemm.hip chooses among them). epi_vec must be set.
#pragma once
#include "common.h"

// fp32 operands: K split over the waves of a block, any K and strides.
void launch_gemm_wave_f32(const GemmArgs& a, hipStream_t s);
