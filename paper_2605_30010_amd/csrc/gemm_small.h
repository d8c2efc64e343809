// Launchers of the GEMM kernels for few rows (gemm_small.hip); the choice between them and the
// persistent kernel is made in gemm_choice.h.
#pragma once
#include "mfma_common.h"

namespace et {

int launch_gemm_wave(const GemmArgs &g, hipStream_t s);      //  64 x  64 tiles, k split over 4 wavefronts
int launch_gemm_strip(const GemmArgs &g, hipStream_t s);     //  64 x  64 tiles, a quadrant per wavefront, k ascending
int launch_gemm_pair64(const GemmArgs &g, hipStream_t s);    // 128 x  64 tiles, k split over 2 or 4 groups of wavefronts
int launch_gemm_pair128(const GemmArgs &g, hipStream_t s);   // 128 x 128 tiles, k split over 2 groups of wavefronts
int launch_gemm_half(const GemmArgs &g, hipStream_t s);      // 256 x 128 tiles, halves of the workgroup alternate

}  // namespace et
