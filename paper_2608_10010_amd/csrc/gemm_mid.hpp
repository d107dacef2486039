// The 128 x 128 tile GEMM on expanded planes (gemm_mid.hip), for gemm.hip's entry points.
#pragma once

#include <cstdint>
#include <hip/hip_runtime.h>

namespace curvefp {

// the operands and the K split (1 or 2) of the 256 x 256 kernel; the same C bit for bit, without its
// partial-sum slots and arrival counters
hipError_t launch_gemm_mid(const char* pa, const char* pb, const int* maxA, const int* maxB, int64_t M, int64_t N,
                           int64_t K, int64_t rta, int64_t rtb, float* c, int64_t ldc, int bias2, int splits,
                           hipStream_t s);

}  // namespace curvefp
