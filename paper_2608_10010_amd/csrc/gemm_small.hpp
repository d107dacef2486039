// The small-product GEMM (gemm_small.hip): its plan, operands and launch, for gemm.hip's entry points.
#pragma once

#include <cstdint>
#include <hip/hip_runtime.h>

#include "device_util.hpp"

namespace curvefp {

// tile of 16 tm x 16 tn outputs per workgroup of `waves` waves (4 or 8), which take groups of four K blocks
// in turn
struct SmallPlan {
    int tm, tn, waves;
};

// what an operand is read from
constexpr int SRC_CODES8 = 0, SRC_CODES7 = 1, SRC_PLANES = 2;

struct SmallOperand {
    const void* data;        // codes, or planes
    const int8_t* scales;    // codes: block scales [rows][nsb]
    const int* rmax;         // planes: row maxima
    int64_t rows, tiles;     // rows; planes: row tiles of 256
    int fidx;                // format: which expansion table
    int64_t nsb;             // codes: scales per row
    Div32 dgq;               // K block kb has scale kb / (G / 32)
};

// whether an M x N x K product is computed by this path, and how (the same answer, and so the same C,
// for every entry point)
bool small_plan(int64_t M, int64_t N, int64_t K, SmallPlan* p);

hipError_t launch_gemm_small(const SmallPlan& p, int sa, const SmallOperand& A, int sb, const SmallOperand& B,
                             int64_t K, float* c, int64_t ldc, int bias2, hipStream_t s);

}  // namespace curvefp
