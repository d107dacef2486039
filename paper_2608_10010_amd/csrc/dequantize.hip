// CurveFP reconstruction x_hat = (-1)^s 2^{a_b} r^{e + k/K} (Eq. curvefp-value),
// written as the nearest fp32 value.  With r = 2^{P/Q} the magnitude is 2^{w + f/N},
// w = floor(P n / N), f = P n mod N, N = QK (binary radix: w = e, f = k).
//
// In the normal range the result is exact bit assembly: the fp32 exponent is
// w + a_b and the mantissa is that of fl32(2^{f/N}) (scaling by a power of two
// commutes with rounding there).  Below 2^-126 the 62-bit significand of
// 2^{f/N} is rounded once at the subnormal position.  HBM-bound: one byte (or 7
// bits) and 1/32 scale byte read, four bytes written per element.
#include "curvefp_internal.hpp"
#include "codec.hpp"
#include "device_util.hpp"
#include "curvefp_tables.inc"

#include <cstring>

namespace curvefp {

// compile-time tables (curvefp_tables.inc, written at build time by gen_tables)
__constant__ uint32_t g_mant[NUM_FORMATS][8] = CURVEFP_MANT_INIT;
__constant__ uint64_t g_sig62[NUM_FORMATS][8] = CURVEFP_SIG62_INIT;
// rational radix: per magnitude rank, (w << 24) | mantissa of fl32(2^{f/N}) and floor(2^{f/N} 2^62)
__constant__ uint32_t g_dq_em[NUM_FORMATS][128] = CURVEFP_DQ_EM_INIT;
__constant__ uint64_t g_dq_sig62[NUM_FORMATS][128] = CURVEFP_DQ_SIG62_INIT;

namespace {

// Four consecutive codes (a quad) and 16 bytes of fp32 per lane and step, so that every store of a wave is one
// contiguous kilobyte and can stream past the caches (eight codes per lane wrote 32 bytes in two halves, each
// store with holes, which wants the caches to merge them); U quads per lane, 256 apart, are requested before
// the first is written.  A level's bits at a scale that keeps it a normal number are its bits at scale 0 plus
// the scale in the exponent field: one table lookup and one add; other scales take value_bits.
// HBM-bound: 4000 x 11008 E4C3 51.0 -> 33.1 us (220 MB, 6.7 TB/s: the largest cache takes part), 32768 x 8192
// 275 -> 234 us (5.8 TB/s), 2048 x 4096 E3C3 13.0 -> 8.2 us, 16 x 4096 3.2 -> 2.7 us.  What reads the result next does
// not pay for the streaming stores: fp32 to E5C2 codes, back, and the result to bf16, 4000 x 11008 144.8 -> 138.0 us
// (140.7 with these stores plain), 8192 x 4096 109.5 -> 106.7, 4096 x 14336 196.9 -> 182.5 (195.1).
template <class F, int U>
__global__ __launch_bounds__(256) void dequantize_kernel(const uint8_t* __restrict__ codes,
                                                         const int8_t* __restrict__ scales, uint64_t nquads,
                                                         uint32_t qpr, bool dense, Div32 dqpr, int64_t ld, float* __restrict__ dst,
                                                         int fidx, Div32 dgq) {
    constexpr int TAB = F::BINARY ? 8 : 128;
    __shared__ uint32_t mant[TAB];
    __shared__ uint64_t sig[TAB];
    __shared__ uint32_t val0[F::NMAG];
    uint32_t w[U];
    int a[U];
    auto fetch = [&](uint64_t q0) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint64_t q = q0 + 256u * u;
            if (q >= nquads) break;
            const uint32_t b = (uint32_t)(q >> 3);   // group of 32; its scale is that of block b / (G / 32)
            a[u] = scales[div32(b, dgq)];
            if (!F::PACKED7) {
                w[u] = *reinterpret_cast<const uint32_t*>(codes + q * 4);
            } else {
                // bits [28 j, 28 j + 28) of the group's 28 bytes: the four bytes from 7 j / 2 hold them
                const uint32_t j = (uint32_t)q & 7u;
                uint32_t x;
                __builtin_memcpy(&x, codes + (uint64_t)b * 28 + ((7 * j) >> 1), 4);
                w[u] = (j & 1) ? x >> 4 : x;
            }
        }
    };
    const uint64_t q0 = (uint64_t)blockIdx.x * (256u * U) + threadIdx.x;
    fetch(q0);
    const int t = (int)threadIdx.x;
    if (t < TAB) {
        mant[t] = F::BINARY ? g_mant[fidx][t] : g_dq_em[fidx][t];
        sig[t] = F::BINARY ? g_sig62[fidx][t] : g_dq_sig62[fidx][t];
    }
    if (t < F::NMAG) {
        uint32_t v = 0;
        if (t > 0) {
            const int n = t - F::B;
            const uint32_t em = F::BINARY ? 0u : g_dq_em[fidx][t & 127];
            v = F::BINARY ? ((uint32_t)((n >> F::C) + 127) << 23) | g_mant[fidx][n & (F::K - 1) & 7]
                          : ((uint32_t)(((int32_t)em >> 24) + 127) << 23) | (em & 0x7FFFFFu);
        }
        val0[t] = v;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; u++) {
        const uint64_t q = q0 + 256u * u;
        if (q >= nquads) break;
        int64_t e = (int64_t)q * 4;
        if (!dense) {
            const uint32_t r = div32((uint32_t)q, dqpr);
            e = (int64_t)r * ld + (int64_t)((uint32_t)q - r * qpr) * 4;
        }
        constexpr int CB = F::PACKED7 ? 7 : 8;
        // every level is a normal number at these scales (octaves OZ + 1 .. OHI)
        if (a[u] >= -127 - F::OZ && a[u] <= 127 - F::OHI) {
            const uint32_t a23 = (uint32_t)a[u] << 23;
            uint32_t o[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t c = (w[u] >> (CB * i)) & ((1u << CB) - 1);
                const uint32_t m = c & F::MAG_MASK;
                o[i] = m != 0 ? (val0[m] + a23) | ((c >> F::EC) << 31) : 0u;
            }
            st16<true>(dst + e, o[0], o[1], o[2], o[3]);
        } else {
            // rare: element by element, so that the common path keeps its registers
            uint32_t x = w[u];
#pragma unroll 1
            for (int i = 0; i < 4; i++, x >>= CB)
                dst[e + i] = __builtin_bit_cast(float, a[u] == -128 ? 0x7FC00000u   // poisoned block
                                                                    : value_bits<F>(x & ((1u << CB) - 1), a[u],
                                                                                    mant, sig));
        }
    }
}

template <class F, int U>
void launch_quads(const uint8_t* codes, const int8_t* scales, int64_t rows, int64_t qpr, float* dst, int64_t ld,
                  int fidx, Div32 dgq, hipStream_t s) {
    const int64_t nquads = rows * qpr, blocks = (nquads + 256 * U - 1) / (256 * U);
    // rows without gaps (a single row among them) need no row index, which is 32 bits wide
    const bool dense = rows == 1 || ld == 4 * qpr;
    const uint32_t q = dense ? 1u : (uint32_t)qpr;
    hipLaunchKernelGGL((dequantize_kernel<F, U>), dim3((unsigned)blocks), dim3(256), 0, s, codes, scales,
                       (uint64_t)nquads, q, dense, make_div32(q), ld, dst, fidx, dgq);
}

template <class F>
hipError_t launch_fmt(const void* codes, const int8_t* scales, int64_t outer, int64_t k, int block, float* dst,
                      int64_t ld, int fidx, hipStream_t s) {
    const Div32 dgq = make_div32((uint32_t)(block / 32));
    const int64_t qpr = k / 4;
    // 32-bit quad indices per launch where rows are told apart (two rows or more)
    const int64_t slab = qpr < ((int64_t)1 << 31) ? ((int64_t)1 << 31) / qpr : 1;
    const uint8_t* cp = reinterpret_cast<const uint8_t*>(codes);
    for (int64_t r0 = 0; r0 < outer; r0 += slab) {
        const int64_t nr = outer - r0 < slab ? outer - r0 : slab;
        const uint8_t* cr = cp + (F::PACKED7 ? r0 * (k / 32) * 28 : r0 * k);
        const int8_t* sr = scales + r0 * (k / block);
        // two quads per lane (one and four are within 5% up to 64 M elements), eight from there on, where the
        // output no longer fits the 256 MB cache: 32768 x 8192 E3C3 267 us with two, 230 with eight
        if (nr * qpr >= (int64_t)1 << 24)
            launch_quads<F, 8>(cr, sr, nr, qpr, dst + r0 * ld, ld, fidx, dgq, s);
        else
            launch_quads<F, 2>(cr, sr, nr, qpr, dst + r0 * ld, ld, fidx, dgq, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_dequantize(const void* codes, const int8_t* scales, int format, int64_t outer,
                             int64_t k, int block, float* dst, int64_t ld_dst, hipStream_t s) {
    switch (format) {
        case 0: return launch_fmt<FmtE4C3>(codes, scales, outer, k, block, dst, ld_dst, 0, s);
        case 1: return launch_fmt<FmtE5C2>(codes, scales, outer, k, block, dst, ld_dst, 1, s);
        case 2: return launch_fmt<FmtE3C3>(codes, scales, outer, k, block, dst, ld_dst, 2, s);
        case 3: return launch_fmt<FmtE4C3R89>(codes, scales, outer, k, block, dst, ld_dst, 3, s);
        default: return launch_fmt<FmtE4C3R34>(codes, scales, outer, k, block, dst, ld_dst, 4, s);
    }
}

}  // namespace curvefp
