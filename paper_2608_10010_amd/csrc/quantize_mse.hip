// Static-operand scales (Sec. 3.1: weights quantized once pick, among representable powers of two, the
// scale that minimizes the squared reconstruction error).
//
// A block is quantized at each candidate scale a_c + u (a_c ceil-absmax; u = 0, -1, .., -(candidates - 1),
// then 1 .. P - 1 when the level pattern spans P > 1 octaves), each element reconstructed to fp32 exactly
// as the dequantizer does, the squared errors summed in fp64 in index order (each product and sum rounded
// once), and the first candidate with the least sum wins.
//
// One thread per block.  The block is read once (blocks of 32 and 64 stay in registers), evaluated at the
// ceil-absmax scale, and its codes at that scale are written.  A scale below that clips the block's largest
// magnitude to its top level, so its sum is at least that one term: (amax - top)^2 >= best so far rules the
// candidate out before it is evaluated (sums of non-negative terms never fall, rounded or not).  Of normally
// distributed weights four blocks in five stop there.  The (block, candidate) pairs left are collected in LDS
// and shared out over the workgroup's threads, so that a wave evaluates 64 of them and not the few of its own
// blocks; the blocks whose scale moved are written again in the same way.  A scale above the ceil-absmax scale
// clips nothing, so nothing rules it out: every thread evaluates those of its own block, before the others, from
// the registers that hold it (E4C3 with radix 2^(3/4), fp32, 8192 x 8192, blocks of 32, one candidate: 527 us from
// the list, 331 from the registers).
//
// What bounds it: waiting.  4096 x 4096 bf16 to E3C3, blocks of 64: vector instructions (about 32 per element, 83% of
// the lanes active) take 28% of a busy unit's slots and LDS 11%; the two waves of a SIMD wait 70% of their time, for the
// serial fp64 sum of a block, its table lookups, and at the barriers of share_out, where one wave works on the few
// blocks listed.  Four candidates, blocks of 32 / 64 / 512: 132 / 142 / 748 -> 46 / 50 / 155 us.
#include "codec.hpp"
#include "curvefp_internal.hpp"
#include "device_util.hpp"
#include "quantize_rules.hpp"
#include "curvefp_tables.inc"

#include <type_traits>

namespace curvefp {

__constant__ uint32_t g_ms_lut[NUM_FORMATS][QLUT_MAX] = CURVEFP_QLUT_INIT;
__constant__ __attribute__((aligned(16))) uint8_t g_ms_lut8[NUM_FORMATS][QLUT_MAX] = CURVEFP_QLUT8_INIT;
__constant__ uint32_t g_ms_lmax_mant[NUM_FORMATS] = CURVEFP_LMAX_MANT_INIT;
__constant__ uint32_t g_ms_mant[NUM_FORMATS][128] = CURVEFP_QR_MANT_INIT;
__constant__ uint64_t g_ms_sig[NUM_FORMATS][128] = CURVEFP_QR_SIG_INIT;

namespace {

// acc + d * d as two roundings (no fused multiply-add), so the sum is the same everywhere
__device__ __forceinline__ double add_square(double acc, double d) {
#pragma clang fp contract(off)
    const double sq = d * d;
    return acc + sq;
}

// fp32 bits as fp64 (fp32 subnormals are kept: the kernels run with them enabled)
__device__ __forceinline__ double f64_of(uint32_t bits) { return (double)__builtin_bit_cast(float, bits); }

// 32 consecutive elements of a block as loaded
template <bool BF16>
struct Group {
    uint32_t w[BF16 ? 16 : 32];

    __device__ __forceinline__ uint32_t mag(int i) const {
        if (!BF16) return w[i] & 0x7FFFFFFFu;
        return (i & 1) ? w[i >> 1] & 0x7FFF0000u : (w[i >> 1] << 16) & 0x7FFF0000u;
    }
    __device__ __forceinline__ uint32_t sign(int i) const {
        if (!BF16) return w[i] >> 31;
        return (i & 1) ? w[i >> 1] >> 31 : (w[i >> 1] >> 15) & 1u;
    }
    __device__ __forceinline__ uint32_t amax() const {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 32; i++) m = max(m, mag(i));
        return m;
    }
};

// blocks of G elements of a source: along its rows (axis 1) or down its columns (axis 0, consecutive
// threads on consecutive columns)
struct Blocks {
    const void* src;
    int64_t ld, nbr, nb, cols;   // blocks per output row, blocks in all, source columns
    int axis, G;
};

template <bool BF16>
struct BlockAt {
    int64_t first, step;   // source index of element 0, distance of consecutive elements
    int64_t orow, oblk;    // output row, block in it

    __device__ __forceinline__ BlockAt(const Blocks& s, int64_t b) {
        if (s.axis == 1) {
            orow = b / s.nbr;
            oblk = b - orow * s.nbr;
            first = orow * s.ld + oblk * s.G;
            step = 1;
        } else {
            oblk = b / s.cols;
            orow = b - oblk * s.cols;
            first = oblk * s.G * s.ld + orow;
            step = s.ld;
        }
    }
    __device__ __forceinline__ Group<BF16> load(const Blocks& s, int g) const {
        Group<BF16> r;
        if (s.axis == 1) {   // 16-byte aligned: the source and its rows are, and G is a multiple of 32
            const uint4* p = reinterpret_cast<const uint4*>(static_cast<const char*>(s.src) +
                                                            (first + 32 * (int64_t)g) * (BF16 ? 2 : 4));
#pragma unroll
            for (int t = 0; t < (BF16 ? 4 : 8); t++) {
                const uint4 v = p[t];
                r.w[4 * t] = v.x;
                r.w[4 * t + 1] = v.y;
                r.w[4 * t + 2] = v.z;
                r.w[4 * t + 3] = v.w;
            }
        } else if (BF16) {
            const uint16_t* p = static_cast<const uint16_t*>(s.src) + first + 32 * (int64_t)g * step;
#pragma unroll
            for (int i = 0; i < 16; i++)
                r.w[i] = (uint32_t)p[2 * i * step] | ((uint32_t)p[(2 * i + 1) * step] << 16);
        } else {
            const uint32_t* p = static_cast<const uint32_t*>(s.src) + first + 32 * (int64_t)g * step;
#pragma unroll
            for (int i = 0; i < 32; i++) r.w[i] = p[i * step];
        }
        return r;
    }
};

// the tables in LDS
template <class F, bool BF16>
struct Tables {
    using T = typename std::conditional<BF16, uint8_t, uint32_t>::type;
    // the quantizer's table behind one rank-0 entry, so that an index below it clamps there.  bfloat16
    // sources use the one-byte table (their low 16 bits never pass a bucket's decision point)
    T lut[F::QLUT_SIZE + 1];
    uint32_t val0[F::NMAG];               // fp32 bits of each rank's level at scale 0
    uint32_t mant[F::BINARY ? 8 : 128];   // value_bits' tables
    uint64_t sig[F::BINARY ? 8 : 128];

    __device__ __forceinline__ void fill(int fidx, int tid) {
        for (int i = tid; i <= F::QLUT_SIZE; i += 256)
            lut[i] = i == 0 ? (T)(BF16 ? 0u : 0xFFFFu) : BF16 ? (T)g_ms_lut8[fidx][i - 1] : (T)g_ms_lut[fidx][i - 1];
        if (tid < F::NMAG) {
            uint32_t v = 0;
            if (tid > 0) {
                if (F::BINARY) {
                    const int n = tid - F::B;
                    v = ((uint32_t)((n >> F::C) + 127) << 23) | g_ms_mant[fidx][n & (F::K - 1)];
                } else {
                    const uint32_t em = g_ms_mant[fidx][tid];
                    v = ((uint32_t)(((int32_t)em >> 24) + 127) << 23) | (em & 0x7FFFFFu);
                }
            }
            val0[tid] = v;
        }
        if (tid < (F::BINARY ? 8 : 128)) {
            mant[tid] = g_ms_mant[fidx][tid];
            sig[tid] = g_ms_sig[fidx][tid];
        }
    }
};

// scales at which every level is a normal fp32 number, and subnormal magnitudes only reach rank 0
template <class F>
__device__ __forceinline__ bool plain_scale(int a) { return a >= F::A_FAST_MIN && a <= 127 - F::OHI; }

// rank of a magnitude and its reconstruction's fp32 bits at a plain scale
template <class F, bool BF16>
__device__ __forceinline__ uint32_t rank_plain(const Tables<F, BF16>& tb, uint32_t mag, int a23, uint32_t& value) {
    const int32_t yb = (int32_t)mag - a23;
    const int idx = min(max((yb >> 16) - ((127 + F::OZ) << 7) + 1, 0), F::QLUT_SIZE);
    uint32_t rk;
    if (BF16) {
        rk = tb.lut[idx];
    } else {
        const uint32_t e = tb.lut[idx];
        rk = (e >> 16) + ((((uint32_t)yb & 0xFFFFu) > (e & 0xFFFFu)) ? 1u : 0u);
    }
    value = rk != 0 ? tb.val0[rk] + (uint32_t)a23 : 0u;
    return rk;
}

// and at any scale
template <class F, bool BF16>
__device__ __forceinline__ uint32_t rank_any(const Tables<F, BF16>& tb, uint32_t mag, int a, uint32_t& value) {
    if (mag == 0) {
        value = 0;
        return 0;
    }
    int32_t yb = (int32_t)mag - (a << 23);
    if ((mag >> 23) == 0) {   // normalize a subnormal input first
        const int p = 31 - __clz(mag);
        yb = (int32_t)(((uint32_t)(p - 22 - a) << 23) | ((mag << (23 - p)) & 0x7FFFFFu));
    }
    const int idx = min(max((yb >> 16) - ((127 + F::OZ) << 7) + 1, 0), F::QLUT_SIZE);
    uint32_t rk;
    if (BF16) {
        // the scaled magnitude's low 16 bits are zero here too (a bfloat16 significand, shifted up)
        rk = tb.lut[idx];
    } else {
        const uint32_t e = tb.lut[idx];
        rk = (e >> 16) + ((((uint32_t)yb & 0xFFFFu) > (e & 0xFFFFu)) ? 1u : 0u);
    }
    value = value_bits<F>(rk, a, tb.mant, tb.sig);
    return rk;
}

// a group at a plain scale a: its squared errors added to acc in index order (ERR) and its codes stored at
// `out` (CODES; 32 bytes, or 28 packed)
template <class F, bool BF16, bool ERR, bool CODES>
__device__ __forceinline__ void group_plain(const Tables<F, BF16>& tb, const Group<BF16>& g, int a, double& acc,
                                            uint8_t* out) {
    uint32_t wd[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 32; i++) {
        const uint32_t m = g.mag(i);
        uint32_t v;
        const uint32_t rk = rank_plain<F, BF16>(tb, m, a << 23, v);
        // the signs of an element and its reconstruction agree, so magnitudes give the same square
        if (ERR) acc = add_square(acc, f64_of(m) - f64_of(v));
        if (CODES) {
            const uint32_t c = rk | ((rk != 0 ? g.sign(i) : 0u) << F::EC);
            const int bit = (F::PACKED7 ? 7 : 8) * i, d = bit >> 5, sh = bit & 31;
            wd[d] |= c << sh;
            if (F::PACKED7 && sh > 25) wd[d + 1] |= c >> (32 - sh);
        }
    }
    if (CODES) {
        if (!F::PACKED7) {
            uint4* o = reinterpret_cast<uint4*>(out);
            o[0] = make_uint4(wd[0], wd[1], wd[2], wd[3]);
            o[1] = make_uint4(wd[4], wd[5], wd[6], wd[7]);
        } else {
            uint32_t* o = reinterpret_cast<uint32_t*>(out);
#pragma unroll
            for (int d = 0; d < 7; d++) o[d] = wd[d];
        }
    }
}

// the same at any scale, for the rare blocks near the ends of fp32's range: element by element from memory
template <class F, bool BF16, bool ERR, bool CODES>
__device__ __forceinline__ void group_any(const Tables<F, BF16>& tb, const Blocks& s, const BlockAt<BF16>& at, int g,
                                          int a, double& acc, uint8_t* out) {
    uint64_t pending = 0;
    int have = 0, word = 0;
#pragma unroll 1
    for (int i = 0; i < 32; i++) {
        const int64_t e = at.first + (32 * (int64_t)g + i) * at.step;
        const uint32_t w = BF16 ? (uint32_t)static_cast<const uint16_t*>(s.src)[e] << 16
                                : static_cast<const uint32_t*>(s.src)[e];
        const uint32_t m = w & 0x7FFFFFFFu;
        uint32_t v;
        const uint32_t rk = rank_any<F, BF16>(tb, m, a, v);
        if (ERR) acc = add_square(acc, f64_of(m) - f64_of(v));
        if (CODES) {
            pending |= (uint64_t)(rk | ((rk != 0 ? w >> 31 : 0u) << F::EC)) << have;
            have += F::PACKED7 ? 7 : 8;
            if (have >= 32) {
                reinterpret_cast<uint32_t*>(out)[word++] = (uint32_t)pending;
                pending >>= 32;
                have -= 32;
            }
        }
    }
}

// HELD: groups of 32 kept in registers (1, 2: blocks of 32, 64), or 0: any G, read again for each use
template <class F, bool BF16, int HELD>
__global__ __launch_bounds__(256, HELD == 2 ? 2 : 3) void quantize_mse_kernel(Blocks s, int candidates, uint8_t* __restrict__ codes,
                                                           int8_t* __restrict__ scales, int fidx) {
    __shared__ Tables<F, BF16> tb;
    __shared__ double best[256];
    __shared__ uint32_t top_mag[256];   // the block's largest magnitude
    __shared__ int8_t ceil_a[256], best_c[256];
    __shared__ uint8_t list[256];
    __shared__ int count;
    const int tid = (int)threadIdx.x;
    tb.fill(fidx, tid);
    if (tid == 0) count = 0;
    __syncthreads();

    const int64_t b0 = (int64_t)blockIdx.x * 256;
    const bool exists = b0 + tid < s.nb;
    const BlockAt<BF16> at(s, exists ? b0 + tid : b0);
    const int groups = s.G / 32;
    const int64_t grow = (int64_t)groups * s.nbr;   // groups of 32 per output row
    constexpr int GB = F::PACKED7 ? 28 : 32;
    uint8_t* out = codes + (at.orow * grow + at.oblk * groups) * GB;
    // a block from memory at scale a
    auto evaluate = [&](const BlockAt<BF16>& o, int a, double& sum, uint8_t* dst, auto err, auto cod) {
        constexpr bool ERR = decltype(err)::value, CODES = decltype(cod)::value;
        if (plain_scale<F>(a)) {
            for (int g = 0; g < groups; g++)
                group_plain<F, BF16, ERR, CODES>(tb, o.load(s, g), a, sum, dst + (int64_t)g * GB);
        } else {
            for (int g = 0; g < groups; g++)
                group_any<F, BF16, ERR, CODES>(tb, s, o, g, a, sum, dst + (int64_t)g * GB);
        }
    };
    bool live = false;
    double acc = 0.0;
    int first_c = 0;   // the best of candidate 0 and those above it
    if (exists) {
        Group<BF16> held[HELD ? HELD : 1];
        uint32_t amax = 0;
        if (HELD) {
#pragma unroll
            for (int g = 0; g < HELD; g++) held[g] = at.load(s, g);
#pragma unroll
            for (int g = 0; g < HELD; g++) amax = max(amax, held[g].amax());
        } else {
            for (int g = 0; g < groups; g++) amax = max(amax, at.load(s, g).amax());
        }
        const int ac = scale_of<F>(amax, g_ms_lmax_mant[fidx]);
        live = ac != -128 && amax != 0;
        ceil_a[tid] = (int8_t)ac;
        top_mag[tid] = amax;
        if (live && HELD && plain_scale<F>(ac)) {
#pragma unroll
            for (int g = 0; g < HELD; g++) group_plain<F, BF16, true, true>(tb, held[g], ac, acc, out + g * GB);
        } else if (live) {
            evaluate(at, ac, acc, out, std::true_type(), std::true_type());
        } else {   // all zero, or a NaN or infinity: zero codes
            for (int g = 0; g < groups; g++)
                for (int d = 0; d < GB / 4; d++) reinterpret_cast<uint32_t*>(out + (int64_t)g * GB)[d] = 0;
        }
        if (F::PERIOD > 1 && live) {
#pragma unroll 1   // (all in one pass over the elements: the sums and codes together spill, twice the time)
            for (int c = candidates; c < candidates + F::PERIOD - 1; c++) {
                const int a = ac + c - candidates + 1;
                if (a > 127) break;
                double e = 0.0;
                if (HELD && plain_scale<F>(a)) {
#pragma unroll
                    for (int g = 0; g < HELD; g++) group_plain<F, BF16, true, false>(tb, held[g], a, e, nullptr);
                } else {
                    evaluate(at, a, e, nullptr, std::true_type(), std::false_type());
                }
                if (e < acc) {
                    acc = e;
                    first_c = c;
                }
            }
        }
    }
    best[tid] = acc;
    best_c[tid] = (int8_t)first_c;

    auto scale_at = [&](int blk, int c) { return (int)ceil_a[blk] + (c < candidates ? -c : c - candidates + 1); };
    // the threads with `want` put their block on the list, and `work` runs once for each, spread over all
    auto share_out = [&](bool want, auto work) {
        if (want) list[atomicAdd(&count, 1)] = (uint8_t)tid;
        __syncthreads();
        const int n = count;
        if (tid < n) work((int)list[tid]);   // n <= 256
        __syncthreads();
        if (tid == 0) count = 0;
        __syncthreads();
    };
    // sum e of candidate c < candidates against a block's best so far: the first in order with the least sum wins, and
    // the candidates above the ceil-absmax scale come after c
    auto wins = [&](double e, int blk) {
        return e < best[blk] || (F::PERIOD > 1 && e == best[blk] && best_c[blk] >= candidates);
    };
    for (int c = 1; c < candidates; c++) {
        bool want = false;
        if (live) {
            const int a = scale_at(tid, c);
            if (a >= -127) {
                const uint32_t v = value_bits<F>(F::NMAG - 1, a, tb.mant, tb.sig);
                want = wins(add_square(0.0, f64_of(top_mag[tid]) - f64_of(v)), tid);   // a bound on the candidate's sum
            }
        }
        share_out(want, [&](int blk) {
            const BlockAt<BF16> o(s, b0 + blk);
            const int a = scale_at(blk, c);
            double e = 0.0;
            evaluate(o, a, e, nullptr, std::true_type(), std::false_type());
            if (wins(e, blk)) {
                best[blk] = e;
                best_c[blk] = (int8_t)c;
            }
        });
    }
    share_out(live && best_c[tid] != 0, [&](int blk) {
        const BlockAt<BF16> o(s, b0 + blk);
        const int a = scale_at(blk, best_c[blk]);
        uint8_t* dst = codes + (o.orow * grow + o.oblk * groups) * GB;
        double none = 0.0;
        evaluate(o, a, none, dst, std::false_type(), std::true_type());
    });
    if (exists) scales[at.orow * s.nbr + at.oblk] = (int8_t)(live ? scale_at(tid, best_c[tid]) : ceil_a[tid]);
}

template <class F, bool BF16>
hipError_t launch_held(const Blocks& s, int candidates, uint8_t* codes, int8_t* scales, int fidx, hipStream_t st) {
    const dim3 grid((unsigned)((s.nb + 255) / 256));
    // 64 fp32 elements in registers leave one wave per SIMD: slower than reading again, unless every block is evaluated
    // at two scales more (radix 2^(3/4), 8192 x 8192 along the rows: 498 us for 613; down the columns 394 for 321)
    constexpr int HELD64 = BF16 || F::PERIOD > 1 ? 2 : 0;
    if (s.G == 32)
        hipLaunchKernelGGL((quantize_mse_kernel<F, BF16, 1>), grid, dim3(256), 0, st, s, candidates, codes, scales, fidx);
    else if (HELD64 == 2 && s.G == 64 && (BF16 || s.axis == 1))
        hipLaunchKernelGGL((quantize_mse_kernel<F, BF16, HELD64>), grid, dim3(256), 0, st, s, candidates, codes, scales, fidx);
    else
        hipLaunchKernelGGL((quantize_mse_kernel<F, BF16, 0>), grid, dim3(256), 0, st, s, candidates, codes, scales, fidx);
    return hipGetLastError();
}

template <class F>
hipError_t launch_fmt(const Blocks& s, int dtype, int candidates, int fidx, void* codes, int8_t* scales, hipStream_t st) {
    uint8_t* cp = static_cast<uint8_t*>(codes);
    return dtype == 1 ? launch_held<F, true>(s, candidates, cp, scales, fidx, st)
                      : launch_held<F, false>(s, candidates, cp, scales, fidx, st);
}

}  // namespace

hipError_t launch_quantize_mse(const void* src, int dtype, int64_t rows, int64_t cols, int64_t ld, int axis,
                               int format, int block, int candidates, void* codes, int8_t* scales, hipStream_t s) {
    Blocks b;
    b.src = src;
    b.ld = ld;
    b.cols = cols;
    b.axis = axis;
    b.G = block;
    b.nbr = (axis == 1 ? cols : rows) / block;
    b.nb = b.nbr * (axis == 1 ? rows : cols);
    switch (format) {
        case 0: return launch_fmt<FmtE4C3>(b, dtype, candidates, 0, codes, scales, s);
        case 1: return launch_fmt<FmtE5C2>(b, dtype, candidates, 1, codes, scales, s);
        case 2: return launch_fmt<FmtE3C3>(b, dtype, candidates, 2, codes, scales, s);
        case 3: return launch_fmt<FmtE4C3R89>(b, dtype, candidates, 3, codes, scales, s);
        default: return launch_fmt<FmtE4C3R34>(b, dtype, candidates, 4, codes, scales, s);
    }
}

}  // namespace curvefp
