// CurveFP GEMM for products whose output is small against the chip: a few rows of activations
// against a weight (decode, short prompts), or small matrices.
//
// The 256 x 256 tiles of gemm.hip leave most compute units idle there (16 rows against a 4096 x 4096
// weight are 16 tiles), and the weight's planes cost five bytes of traffic for every code byte
// although each is used once.  Here a workgroup owns a tile of 16 TM x 16 TN outputs and its waves
// split K between them: wave w takes every W-th group of four K blocks, accumulates its share on
// v_mfma_f32_16x16x32_f16, and the shares are added in LDS in wave order, so the sum does not depend on
// timing and needs neither a workspace nor atomics.  Nothing is staged in LDS but the expansion
// tables: lane l of a fragment is row l % 16, chunk l / 16 of a K block, exactly the 8 codes (or the
// 16-byte chunk of each plane) that the lane loads itself, so operands go from memory to the matrix
// core through registers, several K blocks in flight per wave.
//
// Operands come as codes (8-bit, or E3C3 packed) expanded in registers by the same table and
// multipliers as the planes, or as the planes of a prepared operand.  Both give the same fragments,
// and the order of the sum depends on (M, N, K) alone, so every entry point returns the same C.
//
// What bounds it: from codes the expansion (per 8 codes about 30 vector instructions and 8 LDS gathers, of
// both operands in every tile: 16 x 4096 x 4096 issues a vector instruction in 56% of a busy unit's slots, its waves
// wait for the rest, and filling the table and the first loads take half of the 12 us), from planes the memory:
// 32 x 14336 x 4096 reads 239 MB of them in 35 us (6.9 TB/s).  Measured, weights from HBM,
// 256 x 256 kernel with its preparation -> this one: 16 x 4096 x 4096 E3C3 codes 123 -> 14 us (from planes
// 106 -> 12 us), 32 x 14336 x 4096 E4C3 181 -> 36 us (119 -> 40 us), 128 x 128 x 128 27 -> 6 us.
#include "curvefp_internal.hpp"
#include "gemm_small.hpp"
#include "device_util.hpp"
#include "planes.hpp"
#include "curvefp_tables.inc"

namespace curvefp {

__constant__ uint32_t g_small_dec[NUM_FORMATS][GEMM_DEC_ENTRIES] = CURVEFP_DEC_INIT;

namespace {

constexpr int WMAX = 8;   // waves per workgroup: 4 or 8

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// expansion table in LDS: entry c of lane l at byte 256 c + 4 l, so every lane gathers from its own
// bank and one byte permute forms the address of an 8-bit code
constexpr int LUT_PITCH = 256;
template <bool P7>
constexpr int LUT_ENTRIES = P7 ? 128 : 256;

struct Frag {
    half8 hi, lo;
};

// A workgroup's tile and wave: XCD x (linear id mod 8) takes a contiguous eighth of the column tiles,
// row tiles innermost, so the workgroups that share columns of B share an L2.
struct Place {
    int64_t m0, n0;
    uint32_t cnt;     // K blocks of this wave
    int wave, wlog;   // wave and log2 of the waves
    bool valid;

    __device__ __forceinline__ Place(int rm, int rn, int tiles_m, int tiles_n, uint32_t nkb) {
        const int total = tiles_m * tiles_n, share = (total + 7) / 8;
        const int u = ((int)blockIdx.x & 7) * share + ((int)blockIdx.x >> 3);
        valid = u < total;
        const int tn = u / tiles_m, tm = u - tn * tiles_m;
        m0 = (int64_t)tm * rm;
        n0 = (int64_t)tn * rn;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        wlog = 25 - __builtin_clz(blockDim.x);
        // groups of 4 K blocks go to the waves in turn; only the last group can be short
        const uint32_t ng = (nkb + 3) >> 2, w = 1u << wlog;
        cnt = 0;
        if ((uint32_t)wave < ng) {
            cnt = ((ng - wave + w - 1) >> wlog) << 2;
            if (((ng - 1 - wave) & (w - 1)) == 0) cnt -= (ng << 2) - nkb;
        }
    }
    // first K block of this wave's group i, and its K block i
    __device__ __forceinline__ uint32_t group(uint32_t i) const { return (wave + (i << wlog)) << 2; }
    __device__ __forceinline__ uint32_t block(uint32_t i) const { return group(i >> 2) + (i & 3); }
};

// Codes of 16 rows x 4 K blocks in a wave.  Lane l loads row l % 16 of K block l / 16 whole (32 bytes
// or 28, and one scale: three loads for four blocks, against eight when every lane loads its eight
// codes of each block, which left the kernel waiting on the load path).  The fragments want chunk
// l / 16 of each block, so the 4 x 4 (block, chunk) arrangement is transposed between the four groups
// of 16 lanes by lane swaps.
template <bool P7>
struct CodeRows {
    const uint8_t* codes;    // row l % 16
    const int8_t* scales;
    int alpha;               // the row's largest scale
    uint32_t w[P7 ? 7 : 8];
    int a;

    __device__ __forceinline__ void place(const SmallOperand& op, int64_t r, uint32_t nkb) {
        const int64_t rc = min(r, op.rows - 1);   // rows past the edge repeat the last (never stored)
        codes = static_cast<const uint8_t*>(op.data) + rc * nkb * (P7 ? 28 : 32);
        scales = op.scales + rc * op.nsb;
    }
    // K block kb (this lane's own)
    __device__ __forceinline__ void load(const SmallOperand& op, uint32_t kb) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(codes + (uint64_t)kb * (P7 ? 28 : 32));
        if constexpr (!P7) {
            const u32x4 u = *reinterpret_cast<const u32x4*>(p), v = *reinterpret_cast<const u32x4*>(p + 4);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                w[i] = u[i];
                w[4 + i] = v[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 7; i++) w[i] = p[i];
        }
        a = scales[div32(kb, op.dgq)];
    }
};

__device__ __forceinline__ void swap32(uint32_t& x, uint32_t& y) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}
__device__ __forceinline__ void swap16(uint32_t& x, uint32_t& y) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}

// the four K blocks' chunks of this lane: c[t] = the 8 codes (E3C3: 56 bits) of chunk l / 16 of block
// t, m[t] = the block's multipliers, 2^-min(D, 24) | 2^-min(max(D - 24, 0), 24) << 16 as fp16
struct CodeGroup {
    uint32_t c[4][2], m[4];
    bool far;   // some block of the wave lies more than 24 binades below its row's top
};

template <bool P7>
__device__ __forceinline__ CodeGroup arrange(const CodeRows<P7>& r) {
    CodeGroup g;
    // chunk j of this lane's block
    if constexpr (!P7) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            g.c[j][0] = r.w[2 * j];
            g.c[j][1] = r.w[2 * j + 1];
        }
    } else {
        g.c[0][0] = r.w[0];
        g.c[0][1] = r.w[1];
        g.c[1][0] = __builtin_amdgcn_alignbit(r.w[2], r.w[1], 24);
        g.c[1][1] = __builtin_amdgcn_alignbit(r.w[3], r.w[2], 24);
        g.c[2][0] = __builtin_amdgcn_alignbit(r.w[4], r.w[3], 16);
        g.c[2][1] = __builtin_amdgcn_alignbit(r.w[5], r.w[4], 16);
        g.c[3][0] = __builtin_amdgcn_alignbit(r.w[6], r.w[5], 8);
        g.c[3][1] = r.w[6] >> 8;
    }
#pragma unroll
    for (int d = 0; d < 2; d++) {
        swap32(g.c[0][d], g.c[2][d]);
        swap32(g.c[1][d], g.c[3][d]);
        swap16(g.c[0][d], g.c[1][d]);
        swap16(g.c[2][d], g.c[3][d]);
    }
    const int D = r.alpha - r.a;
    g.far = __any(D > 24);
    const uint32_t m = f16_pow2_neg(min(max(D, 0), 24)) | (f16_pow2_neg(min(max(D - 24, 0), 24)) << 16);
    // every lane gets all four blocks' multipliers
    uint32_t x = m, y = m;
    swap32(x, y);
    g.m[0] = g.m[1] = x;
    g.m[2] = g.m[3] = y;
    swap16(g.m[0], g.m[1]);
    swap16(g.m[2], g.m[3]);
    return g;
}

// fragment of block t: lut = the operand's expansion table, l4 = 4 * lane.  The values are
// expand_chunk8's (the second multiply is by one where D <= 24)
template <bool P7>
__device__ __forceinline__ Frag fragment(const CodeGroup& g, int t, const char* lut, uint32_t l4) {
    uint32_t e[8], hv[4], lv[4];
#pragma unroll
    for (int i = 0; i < 8; i++) {
        uint32_t at;
        if constexpr (!P7) {
            // byte 0 from l4, byte 1 the code, zeros above
            at = __builtin_amdgcn_perm(g.c[t][i >> 2], l4, 0x0C0C0000u | ((4u + (i & 3)) << 8));
        } else {
            uint32_t c;
            if (7 * i + 7 <= 32) c = (g.c[t][0] >> (7 * i)) & 0x7Fu;
            else if (7 * i >= 32) c = (g.c[t][1] >> (7 * i - 32)) & 0x7Fu;
            else c = __builtin_amdgcn_alignbit(g.c[t][1], g.c[t][0], 7 * i) & 0x7Fu;
            at = c * LUT_PITCH + l4;
        }
        e[i] = *reinterpret_cast<const uint32_t*>(lut + at);
    }
    const half2v mm = __builtin_bit_cast(half2v, g.m[t]);
    const half2v m1 = {mm.x, mm.x};
#pragma unroll
    for (int p = 0; p < 4; p++) {
        hv[p] = pk_mul(__builtin_amdgcn_perm(e[2 * p + 1], e[2 * p], 0x05040100u), m1);
        lv[p] = pk_mul(__builtin_amdgcn_perm(e[2 * p + 1], e[2 * p], 0x07060302u), m1);
    }
    if (g.far) {   // rare; the empty asm keeps the compiler from computing it always and selecting
        asm volatile("");
        const half2v m2 = {mm.y, mm.y};
#pragma unroll
        for (int p = 0; p < 4; p++) {
            hv[p] = pk_mul(hv[p], m2);
            lv[p] = pk_mul(lv[p], m2);
        }
    }
    Frag f;
    f.hi = __builtin_bit_cast(half8, make_uint4(hv[0], hv[1], hv[2], hv[3]));
    f.lo = __builtin_bit_cast(half8, make_uint4(lv[0], lv[1], lv[2], lv[3]));
    return f;
}

// planes of 16 rows: row l % 16, chunk l / 16
struct PlaneRows {
    const char* hi;
    u32x4 h, l;

    __device__ __forceinline__ void place(const SmallOperand& op, int64_t r, int q) {
        // rows past the operand's last exist in its planes up to the next tile of 256
        hi = static_cast<const char*>(op.data) + (r / BM) * (2 * PLANE) + swz((int)(r % BM), q);
    }
};

// Largest scale key of each of a tile's `rows` rows, 0 past the operand's last: nthr / rows adjacent lanes
// share a row (4 to 32 of them: rows is 16 to 64, nthr 256 or 512).  The first dwords are requested by start()
// so that their latency passes under other loads.
struct RowMax {
    static constexpr int EARLY = 4;
    const int8_t* sp;
    int n4, part, per, row;
    bool live;
    uint32_t w[EARLY];

    __device__ __forceinline__ void start(const SmallOperand& op, int64_t r0, int rows, int tid, int nthr) {
        per = nthr / rows;
        part = tid & (per - 1);
        row = tid / per;
        live = r0 + row < op.rows;
        sp = op.scales + (live ? r0 + row : r0) * op.nsb;
        n4 = (int)(op.nsb >> 2);
#pragma unroll
        for (int k = 0; k < EARLY; k++) {
            w[k] = 0x81818181u;   // -127: at or below every key
            const int d = part + k * per;
            if (d < n4) __builtin_memcpy(&w[k], sp + 4 * d, 4);   // any alignment
        }
    }
    __device__ __forceinline__ void finish(const SmallOperand& op, int* out) const {
        int m = -128;
        auto four = [&](uint32_t x) {
#pragma unroll
            for (int b = 0; b < 4; b++) m = max(m, scale_key((int)(int8_t)(x >> (8 * b))));
        };
#pragma unroll
        for (int k = 0; k < EARLY; k++) four(w[k]);
#pragma unroll 4
        for (int d = part + EARLY * per; d < n4; d += per) {
            uint32_t x;
            __builtin_memcpy(&x, sp + 4 * d, 4);
            four(x);
        }
        for (int64_t i = 4 * (int64_t)n4 + part; i < op.nsb; i += per) m = max(m, scale_key((int)sp[i]));
        for (int o = per >> 1; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
        if (part == 0) out[row] = live ? m : 0;
    }
};

// the expansion table of a format, filled by all threads: the entries are requested by start()
template <bool P7>
struct TableFill {
    static constexpr int PIECES = LUT_ENTRIES<P7> * (LUT_PITCH / 16);   // 16-byte pieces
    static constexpr int EARLY = 4;
    uint32_t v[EARLY];

    __device__ __forceinline__ void start(int fidx, int tid, int nthr) {
#pragma unroll
        for (int k = 0; k < EARLY; k++) {
            const int i = tid + k * nthr;
            if (i < PIECES) v[k] = g_small_dec[fidx][i / (LUT_PITCH / 16)];
        }
    }
    __device__ __forceinline__ void finish(int fidx, int tid, int nthr, char* lut) const {
#pragma unroll
        for (int k = 0; k < EARLY; k++) {
            const int i = tid + k * nthr;
            if (i < PIECES) reinterpret_cast<uint4*>(lut)[i] = make_uint4(v[k], v[k], v[k], v[k]);
        }
#pragma unroll 4
        for (int i = tid + EARLY * nthr; i < PIECES; i += nthr) {
            const uint32_t x = g_small_dec[fidx][i / (LUT_PITCH / 16)];
            reinterpret_cast<uint4*>(lut)[i] = make_uint4(x, x, x, x);
        }
    }
};

template <int TM, int TN>
__device__ __forceinline__ void multiply(const Frag* fa, const Frag* fb, f32x4 (&acc)[TM][TN]) {
#pragma unroll
    for (int p = 0; p < 3; p++)   // hi.hi, hi.lo, lo.hi
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(p == 2 ? fa[i].lo : fa[i].hi,
                                                                   p == 1 ? fb[j].lo : fb[j].hi, acc[i][j], 0, 0, 0);
}

// the waves' sums through LDS (`mem`), added in wave order, scaled and stored
template <int TM, int TN>
__device__ __forceinline__ void finish(const f32x4 (&acc)[TM][TN], char* mem, const int* sAlpha, const int* sBeta,
                                       const Place& pl, int64_t M, int64_t N, float* __restrict__ C, int64_t ldc,
                                       int bias2) {
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, W = nthr >> 6;
    f32x4* red = reinterpret_cast<f32x4*>(mem);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) red[(pl.wave * TM * TN + i * TN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    for (int e = tid; e < TM * TN * 64; e += nthr) {
        f32x4 s = red[e];
        for (int w = 1; w < W; w++) s += red[w * TM * TN * 64 + e];
        // element v of lane l: row 4 (l / 16) + v, column l % 16 of its 16 x 16 tile
        const int t = e >> 6, l = e & 63;
        const int li = 16 * (t / TN) + 4 * (l >> 4), lj = 16 * (t % TN) + (l & 15);
        const int cmax = sBeta[lj];
        if (pl.n0 + lj < N) {
#pragma unroll
            for (int v = 0; v < 4; v++) {
                if (pl.m0 + li + v >= M) break;
                const int rmax = sAlpha[li + v];
                float val = __builtin_amdgcn_ldexpf(s[v], rmax + cmax - bias2);
                if (rmax >= POISON_KEY || cmax >= POISON_KEY) val = __builtin_nanf("");
                C[(pl.m0 + li + v) * ldc + pl.n0 + lj] = val;
            }
        }
    }
}

template <bool PA, bool PB, bool SAME, int TM, int TN>
__global__ __launch_bounds__(64 * WMAX) void small_codes_kernel(SmallOperand A, SmallOperand B, uint32_t nkb,
                                                                float* __restrict__ C, int64_t ldc, int bias2,
                                                                int tiles_m, int tiles_n) {
    constexpr int RM = 16 * TM, RN = 16 * TN;
    // the expansion tables (two when the formats' packings differ, or the formats do), then, after the
    // last gather, the waves' partial sums
    constexpr int LUT_A = LUT_ENTRIES<PA> * LUT_PITCH, LUT_B = SAME ? 0 : LUT_ENTRIES<PB> * LUT_PITCH;
    constexpr int RED = WMAX * TM * TN * 1024;
    constexpr int SMEM = LUT_A + LUT_B > RED ? LUT_A + LUT_B : RED;
    __shared__ __attribute__((aligned(16))) char smem[SMEM];
    __shared__ int sAlpha[RM], sBeta[RN];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    const Place pl(RM, RN, tiles_m, tiles_n, nkb);
    if (!pl.valid) return;   // uniform per workgroup
    const int lr = lane & 15;
    const uint32_t q = lane >> 4;

    CodeRows<PA> ra[TM];
    CodeRows<PB> rb[TN];
#pragma unroll
    for (int t = 0; t < TM; t++) ra[t].place(A, pl.m0 + 16 * t + lr, nkb);
#pragma unroll
    for (int t = 0; t < TN; t++) rb[t].place(B, pl.n0 + 16 * t + lr, nkb);
    auto fetch = [&](uint32_t g) {
        const uint32_t kb = min(pl.group(g) + q, nkb - 1);   // past the end: the last block (not used)
#pragma unroll
        for (int t = 0; t < TM; t++) ra[t].load(A, kb);
#pragma unroll
        for (int t = 0; t < TN; t++) rb[t].load(B, kb);
    };
    // loads return in order: the tables' and the scales', needed first, go out before the codes
    TableFill<PA> fa0;
    TableFill<PB> fb0;
    RowMax xa, xb;
    fa0.start(A.fidx, tid, nthr);
    if (!SAME) fb0.start(B.fidx, tid, nthr);
    xa.start(A, pl.m0, RM, tid, nthr);
    xb.start(B, pl.n0, RN, tid, nthr);
    fetch(0);
    fa0.finish(A.fidx, tid, nthr, smem);
    if (!SAME) fb0.finish(B.fidx, tid, nthr, smem + LUT_A);
    xa.finish(A, sAlpha);
    xb.finish(B, sBeta);
    __syncthreads();
    const char* lutA = smem;
    const char* lutB = smem + (SAME ? 0 : LUT_A);
    const uint32_t l4 = 4 * lane;
    // a poisoned row expands against the largest scale, its outputs are NaN whatever it accumulates
#pragma unroll
    for (int t = 0; t < TM; t++) ra[t].alpha = min(sAlpha[16 * t + lr], 127);
#pragma unroll
    for (int t = 0; t < TN; t++) rb[t].alpha = min(sBeta[16 * t + lr], 127);

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t groups = (pl.cnt + 3) >> 2;
    for (uint32_t g = 0; g < groups; g++) {
        CodeGroup ga[TM], gb[TN];
#pragma unroll
        for (int t = 0; t < TM; t++) ga[t] = arrange<PA>(ra[t]);
#pragma unroll
        for (int t = 0; t < TN; t++) gb[t] = arrange<PB>(rb[t]);
        fetch(g + 1);   // past the last group: not used
        const uint32_t have = pl.cnt - 4 * g;
#pragma unroll
        for (int t = 0; t < 4; t++) {
            if ((uint32_t)t >= have) break;   // wave-uniform: only in the last group
            Frag fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; i++) fa[i] = fragment<PA>(ga[i], t, lutA, l4);
#pragma unroll
            for (int j = 0; j < TN; j++) fb[j] = fragment<PB>(gb[j], t, lutB, l4);
            multiply<TM, TN>(fa, fb, acc);
        }
    }
    __syncthreads();   // the tables are no longer read
    finish<TM, TN>(acc, smem, sAlpha, sBeta, pl, A.rows, B.rows, C, ldc, bias2);
}

template <int TM, int TN, int U>
__global__ __launch_bounds__(64 * WMAX) void small_planes_kernel(SmallOperand A, SmallOperand B, uint32_t nkb,
                                                                 float* __restrict__ C, int64_t ldc, int bias2,
                                                                 int tiles_m, int tiles_n) {
    constexpr int RM = 16 * TM, RN = 16 * TN;
    __shared__ __attribute__((aligned(16))) char smem[WMAX * TM * TN * 1024];
    __shared__ int sAlpha[RM], sBeta[RN];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    const Place pl(RM, RN, tiles_m, tiles_n, nkb);
    if (!pl.valid) return;   // uniform per workgroup
    // U K blocks in flight per wave
    PlaneRows ra[U][TM], rb[U][TN];
#pragma unroll
    for (int t = 0; t < TM; t++) ra[0][t].place(A, pl.m0 + 16 * t + (lane & 15), lane >> 4);
#pragma unroll
    for (int t = 0; t < TN; t++) rb[0][t].place(B, pl.n0 + 16 * t + (lane & 15), lane >> 4);
    const int64_t sa = A.tiles * (2 * PLANE), sb = B.tiles * (2 * PLANE);
    auto fetch = [&](uint32_t i, int u) {
        const int64_t kb = pl.block(min(i, pl.cnt - 1));   // past the end: the last block again (not used)
#pragma unroll
        for (int t = 0; t < TM; t++) {
            const char* p = ra[0][t].hi + kb * sa;
            ra[u][t].h = *reinterpret_cast<const u32x4*>(p);
            ra[u][t].l = *reinterpret_cast<const u32x4*>(p + PLANE);
        }
#pragma unroll
        for (int t = 0; t < TN; t++) {
            const char* p = rb[0][t].hi + kb * sb;
            rb[u][t].h = *reinterpret_cast<const u32x4*>(p);
            rb[u][t].l = *reinterpret_cast<const u32x4*>(p + PLANE);
        }
    };
    if (pl.cnt > 0) {
#pragma unroll
        for (int u = 0; u < U; u++) fetch(u, u);
    }
    for (int i = tid; i < RM; i += nthr) sAlpha[i] = A.rmax[pl.m0 + i];
    for (int i = tid; i < RN; i += nthr) sBeta[i] = B.rmax[pl.n0 + i];

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto block = [&](uint32_t i, int u, bool refill) {
        Frag fa[TM], fb[TN];
#pragma unroll
        for (int t = 0; t < TM; t++)
            fa[t] = {__builtin_bit_cast(half8, ra[u][t].h), __builtin_bit_cast(half8, ra[u][t].l)};
#pragma unroll
        for (int t = 0; t < TN; t++)
            fb[t] = {__builtin_bit_cast(half8, rb[u][t].h), __builtin_bit_cast(half8, rb[u][t].l)};
        multiply<TM, TN>(fa, fb, acc);
        if (refill) fetch(i + U, u);
    };
    uint32_t i0 = 0;
    for (; i0 + U < pl.cnt; i0 += U) {
#pragma unroll
        for (int u = 0; u < U; u++) block(i0 + u, u, true);
    }
#pragma unroll
    for (int u = 0; u < U; u++)
        if (i0 + u < pl.cnt) block(i0 + u, u, false);   // wave-uniform
    finish<TM, TN>(acc, smem, sAlpha, sBeta, pl, A.rows, B.rows, C, ldc, bias2);
}

struct SmallGrid {
    int tiles_m, tiles_n;
    dim3 grid, block;
};

SmallGrid small_grid(const SmallPlan& p, int64_t M, int64_t N) {
    SmallGrid g;
    g.tiles_m = (int)((M + 16 * p.tm - 1) / (16 * p.tm));
    g.tiles_n = (int)((N + 16 * p.tn - 1) / (16 * p.tn));
    g.grid = dim3((unsigned)((g.tiles_m * g.tiles_n + 7) / 8 * 8));
    g.block = dim3((unsigned)(64 * p.waves));
    return g;
}

template <bool PA, bool PB, bool SAME>
hipError_t launch_codes(const SmallPlan& p, const SmallOperand& A, const SmallOperand& B, uint32_t nkb, float* c,
                        int64_t ldc, int bias2, hipStream_t s) {
    const SmallGrid g = small_grid(p, A.rows, B.rows);
#define CURVEFP_SMALL(TM, TN)                                                                                    \
    if (p.tm == TM && p.tn == TN) {                                                                              \
        hipLaunchKernelGGL((small_codes_kernel<PA, PB, SAME, TM, TN>), g.grid, g.block, 0, s, A, B, nkb, c, ldc,    \
                           bias2, g.tiles_m, g.tiles_n);                                                         \
        return hipGetLastError();                                                                                \
    }
    CURVEFP_SMALL(1, 1)
    CURVEFP_SMALL(1, 2)
    CURVEFP_SMALL(2, 1)
    CURVEFP_SMALL(2, 2)
    CURVEFP_SMALL(4, 2)
    CURVEFP_SMALL(2, 4)
#undef CURVEFP_SMALL
    return hipErrorInvalidValue;
}

hipError_t launch_planes(const SmallPlan& p, const SmallOperand& A, const SmallOperand& B, uint32_t nkb, float* c,
                         int64_t ldc, int bias2, hipStream_t s) {
    const SmallGrid g = small_grid(p, A.rows, B.rows);
#define CURVEFP_SMALL(TM, TN, U)                                                                                 \
    if (p.tm == TM && p.tn == TN) {                                                                              \
        hipLaunchKernelGGL((small_planes_kernel<TM, TN, U>), g.grid, g.block, 0, s, A, B, nkb, c, ldc, bias2, \
                           g.tiles_m, g.tiles_n);                                                                \
        return hipGetLastError();                                                                                \
    }
    CURVEFP_SMALL(1, 1, 4)
    CURVEFP_SMALL(1, 2, 2)
    CURVEFP_SMALL(2, 1, 2)
    CURVEFP_SMALL(2, 2, 2)
    CURVEFP_SMALL(4, 2, 2)
    CURVEFP_SMALL(2, 4, 2)
#undef CURVEFP_SMALL
    return hipErrorInvalidValue;
}

}  // namespace

// Up to 2^20 outputs.  There the time of the 256 x 256 and 128 x 128 kernels is that of one round whatever
// the size, and this kernel's grows with M N K; the lines cross near 2^20 from codes (1024 x 1024 x 4096:
// 58.6 us here, 67 us there) and near 2^21 from planes (512 x 4096 x 4096: 68 us on both).  The
// second condition leaves room for C in the workspace of the product's planes (4 K bytes per padded row of
// either operand), where curvefp_gemm_requant keeps it.
// The tile is the largest that still makes 192 workgroups for the 256 compute units (each operand row is
// expanded once per tile that needs it), without going past twice the operand's rows.  Eight waves share K
// where a unit has one workgroup, four where it has several (E4C3 codes, 128 x 4096 x 4096, 256 workgroups: 32.7 us
// with eight, 37.2 with four; 250 x 4096 x 4096, 512: 62.3 and 53.0 us).
bool small_plan(int64_t M, int64_t N, int64_t K, SmallPlan* p) {
    constexpr int64_t MOST = (int64_t)1 << 20;
    if (M > MOST || N > MOST || M * N > MOST) return false;
    if (M * N > K * ((M + BM - 1) / BM + (N + BM - 1) / BM) * BM) return false;
    static constexpr int shapes[][2] = {{4, 2}, {2, 4}, {2, 2}, {2, 1}, {1, 2}, {1, 1}};
    for (const auto& t : shapes) {
        const int64_t tiles = ((M + 16 * t[0] - 1) / (16 * t[0])) * ((N + 16 * t[1] - 1) / (16 * t[1]));
        if (t[0] + t[1] > 2 && (tiles < 192 || (t[0] > 1 && M <= 8 * t[0]) || (t[1] > 1 && N <= 8 * t[1]))) continue;
        *p = SmallPlan{t[0], t[1], tiles >= 512 || K <= 512 ? 4 : 8};
        break;
    }
    return true;
}

hipError_t launch_gemm_small(const SmallPlan& p, int sa, const SmallOperand& A, int sb, const SmallOperand& B,
                             int64_t K, float* c, int64_t ldc, int bias2, hipStream_t s) {
    const uint32_t nkb = (uint32_t)(K / 32);
    if (sa == SRC_PLANES && sb == SRC_PLANES) return launch_planes(p, A, B, nkb, c, ldc, bias2, s);
    if (A.fidx == B.fidx)
        return sa == SRC_CODES7 ? launch_codes<true, true, true>(p, A, B, nkb, c, ldc, bias2, s)
                                : launch_codes<false, false, true>(p, A, B, nkb, c, ldc, bias2, s);
    if (sa == SRC_CODES8)
        return sb == SRC_CODES8 ? launch_codes<false, false, false>(p, A, B, nkb, c, ldc, bias2, s)
                                : launch_codes<false, true, false>(p, A, B, nkb, c, ldc, bias2, s);
    return launch_codes<true, false, false>(p, A, B, nkb, c, ldc, bias2, s);   // one packed format exists
}

}  // namespace curvefp
