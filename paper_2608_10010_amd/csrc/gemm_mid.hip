// CurveFP GEMM on expanded planes with 128 x 128 tiles, for products whose 256 x 256 tiles (gemm.hip)
// leave compute units idle: prompts and batches of a few hundred rows.
//
// The planes, the order of the MFMAs within an output and the split of K are those of gemm.hip's
// 256 x 256 kernel, so C is the same bit for bit; only the tile shrinks.  Four waves of 64 x 64 (2 x 2
// MFMA 32x32x16 tiles) take a tile's K range on two 32 KB LDS stages.  Where K is split in two, both
// halves run in one workgroup (eight waves, two stages each) and their sums meet in LDS: no partial sums
// through memory, no arrival counters to clear, and two waves per SIMD, so that one's matrix instructions
// run under the other's fragment reads.  A step (one K block) has the 256 x 256 kernel's two phases: the
// second slice's fragments are read under the first slice's MFMAs; then, after the barrier, block s + 2 is
// copied into the stage just freed and block s + 1's first slice is read under the second slice's MFMAs.
//
// What bounds it: on a compute unit with a workgroup the matrix pipe is 72% busy (333 x 6144 x 4096, the whole
// kernel; the LDS half of the time), the rest is the barrier and the fragment reads, which a quarter-size tile has
// twice as many of per MFMA; there 144 workgroups on 256 units leave the others idle.  With the chip full it is the
// power limit.
// Measured, E4C3, operands prepared, 256 x 256 kernel -> this one: 512 x 4096 x 4096 107 -> 66 us,
// 1024 x 4096 x 1024 50 -> 31 us, 1000 x 2500 x 2080 85 -> 41 us.  Variants on 1024 x 4096 x 4096 (95 us):
// the halves in two workgroups with partial sums through memory 98 us (and 5 us to clear the counters);
// one workgroup of four 32 KB stages per unit 117 us; two waves of 128 x 64 per half (fewer fragment reads,
// one wave per SIMD) 98 us.
#include "curvefp_internal.hpp"
#include "gemm_mid.hpp"
#include "planes.hpp"

#include <type_traits>

namespace curvefp {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TB = 128;                        // tile rows and columns
constexpr int PIECE = TB * ROW_BYTES;          // 8 KB: one plane of one operand's tile rows
constexpr int STAGE = 4 * PIECE;               // A hi, A lo, B hi, B lo
constexpr int TM = 2, TN = 2;                  // 32 x 32 tiles of a wave
constexpr int MPS = TM * TN * 3;               // MFMAs per 16-wide K slice

// a pointer every lane holds alike, in scalar registers (buffer descriptors want it there)
__device__ __forceinline__ const char* uniform(const char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

struct Frag {
    half8 ah[TM], al[TM], bh[TN], bl[TN];
};

// XCD x (linear id mod 8) takes the x-th eighth of the work items, walking groups of 8 tile rows column
// by column, so that the workgroups resident on an XCD share their stages in its L2
struct WorkItem {
    int ty, tx;
    bool valid;
};

__device__ __forceinline__ WorkItem work_item(int tiles_y, int tiles_x) {
    constexpr int XCDS = 8, GROUP = 8;
    const int total = tiles_y * tiles_x;
    const int share = (total + XCDS - 1) / XCDS;
    const int t = ((int)blockIdx.x % XCDS) * share + (int)blockIdx.x / XCDS;
    WorkItem w;
    w.valid = t < total;
    const int g = t / (GROUP * tiles_x);
    const int gh = min(GROUP, tiles_y - g * GROUP);
    const int local = t - g * GROUP * tiles_x;
    w.ty = g * GROUP + local % gh;
    w.tx = local / gh;
    return w;
}

// HALVES: the parts K is split in (1 or 2)
template <int HALVES>
__global__ __launch_bounds__(256 * HALVES, HALVES == 1 ? 2 : 1) void gemm_mid_kernel(
    const char* __restrict__ PA, const char* __restrict__ PB, const int* __restrict__ maxA,
    const int* __restrict__ maxB, int64_t M, int64_t N, int nkb, int64_t RTA, int64_t RTB, float* __restrict__ C,
    int64_t ldc, int bias2, int tiles_y, int tiles_x) {
    // two stages (per half) as separate arrays, every access naming its stage statically: the compiler then
    // sees that copies into one and fragment reads from the other do not overlap
    __shared__ __attribute__((aligned(16))) char sh0[HALVES * STAGE];
    __shared__ __attribute__((aligned(16))) char sh1[HALVES * STAGE];
    __shared__ __attribute__((aligned(16))) int sAB[2 * TB];
    int* sAlpha = sAB;
    int* sBeta = sAB + TB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave8 & 3, half = wave8 >> 2;
    char* st0 = sh0 + half * STAGE;
    char* st1 = sh1 + half * STAGE;
    const WorkItem wi = work_item(tiles_y, tiles_x);
    if (!wi.valid) return;   // uniform per workgroup
    const int64_t m0 = (int64_t)wi.ty * TB, n0 = (int64_t)wi.tx * TB;
    // both halves run nsteps steps; with an odd block count the second half's last step has no block: its
    // copy repeats the last block and its MFMAs are left out
    const int nsteps = (nkb + HALVES - 1) / HALVES;
    const int kb0 = half * nsteps;
    const bool whole = kb0 + nsteps <= nkb;
    if (tid < TB) sAlpha[tid] = maxA[m0 + tid];
    else if (tid < 2 * TB) sBeta[tid - TB] = maxB[n0 + tid - TB];

    // wave w copies piece w of a stage (A hi, A lo, B hi, B lo): eight contiguous kilobytes of a plane
    using lds_ptr = __attribute__((address_space(3))) void*;
    const char* src = wave < 2 ? PA + (wi.ty >> 1) * (2 * (int64_t)PLANE) + (wi.ty & 1) * PIECE
                               : PB + (wi.tx >> 1) * (2 * (int64_t)PLANE) + (wi.tx & 1) * PIECE;
    src += (wave & 1) * PLANE;
    const int64_t src_step = (wave < 2 ? RTA : RTB) * (2 * (int64_t)PLANE);
    const int piece = wave * PIECE;
    src = uniform(src);
    auto dma = [&](int kb, char* st) {
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((void*)(src + (int64_t)min(kb, nkb - 1) * src_step), (short)0, PIECE, 0x00020000);
#pragma unroll
        for (int i = 0; i < 8; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)(st + piece + 1024 * i), 16, 16 * lane, 1024 * i, 0, 0);
    };

    auto dma_wait = [] { __builtin_amdgcn_s_waitcnt(0x0F70); };   // vmcnt(0)

    const int wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31;
    const int fsw = ((lr >> 1) ^ (lr >> 3)) & 3;
    const int foff0 = lr * ROW_BYTES + 16 * ((0 + (lane >> 5)) ^ fsw);
    const int foff1 = lr * ROW_BYTES + 16 * ((2 + (lane >> 5)) ^ fsw);
    const int abase = wm * 64 * ROW_BYTES, bbase = 2 * PIECE + wn * 64 * ROW_BYTES;
    auto load_frag = [&](Frag& f, const char* st, int kq) {
        const char* pa = st + abase + (kq ? foff1 : foff0);
        const char* pb = st + bbase + (kq ? foff1 : foff0);
#pragma unroll
        for (int t = 0; t < TM; t++) f.ah[t] = *reinterpret_cast<const half8*>(pa + t * 32 * ROW_BYTES);
#pragma unroll
        for (int t = 0; t < TN; t++) f.bh[t] = *reinterpret_cast<const half8*>(pb + t * 32 * ROW_BYTES);
#pragma unroll
        for (int t = 0; t < TN; t++) f.bl[t] = *reinterpret_cast<const half8*>(pb + PIECE + t * 32 * ROW_BYTES);
#pragma unroll
        for (int t = 0; t < TM; t++) f.al[t] = *reinterpret_cast<const half8*>(pa + PIECE + t * 32 * ROW_BYTES);
    };
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
    // products hi.hi, hi.lo, lo.hi over the tiles in snake order
    auto mfma = [&](const Frag& f, int idx) {
        const int p = idx / (TM * TN), i = (idx / TN) % TM, j = (i & 1) ? TN - 1 - idx % TN : idx % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(p == 2 ? f.al[i] : f.ah[i], p == 1 ? f.bl[j] : f.bh[j],
                                                           acc[i][j], 0, 0, 0);
    };
    constexpr int SG_MFMA = 0x008, SG_VMEM = 0x010, SG_DSR = 0x100;
    Frag f0, f1;
    auto phase1 = [&](char* st) {
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): f0's reads went out a phase ago
        load_frag(f1, st, 1);
#pragma unroll
        for (int m = 0; m < MPS; m++) mfma(f0, m);
#pragma unroll
        for (int i = 0; i < 8; i++) {
            __builtin_amdgcn_sched_group_barrier(SG_DSR, 1, 0);
            __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(SG_MFMA, MPS - 8, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto handover = [&] {
        dma_wait();
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto phase2 = [&](char* nx, bool copy, int kb, char* st) {
        if (copy) dma(kb, st);
        load_frag(f0, nx, 0);
#pragma unroll
        for (int m = 0; m < MPS; m++) mfma(f1, m);
#pragma unroll
        for (int i = 0; i < 8; i++) {
            __builtin_amdgcn_sched_group_barrier(SG_DSR, 1, 0);
            if (copy) __builtin_amdgcn_sched_group_barrier(SG_VMEM, 1, 0);
            __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(SG_MFMA, MPS - 8, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step_copy = [&](char* cur, char* nxt, int kb) {
        phase1(cur);
        handover();
        phase2(nxt, true, kb, cur);
    };
    auto step_nocopy = [&](char* cur, char* nxt) {
        phase1(cur);
        handover();
        phase2(nxt, false, 0, cur);
    };
    auto step_final = [&](char* cur) {
        if (!whole) return;   // wave-uniform, and no barrier below
        phase1(cur);
#pragma unroll
        for (int m = 0; m < MPS; m++) mfma(f1, m);
    };
    // stages alternate, and the last two steps always run on st0 then st1: with an odd step count the
    // first block goes to st1, and one step runs before the paired loop
    const bool odd = (nsteps & 1) != 0;
    char* first = odd ? st1 : st0;
    char* second = odd ? st0 : st1;
    dma(kb0, first);
    dma_wait();
    __syncthreads();
    if (nsteps > 1) dma(kb0 + 1, second);
    load_frag(f0, first, 0);
    if (nsteps == 1) {
        step_final(first);
    } else {
        int s = 0;
        if (odd) {   // nsteps >= 3: block kb0 + 2 exists
            step_copy(st1, st0, kb0 + 2);
            s = 1;
        }
        for (; s + 3 < nsteps; s += 2) {
            step_copy(st0, st1, kb0 + s + 2);
            step_copy(st1, st0, kb0 + s + 3);
        }
        step_nocopy(st0, st1);
        step_final(st1);
    }

    // register v of lane l of MFMA tile (ti, tj): row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
    const int lrow = wm * 64 + 4 * (lane >> 5), lcol = wn * 64 + (lane & 31);
#pragma unroll
    for (int ti = 0; ti < TM; ti++)
#pragma unroll
        for (int tj = 0; tj < TN; tj++) {
            const int beta = sBeta[lcol + 32 * tj] - bias2;
#pragma unroll
            for (int v = 0; v < 16; v++)
                acc[ti][tj][v] = __builtin_amdgcn_ldexpf(
                    acc[ti][tj][v], sAlpha[lrow + 32 * ti + 8 * (v >> 2) + (v & 3)] + beta);
        }
    // with two halves, the wave of each half keeps one 32-row tile of its 64 and gives the other half the
    // sums of the other: 32 registers per lane through the stages
    if (HALVES == 2) {
        __syncthreads();   // the stages are no longer read
        f32x4* give = reinterpret_cast<f32x4*>((half ? sh1 : sh0) + wave * 8192);
        const f32x4* take = reinterpret_cast<const f32x4*>((half ? sh0 : sh1) + wave * 8192);
        auto put = [&](const f32x16 (&a)[TN]) {
#pragma unroll
            for (int i = 0; i < TN * 4; i++) {
                const f32x16& x = a[i >> 2];
                give[i * 64 + lane] = f32x4{x[4 * (i & 3)], x[4 * (i & 3) + 1], x[4 * (i & 3) + 2], x[4 * (i & 3) + 3]};
            }
        };
        auto add = [&](f32x16 (&a)[TN]) {
#pragma unroll
            for (int i = 0; i < TN * 4; i++) {
                const f32x4 x = take[i * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; r++) a[i >> 2][4 * (i & 3) + r] += x[r];
            }
        };
        if (half == 0) put(acc[1]);
        else put(acc[0]);
        __syncthreads();
        if (half == 0) add(acc[0]);
        else add(acc[1]);
    }
    float* c0 = C + m0 * ldc + n0;
    auto store = [&](auto edge) {
#pragma unroll
        for (int ti = 0; ti < TM; ti++) {
            if (HALVES == 2 && half != ti) continue;   // wave-uniform
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const int li = lrow + 32 * ti + 8 * (v >> 2) + (v & 3);
                const int rmax = sAlpha[li];
#pragma unroll
                for (int tj = 0; tj < TN; tj++) {
                    const int lj = lcol + 32 * tj;
                    float val = acc[ti][tj][v];
                    if (rmax >= POISON_KEY || sBeta[lj] >= POISON_KEY) val = __builtin_nanf("");
                    if (!decltype(edge)::value || (m0 + li < M && n0 + lj < N)) c0[li * ldc + lj] = val;
                }
            }
        }
    };
    if (m0 + TB <= M && n0 + TB <= N) store(std::false_type());
    else store(std::true_type());
}

}  // namespace

hipError_t launch_gemm_mid(const char* pa, const char* pb, const int* maxA, const int* maxB, int64_t M, int64_t N,
                           int64_t K, int64_t rta, int64_t rtb, float* c, int64_t ldc, int bias2, int splits,
                           hipStream_t s) {
    const int ty = (int)((M + TB - 1) / TB), tx = (int)((N + TB - 1) / TB);
    const dim3 grid((unsigned)(((int64_t)ty * tx + 7) / 8 * 8));
    if (splits == 2)
        hipLaunchKernelGGL(gemm_mid_kernel<2>, grid, dim3(512), 0, s, pa, pb, maxA, maxB, M, N, (int)(K / 32), rta, rtb, c,
                           ldc, bias2, ty, tx);
    else
        hipLaunchKernelGGL(gemm_mid_kernel<1>, grid, dim3(256), 0, s, pa, pb, maxA, maxB, M, N, (int)(K / 32), rta, rtb, c,
                           ldc, bias2, ty, tx);
    return hipGetLastError();
}

}  // namespace curvefp
