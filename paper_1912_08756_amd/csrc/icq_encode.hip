// Encoding, the step before the search path (arxiv 1912.08756, Sec. 1: an item is
// stored as one codeword index per codebook, xbar_i = sum_k c_{k,code_k(i)}).  The
// paper gives no assignment algorithm; this is the greedy residual assignment in
// codebook order:
//     r_0 = x_i;  code_k(i) = argmin_j ||r_k - c_{k,j}||^2 (ties: smallest j);
//     r_{k+1} = r_k - c_{k,code_k(i)}.
// ||r - c||^2 = ||r||^2 - 2<r,c> + ||c||^2 and ||r||^2 does not depend on j, so a level is one
// [N x d].[d x 256] contraction with the epilogue argmin_j (||c_j||^2 - 2<r,c_j>).
//
// icq_encode_refine revisits given codes by coordinate descent over the codebooks (iterated
// conditional modes): with the other sub-codes of an item fixed, codebook k's codeword becomes the
// nearest one to r = x - sum_{l != k} c_l, and only if that is strictly nearer than the current
// one.  The residual holds x - xbar, a level adds the current codeword back, the argmin prefers the
// current codeword among equal scores, and only items whose sub-code changed get a new residual.
//
// Two kernels do both, all levels (and sweeps) of a block's items in one launch: encode_wave_kernel (icq_encode_wave.hip) holds
// the residuals in registers, up to 128 dimensions always and up to 512 where launch_encode says so; encode_kernel below keeps
// them in memory.  Two steps per level:
//  1. The contraction on half-precision copies of residual and codewords (v_mfma_f32_32x32x16_f16, sixteen
//     times the rate of the fp32 instruction) leaves, with a bound E on its error, a SUPERSET of the
//     codewords that can be the argmin: those whose score is within 2 E of the best.  E comes from
//     Cauchy-Schwarz: |<r,c> - <r',c'>| <= ||r|| ||c - c'|| + ||r - r'|| ||c'||, with ||c - c'|| measured
//     when the index is made, ||r - r'|| <= 2^-11 ||r||, and the accumulation's roundings.  All scales
//     are powers of two, so nothing else is rounded.
//  2. Items with more than one candidate (a few per cent) form the candidates' fp32 scores from the fp32
//     residual and codewords and take the argmin of those.  The result is the fp32 argmin, as before.
// Where more than eight codewords of an item are within the bound, encode_kernel repeats the level with both
// operands split in two halves (three products: E's operand part is smaller by 2^-10, its accumulation part
// three times as large).  Where it is more than eight after that (equal codewords), or the bound is no number
// (infinities, NaN, norms beyond fp32), the block forms all its scores in fp32 on the matrix cores.
// (encode_wave_kernel does so at once: its fp32 products cost a wavefront about what a second round would.)
//
// What bounds encode_kernel: the residuals' way through memory (4 TB/s at d = 960).
#include "icq_internal.h"
#include "icq_sort.h"
#include "icq_encode.h"

#include <math.h>

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4v __attribute__((ext_vector_type(4)));
constexpr int EB = 128;           // items per block
constexpr int E_THREADS = 512;
constexpr int E_P = EB * 16 / E_THREADS;   // items per owner group of 16 threads
constexpr int E_G = E_THREADS / 16;        // owner groups
constexpr int E_CAND = 8;         // candidates listed per item
constexpr int E_FROW = EB + 1;    // 16-byte pieces per reduction group of the residual's fragments: one to spare, so
                                  // that the 16 threads that write one row's groups meet different banks
constexpr float E_U = 4.8828125e-4f;       // 2^-11: relative rounding error of a half

struct EncShared {
    uint4 frag[16 * E_FROW];               // a 128-wide slice of the residuals: [reduction index / 8][item]
    uint4 cbs[2][4 * ICQ_LUT_W];           // a 32-wide slice of the codebook: [reduction index / 8][codeword]
    float cnh[ICQ_LUT_W];                  // -||c||^2 / 2, scaled: what the accumulators start from
    float nrm2[EB];                        // ||r||^2 (an item's entry, like its codes, belongs to its 16 threads)
    float smax[4][EB];                     // best score among each 64 codewords
    uint32_t ccount[EB];                   // candidates
    uint8_t cand[EB][E_CAND];
    uint8_t code[ICQ_MAX_K][EB];
    uint8_t before[EB];                    // the sub-code the level before found
    uint32_t over;                         // some item has more than E_CAND candidates
};
static_assert(sizeof(EncShared) <= 81920, "two blocks per CU");

// x, from here on: what is derived from it is computed again instead of kept in a register since the kernel's start
template <typename T>
__device__ __forceinline__ T fresh(T x) {
    asm volatile("" : "+v"(x));
    return x;
}

// sum over the 16 lanes of a DPP row, in every lane
__device__ __forceinline__ float row_sum(float x) {
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x128, 0xf, 0xf, false));   // row_ror:8
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x124, 0xf, 0xf, false));
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x122, 0xf, 0xf, false));
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x121, 0xf, 0xf, false));
    return x;
}

// x [N][d]; cb [K*256][d_pad] fp32; half_hi / half_lo: see encode_pack_kernel; meta[k] = scale, largest ||c||, largest ||c - c'||;
// the residuals in res [N][d_pad].  ICM: `codes` is in and out, `changed` (or nullptr) counts per sweep.
//
// Thread t owns the 8 dimensions from 8 (t % 16) on of the items t / 16 + 32 p, p = 0 .. 3 (of every 128-wide slice):
// residual rows and codewords are read in whole pieces of 16 threads.  In the contraction the codewords are the rows of
// the matrix instruction (wavefront w: the 64 from 64 (w % 4) on) and the items its columns (the 64 from 64 (w / 4) on),
// so a lane holds 32 scores of one item per column block and the maximum is taken inside the lane.  64 x 64 scores per
// wavefront are 64 registers, which leave room for four wavefronts per SIMD.  7 of the 128 registers' values are spilled
// (ICM: 41, mostly around the round of fp32 scores).
template <bool ICM>
__global__ __launch_bounds__(E_THREADS, 4) void encode_kernel(
    const float *__restrict__ x, int d, const float *__restrict__ cb, int d_pad, const float *__restrict__ cnorm,
    const uint4 *__restrict__ half_hi, const uint4 *__restrict__ half_lo, const float4 *__restrict__ meta, int K, int slices,
    int64_t N, uint8_t *codes, int sweeps, float *res, uint32_t *changed) {
    extern __shared__ __attribute__((aligned(16))) unsigned char enc_smem[];
    EncShared &sh = *reinterpret_cast<EncShared *>(enc_smem);
    const int tid0 = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
    const int64_t i0 = (int64_t)blockIdx.x * EB;
    const int cw = wave & 3, ih = wave >> 2;
    const int nks = (d_pad + 31) / 32;                     // 32-wide codebook slices
    const int nsl = (nks + 3) / 4;                         // 128-wide residual slices
    const int live = N - i0 < EB ? (int)(N - i0) : EB;     // items of this block; rows past them read the last one's x
    auto row = [&](int rg, int p) { return i0 + (rg + E_G * p < live ? rg + E_G * p : live - 1); };
    // a residual in memory is its owner's alone; rows past N read a codeword instead of racing with it
    auto res_row = [&](int rg, int p) -> const float * {
        return rg + E_G * p < live ? res + (i0 + rg + E_G * p) * d_pad : cb;
    };

    auto load_x = [&](int rg, int p, int e0, float (&v)[8]) __attribute__((always_inline)) {
        // Pieces need no alignment.  What lies outside the row is masked by bits: a select between a load and zero ends
        // as a branch around the load, one wait per piece instead of all pieces in flight together.
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
        const int64_t at = row(rg, p) * d + (e0 < d ? e0 : 0);
        const uint32_t *s = reinterpret_cast<const uint32_t *>(x) + at;
        if (at + 8 <= N * d) {
            const u32x4 a = *reinterpret_cast<const u32x4 *>(s), b = *reinterpret_cast<const u32x4 *>(s + 4);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = __uint_as_float((i < 4 ? a[i & 3] : b[i & 3]) & (e0 + i < d ? ~0u : 0u));
        } else {                                           // the end of x
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = e0 + i < d ? __uint_as_float(s[i]) : 0.0f;
        }
    };
    // eight values of a row of d_pad floats (a multiple of 16: the piece is inside or outside as a whole)
    auto load8 = [&](const float *s, int e0, float (&v)[8]) __attribute__((always_inline)) {
        const bool in = e0 < d_pad;
        const uint4 a = *reinterpret_cast<const uint4 *>(s + (in ? e0 : 0));
        const uint4 b = *reinterpret_cast<const uint4 *>(s + (in ? e0 + 4 : 4));
        const uint32_t m = in ? ~0u : 0u;
        const uint32_t w[8] = {a.x & m, a.y & m, a.z & m, a.w & m, b.x & m, b.y & m, b.z & m, b.w & m};
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = __uint_as_float(w[i]);
    };
    auto codeword = [&](int k, uint32_t j) -> const float * {
        return cb + ((int64_t)k * ICQ_LUT_W + j) * d_pad;
    };
    auto store_res = [&](int rg, int p, int e0, const float (&v)[8]) __attribute__((always_inline)) {
        if (rg + E_G * p < live && e0 < d_pad) {
            float *o = res + row(rg, p) * d_pad + e0;
            *reinterpret_cast<float4v *>(o) = float4v{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<float4v *>(o + 4) = float4v{v[4], v[5], v[6], v[7]};
        }
    };

    if (ICM) {
        for (int i = tid0; i < K * EB; i += E_THREADS) {
            const int64_t at = i0 + i % EB;
            sh.code[i / EB][i % EB] = codes[(int64_t)(i / EB) * N + (at < N ? at : N - 1)];
        }
        __syncthreads();
    }
    // the starting residuals and the largest norm among them (it sets the first level's scale)
    auto add_norm = [&](int tid, int rg, int p, int sl, float x) __attribute__((always_inline)) {
        x = row_sum(x);
        const int item = rg + E_G * p;
        if ((tid & 15) == 0) sh.nrm2[item] = item >= live ? 0.0f : sl == 0 ? x : sh.nrm2[item] + x;
    };
    for (int sl = 0; sl < nsl; ++sl) {
        const int tid = fresh(tid0), e0 = sl * 128 + (tid & 15) * 8, rg = tid >> 4;
        float v[E_P][8];
#pragma unroll
        for (int p = 0; p < E_P; ++p) load_x(rg, p, e0, v[p]);
        if (ICM) {                                         // x - sum_k c_k, k ascending
            for (int k = 0; k < K; ++k) {
                float c[E_P][8];
#pragma unroll
                for (int p = 0; p < E_P; ++p) load8(codeword(k, sh.code[k][rg + E_G * p]), e0, c[p]);
#pragma unroll
                for (int p = 0; p < E_P; ++p)
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[p][i] -= c[p][i];
            }
        }
#pragma unroll
        for (int p = 0; p < E_P; ++p) {
            float s = 0.0f;
            if (ICM) store_res(rg, p, e0, v[p]);
#pragma unroll
            for (int i = 0; i < 8; ++i) s = fmaf(v[p][i], v[p][i], s);
            add_norm(tid, rg, p, sl, s);
        }
    }
    __syncthreads();
    bool wild = false;                                     // some norm of the block is no number
    auto largest_norm = [&]() __attribute__((always_inline)) -> float {                   // behind a barrier after nrm2 was written
        const int lane = fresh(tid0) & 63;
        // as bits, which order as the squares do; an item whose norm is no number would take the others' halves from
        // them and has no bound anyway
        const uint32_t a = __float_as_uint(sh.nrm2[lane]), b = __float_as_uint(sh.nrm2[lane + 64]);
        const uint32_t a1 = a < 0x7f800000u ? a : 0u, b1 = b < 0x7f800000u ? b : 0u;
        wild = __builtin_amdgcn_ballot_w64(a1 != a || b1 != b) != 0;
        const float v = __uint_as_float(wave_max_u32(a1 > b1 ? a1 : b1));
        return __builtin_amdgcn_sqrtf(v) * 1.0001f;
    };
    float reach = largest_norm();                          // no residual of the block is longer
    uint32_t nchanged = 0;

    // slice g of codebook k's halves -> LDS, straight from memory
    const int chunk = slices * 128;                        // 32 codewords
    auto fetch = [&](const uint4 *src, int k, int g) __attribute__((always_inline)) {
        const int lane = fresh(tid0) & 63;
        const uint4 *s = src + ((int64_t)(k * 8 + (wave & 1) * 4) * chunk + (g * 4 + (wave >> 1)) * 32);
        const uint32_t at = (uint32_t)((lane >> 5) * chunk + (lane & 31));
        uint4 *dst = sh.cbs[g & 1] + wave * 128;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(s + i * 2 * chunk + at),
                                             (__attribute__((address_space(3))) void *)(dst + i * 64), 16, 0, 0);
    };
    // what a level needs first: its first two slices, its codebook's scale and norms (asked for a level ahead)
    float4 mt;
    float cn = 0.0f;
    auto ahead = [&](int k) __attribute__((always_inline)) {
        fetch(half_hi, k, 0);
        if (nks > 1) fetch(half_hi, k, 1);
        mt = meta[k];
        if (tid0 < ICQ_LUT_W) cn = cnorm[k * ICQ_LUT_W + tid0];
    };
    ahead(0);
    // scale of the residuals of the level to come, and what its scores start from
    float sr;
    auto rescale = [&]() __attribute__((always_inline)) {
        sr = icq_enc_scale_below(fmaxf(reach + (ICM ? mt.y : 0.0f), mt.y), 14);        // no r of that level is longer than this
        if (tid0 < ICQ_LUT_W) sh.cnh[tid0] = -0.5f * (sr * mt.x) * cn;         // -inf beyond m
    };
    rescale();
    __syncthreads();

    const int levels = ICM ? K * sweeps : K;
    bool equal = false;                                    // the second round left too many candidates at some level: no use
    for (int lev = 0; lev < levels; ++lev) {
        const int k = ICM ? lev % K : lev;
        const int kp = k == 0 ? K - 1 : k - 1, kn = k == K - 1 ? 0 : k + 1;        // the codebooks of the levels around it
        const float cmax = mt.y, dmax = mt.z, sc = mt.x, S = sr * sc;

        // the residual of this level in item p's piece at e0, before (ICM) the current codeword is added back
        auto residual = [&](int rg, int p, int e0, float (&v)[8]) __attribute__((always_inline)) {
            if (!ICM && lev == 0) {
                load_x(rg, p, e0, v);
            } else {
                load8(res_row(rg, p), e0, v);
            }
        };
        // the residuals of slice sl as halves -> LDS.  UPDATE: first bring them up to date with the level before
        // and sum their squares.  LOW: the second halves.
        auto stage = [&](int sl, bool update, bool low) __attribute__((always_inline)) {
            const int tid = fresh(tid0), rg = tid >> 4, e0 = sl * 128 + (tid & 15) * 8;
            const float scale = fresh(sr), zero = fresh(0.0f);
#pragma unroll 2
            for (int p = 0; p < E_P; ++p) {
                float v[8];
                if (update && lev > 0) {
                    const uint32_t oldc = sh.before[rg + E_G * p], newc = sh.code[kp][rg + E_G * p];
                    const bool moved = !ICM || newc != oldc;
                    if (!ICM && lev == 1) load_x(rg, p, e0, v);
                    else load8(res_row(rg, p), e0, v);
                    if (moved) {
                        float c[8];
                        if (ICM) {
                            load8(codeword(kp, oldc), e0, c);
#pragma unroll
                            for (int i = 0; i < 8; ++i) v[i] += c[i];
                        }
                        load8(codeword(kp, newc), e0, c);
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[i] -= c[i];
                        store_res(rg, p, e0, v);
                    }
                } else {
                    residual(rg, p, e0, v);
                }
                if (ICM) {
                    float c[8];
                    load8(codeword(k, sh.code[k][rg + E_G * p]), e0, c);
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] += c[i];
                }
                half8 h;
                float n2 = zero;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    n2 = fmaf(v[i], v[i], n2);
                    const float s = v[i] * scale;
                    h[i] = (_Float16)s;
                    if (low) h[i] = (_Float16)(s - (float)h[i]);
                }
                if (update) add_norm(tid, rg, p, sl, n2);
                if (e0 < nks * 32) sh.frag[(tid & 15) * E_FROW + rg + E_G * p] = __builtin_bit_cast(uint4, h);
            }
        };
        // acc += residual halves x codeword halves over all dimensions
        auto contract = [&](float16v (&acc)[2][2], const uint4 *src, int pass, bool update) __attribute__((always_inline)) {
            const int lane = fresh(tid0) & 63, half = lane >> 5, l32 = lane & 31;
            if (!update || pass > 0) {
                fetch(src, k, 0);
                if (nks > 1) fetch(src, k, 1);
            }
            for (int g = 0; g < nks; ++g) {
                if ((g & 3) == 0) {
                    if (g > 0) __syncthreads();            // the last slice's fragments are consumed
                    stage(g >> 2, update, pass == 1);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this thread's part of slice g is in LDS
                __syncthreads();
                if (g > 0 && g + 1 < nks) fetch(src, k, g + 1);
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    half8 a[2], b[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        a[t] = __builtin_bit_cast(half8, sh.cbs[g & 1][(kk * 2 + half) * ICQ_LUT_W + cw * 64 + t * 32 + l32]);
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        b[u] = __builtin_bit_cast(half8, sh.frag[((g & 3) * 4 + kk * 2 + half) * E_FROW + ih * 64 + u * 32 + l32]);
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int t = 0; t < 2; ++t) acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[t], b[u], acc[u][t], 0, 0, 0);
                }
            }
        };

        const int tid = fresh(tid0);
        if (tid < EB) sh.ccount[tid] = 0;
        if (tid == 0) sh.over = 0;
        // ---- candidates: codewords whose score is within twice the error bound of the item's best
        auto candidates = [&](const float16v (&acc)[2][2], float u_r, float d_c, int passes) __attribute__((always_inline)) {
            const int lane = fresh(tid0) & 63, half = lane >> 5, l32 = lane & 31;
            float best[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float b = acc[u][0][0];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) b = fmaxf(b, acc[u][t][v]);
                b = fmaxf(b, __shfl_xor(b, 32, 64));
                if (half == 0) sh.smax[cw][ih * 64 + u * 32 + l32] = b;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int item = ih * 64 + u * 32 + l32;
                const float b = fmaxf(fmaxf(sh.smax[0][item], sh.smax[1][item]), fmaxf(sh.smax[2][item], sh.smax[3][item]));
                const float rn = __builtin_amdgcn_sqrtf(sh.nrm2[item]) * 1.0001f;
                // |<r,c> - <r',c'>|, scaled; the third term: halves below the normal range (2^-25 each at most; of the
                // codewords' second halves that is less than u_r * cmax allows); the last: every pass's roundings
                const float E = S * rn * (u_r * cmax + (1.0f + u_r) * d_c) + __builtin_amdgcn_sqrtf((float)(nks * 32)) * 2.98e-8f * sc * cmax +
                                (float)(passes * nks * 32 + 8) * 1.2e-7f * S * cmax * (rn + cmax);
                // a bound that is no number (infinities, NaN, components beyond the halves' range) admits nobody: what its
                // differences' signs say would be a matter of which NaN the instructions make
                best[u] = E < INFINITY && item < live ? b - 2.0f * E - fabsf(b) * 1e-6f - 1e-30f : INFINITY;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int item = ih * 64 + u * 32 + l32;
                uint32_t bits = 0;                         // the sign of bound - score, first score in bit 31
#pragma unroll
                for (int i = 0; i < 32; ++i)
                    bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(best[u] - acc[u][i >> 4][i & 15]), 31);
                if (!(best[u] < INFINITY)) bits = 0;
                while (bits != 0) {
                    const int i = __builtin_clz(bits);
                    bits &= ~(0x80000000u >> i);
                    const uint32_t code = (uint32_t)(cw * 64 + (i >> 4) * 32 + (i & 3) + 4 * half + 8 * ((i & 15) >> 2));
                    const uint32_t slot = atomicAdd(&sh.ccount[item], 1u);
                    if (slot < (uint32_t)E_CAND) sh.cand[item][slot] = (uint8_t)code;
                    else sh.over = 1;
                }
            }
            __syncthreads();
        };
        // ---- for the items whose candidates say nothing: the fp32 argmin over all codewords as the only candidate.  (The
        // 256 scores one by one instead, sixteen threads an item, took 0.35 us each: 12 times as long.)
        auto exact = [&]() __attribute__((always_inline)) {
            const int tid = fresh(tid0), lane = tid & 63, half = lane >> 5, l32 = lane & 31, rg = tid >> 4;
            float *F = reinterpret_cast<float *>(sh.frag);                 // [64 dimensions][E_FROW]
            float *C = reinterpret_cast<float *>(sh.cbs);                  // [256 codewords][17]: 16 dimensions
            u64 *best = reinterpret_cast<u64 *>(sh.frag);                  // [4][EB]
            static_assert(64 * E_FROW * sizeof(float) <= sizeof(sh.frag) && ICQ_LUT_W * 17 * sizeof(float) <= sizeof(sh.cbs), "");
            float16v acc[2][2];
#pragma unroll
            for (int i = 0; i < 64; ++i) acc[i >> 5][(i >> 4) & 1][i & 15] = 0.0f;
#pragma nounroll
            for (int e = 0; e < d_pad; e += 16) {
                __syncthreads();                           // the slice before is consumed
                const int e0 = (e & ~127) + (tid & 15) * 8;
                if ((e & 63) == 0 && (e0 & ~63) == e) {
#pragma unroll
                    for (int p = 0; p < E_P; ++p) {
                        asm volatile("" ::: "memory");
                        float v[8];
                        residual(rg, p, e0, v);
                        if (ICM) {
                            float c[8];
                            load8(codeword(k, sh.code[k][rg + E_G * p]), e0, c);
#pragma unroll
                            for (int i = 0; i < 8; ++i) v[i] += c[i];
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) F[((e0 & 63) + i) * E_FROW + rg + E_G * p] = v[i];
                    }
                }
                {
                    float c[8];
                    load8(codeword(k, (uint32_t)tid >> 1), e + (tid & 1) * 8, c);
#pragma unroll
                    for (int i = 0; i < 8; ++i) C[(tid >> 1) * 17 + (tid & 1) * 8 + i] = c[i];
                }
                __syncthreads();
#pragma unroll 2
                for (int s = 0; s < 8; ++s) {
                    float a[2], b[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) a[t] = C[(cw * 64 + t * 32 + l32) * 17 + 2 * s + half];
#pragma unroll
                    for (int u = 0; u < 2; ++u) b[u] = F[((e & 63) + 2 * s + half) * E_FROW + ih * 64 + u * 32 + l32];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int t = 0; t < 2; ++t) acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[u], acc[u][t], 0, 0, 0);
                }
            }
            __syncthreads();                               // the fragments are consumed
            // key: order-preserving bits of the score, index + 1 (ICM: 0 for the current codeword); no number, no key
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int item = ih * 64 + u * 32 + l32;
                const uint32_t old = ICM ? sh.code[k][item] : ~0u;
                float b = INFINITY;                        // the least score and, below, the first field that has it
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        asm volatile("" ::: "memory");     // (four norms at a time: all 32 would push residuals out of registers)
                        const float4v cn = *reinterpret_cast<const float4v *>(cnorm + k * ICQ_LUT_W + cw * 64 + t * 32 + w * 8 + half * 4);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc[u][t][w * 4 + i] = cn[i] - 2.0f * acc[u][t][w * 4 + i];
                            b = fminf(b, acc[u][t][w * 4 + i]);            // not NaN
                        }
                    }
                const uint32_t first = (uint32_t)(cw * 64 + 4 * half);
                uint32_t f = 0;
                bool keep = false;                         // the current codeword has it
#pragma unroll
                for (int i = 31; i >= 0; --i) {
                    const uint32_t at = (uint32_t)((i >> 4) * 32 + (i & 3) + 8 * ((i & 15) >> 2));
                    f = acc[u][i >> 4][i & 15] == b ? at : f;
                    if (ICM) keep |= acc[u][i >> 4][i & 15] == b && old == first + at;
                }
                f = keep ? 0u : first + f + 1u;
                u64 key = b < INFINITY ? ((u64)icq_order_bits(b + 0.0f) << 32) | f : ~0ull;
                const u64 other = __shfl_xor(key, 32, 64);
                key = other < key ? other : key;
                if (half == 0) best[cw * EB + item] = key;
            }
            __syncthreads();
            if (tid < live) {
                const uint32_t n = sh.ccount[tid];
                if (n == 0 || n > (uint32_t)E_CAND) {
                    u64 key = best[tid];
#pragma unroll
                    for (int w = 1; w < 4; ++w) key = best[w * EB + tid] < key ? best[w * EB + tid] : key;
                    // no score a number: index 0 (ICM: the current one) stays
                    const uint32_t old = ICM ? sh.code[k][tid] : 0u;
                    sh.cand[tid][0] = (uint8_t)(key == ~0ull || (uint32_t)key == 0u ? old : (uint32_t)key - 1u);
                    sh.ccount[tid] = 1;
                }
            }
            __syncthreads();
        };
        // ---- first halves only; then, if that left some item too many candidates, both halves of both sides but the
        // product of the two second ones
        bool over;
#pragma nounroll
        for (int round = 0;; ++round) {
            // accumulator register v of lane l is codeword (v % 4) + 4 (l / 32) + 8 (v / 4), item l % 32 of its tile
            float16v acc[2][2];
            const int half = (fresh(tid0) >> 5) & 1;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float4v c = *reinterpret_cast<const float4v *>(&sh.cnh[cw * 64 + t * 32 + w * 8 + half * 4]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[0][t][w * 4 + i] = acc[1][t][w * 4 + i] = c[i];
                }
#pragma nounroll
            for (int pass = 0; pass < (round == 0 ? 1 : 3); ++pass) {
                if (pass > 0) __syncthreads();             // the fragments of the pass before are consumed
                contract(acc, pass == 2 ? half_lo : half_hi, pass, round == 0);
            }
            candidates(acc, round == 0 ? E_U : 4.0f * E_U * E_U, round == 0 ? dmax : 2.0f * E_U * dmax, round == 0 ? 1 : 3);
            over = sh.over != 0;
            if (round != 0) equal |= over;
            if (round != 0 || !over || equal) break;   // block-uniform: read between barriers
            __syncthreads();
            if (tid < EB) sh.ccount[tid] = 0;
            if (tid == 0) sh.over = 0;
        }
        reach = largest_norm() + cmax;                     // of the residuals the level leaves
        // some item has no bound: a norm or (for all items) a codeword is no number.  All else is finite: what the scales
        // multiply is below 2^14 and 2^10
        if (over || wild || !(dmax < INFINITY)) exact();   // block-uniform
        // ---- the sub-codes: the only candidate, or the argmin of the candidates' fp32 scores
        const bool last = lev + 1 == levels;
        if (!last) ahead(kn);
        const int rg = tid >> 4, c8 = (tid & 15) * 8;
#pragma unroll
        for (int p = 0; p < E_P; ++p) {
            const int item = rg + E_G * p;
            const uint32_t n = item < live ? sh.ccount[item] : 1u;
            const uint32_t old = ICM ? sh.code[k][item] : 0u;
            uint32_t code = n - 1u < (uint32_t)E_CAND && item < live ? sh.cand[item][0] : old;
            if (__builtin_amdgcn_ballot_w64(n != 1) != 0) {        // wavefront-uniform: four items at a time
                float best = INFINITY;
                uint32_t bf = 0xFFFFFFFFu;                         // ICM: 0 for the current codeword, else index + 1
                const uint32_t todo = n != 1 ? n : 0u;             // at most E_CAND
                for (uint32_t i = 0; __builtin_amdgcn_ballot_w64(i < todo) != 0; ++i) {
                    const uint32_t j = sh.cand[item][i < n ? i : 0];
                    float dot = 0.0f, c[8];
                    for (int sl = 0; sl < nsl; ++sl) {
                        const int e0 = sl * 128 + c8;
                        float v[8];
                        load8(codeword(k, j), e0, c);
                        residual(rg, p, e0, v);
                        if (ICM) {
                            float o[8];
                            load8(codeword(k, old), e0, o);
#pragma unroll
                            for (int q = 0; q < 8; ++q) v[q] += o[q];
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q) dot = fmaf(v[q], c[q], dot);
                    }
                    dot = row_sum(dot);
                    const float score = cnorm[k * ICQ_LUT_W + j] - 2.0f * dot;
                    const uint32_t f = ICM && j == old ? 0u : j + 1u;
                    if (i < todo && (score < best || (score == best && f < bf))) {
                        best = score;
                        bf = f;
                    }
                }
                if (todo != 0 && bf != 0xFFFFFFFFu) code = bf == 0u ? old : bf - 1u;
            }
            if ((tid & 15) == 0) {
                if (ICM) sh.before[item] = (uint8_t)old;
                sh.code[k][item] = (uint8_t)code;
            }
            if (ICM && code != old && (tid & 15) == 0 && item < live) ++nchanged;
        }
        wave_lds_order();                                  // the sixteen lanes of an item read what one of them wrote
        if (ICM && k == K - 1 && changed) {
            const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(nchanged), 63);
            if ((tid & 63) == 0 && n != 0) atomicAdd(&changed[lev / K], n);
            nchanged = 0;
        }
        if (!last) rescale();
        __syncthreads();
    }
    for (int i = tid0; i < K * EB; i += E_THREADS)
        if (i0 + i % EB < N) codes[(int64_t)(i / EB) * N + i0 + i % EB] = sh.code[i / EB][i % EB];
}

// The codewords as halves, laid out as the contractions read them, times the codebook's scale: the first halves in hi and
// (where the second round of encode_kernel reads them) what they leave in lo.  Piece ((k * 8 + j / 32) * slices * 4 + e / 8) * 32
// + j % 32 holds the eight dimensions e .. e + 7 of codeword j (zero beyond d).  16 threads per codeword.  meta[k].z is zero
// on entry.
__global__ __launch_bounds__(256) void encode_pack_kernel(const float *__restrict__ cb, int d_pad, int slices,
                                                          const float *__restrict__ cnorm, uint4 *__restrict__ hi,
                                                          uint4 *__restrict__ lo, float4 *__restrict__ meta) {
    __shared__ float red[4];
    const int tid = threadIdx.x, k = blockIdx.x / 16, j = (blockIdx.x % 16) * 16 + tid / 16;
    float v = cnorm[k * ICQ_LUT_W + tid];
    v = v < INFINITY ? v : 0.0f;
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    const float cmax = sqrtf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))) * 1.0001f;
    const float sc = icq_enc_scale_below(cmax, 10);
    float err = 0.0f;
    for (int c = tid & 15; c < slices * 4; c += 16) {
        half8 a, b;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int e = c * 8 + i;
            const float s = e < d_pad ? cb[((int64_t)k * ICQ_LUT_W + j) * d_pad + e] * sc : 0.0f;
            a[i] = (_Float16)s;
            const float rest = s - (float)a[i];
            b[i] = (_Float16)rest;
            err = fmaf(rest, rest, err);
        }
        const int64_t at = (((int64_t)k * 8 + j / 32) * slices * 4 + c) * 32 + j % 32;
        hi[at] = __builtin_bit_cast(uint4, a);
        if (lo) lo[at] = __builtin_bit_cast(uint4, b);
    }
    err = sqrtf(row_sum(err)) / sc * 1.0001f;
    if ((tid & 15) == 0) atomicMax(reinterpret_cast<unsigned int *>(&meta[k].z), __float_as_uint(err));
    if (blockIdx.x % 16 == 0 && tid == 0) {
        meta[k].x = sc;
        meta[k].y = cmax;
    }
}

// One wavefront per item: ||x - sum_k c_{k,code_k}||^2 accumulated in double.
__global__ __launch_bounds__(256) void quantization_error_kernel(const float *__restrict__ x, int d, int d_pad,
                                                                 const float *__restrict__ cb, int K,
                                                                 const uint8_t *__restrict__ codes, int64_t N,
                                                                 double *__restrict__ err) {
    const int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;                            // whole wavefronts leave together
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    for (int e = lane; e < d; e += 64) {
        double xb = 0.0;
        for (int k = 0; k < K; ++k) xb += (double)cb[((int64_t)k * ICQ_LUT_W + codes[(int64_t)k * N + n]) * d_pad + e];
        const double diff = (double)x[n * d + e] - xb;
        s += diff * diff;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) err[n] = s;
}

}  // namespace

ICQ_EXPORT int icq_encode_workspace_bytes(const icq_index *ix, int64_t N, size_t *out) {
    if (!ix || !out || N < 0 || N > ICQ_MAX_N) return ICQ_ERR_ARG;
    const size_t need = sizeof(float) * (size_t)N * (size_t)ix->d_pad;
    *out = need > ICQ_ALIGN ? icq_align_up(need, ICQ_ALIGN) : ICQ_ALIGN;
    return ICQ_OK;
}

template <bool ICM>
static int launch_encode(const icq_index *ix, const float *x, int64_t N, uint8_t *codes, int sweeps, float *res,
                         uint32_t *changed, hipStream_t s) {
    const int slices = icq_enc_slices(ix->d_pad);
    // Residuals in registers: always up to 128 dimensions (icq_enc_wave_only).  Above, by what a CU then holds (the register form's
    // time over encode_kernel's):
    //  - coordinate descent has one wavefront per SIMD there, two with few items.  Up to 256 dimensions while blocks find room in one
    //    round (d = 144, 192, 200, 256, K = 8; 16384 items 0.44 .. 0.51, 32768 0.52, 0.49, 0.79, 0.79; 33000 1.08, 1.01, 1.05,
    //    1.04, K = 16 1.05, 1.12, 1.26, 1.33, 131000 1.0 .. 1.1; with vectors that have no bound 1.3 to 1.6), beyond that while
    //    blocks of 64 items do (d = 288, 384, 512, K = 8; 16384 items 0.60, 0.55, 0.58; 17000 1.10, 1.08, 1.28);
    //  - greedy assignment up to 256 dimensions throughout.  Beyond that one block of 128 items per CU against two of
    //    encode_kernel's: ahead in the first round of blocks, in those that leave the CUs a single block there and (12 slices) in
    //    well filled others (d = 320, 384, 448, K = 16; 32768 items 0.71, 0.65, 0.70; 1.03, 1.15, 1.45, 1.9 rounds 1.22 .. 0.97,
    //    1.20 .. 0.93, 1.01 .. 1.05; 2.05, 2.9 rounds 1.00, 0.97, 0.92 and 0.84, 0.82, 0.90; 3.05 .. 3.6 1.13 .. 1.00, 1.05 .. 0.94,
    //    1.09 .. 1.02).  With 15 or 16 slices, of which the register form wastes none, throughout (d = 512: 0.81 .. 1.08).
    const int64_t cu = ix->num_cu, blocks = (N + EB - 1) / EB, rounds = (blocks + cu - 1) / cu;
    const bool full = slices == 12 && 5 * (blocks - (rounds - 1) * cu) > 3 * cu;
    const bool wave = ICM ? N <= (slices <= 8 ? 128 : 64) * cu : slices <= 8 || rounds % 2 == 1 || full || ix->d_pad > 448;
    if (icq_enc_wave_only(ix->d_pad) || (slices <= 16 && wave))
        return icq_launch_encode_wave(ix, x, N, codes, ICM, sweeps, res, changed, s);
    ICQ_HIP_TRY(icq_allow_lds(reinterpret_cast<const void *>(encode_kernel<ICM>), sizeof(EncShared)));
    encode_kernel<ICM><<<(unsigned)blocks, E_THREADS, sizeof(EncShared), s>>>(
        x, ix->d, ix->cb, ix->d_pad, ix->cnorm, ix->half_hi, ix->half_lo, ix->enc_meta, ix->K, slices, N, codes, sweeps, res, changed);
    return icq_check_launch();
}

int icq_encode_pack(icq_index *ix, hipStream_t s) {
    encode_pack_kernel<<<ix->K * 16, 256, 0, s>>>(ix->cb, ix->d_pad, icq_enc_slices(ix->d_pad), ix->cnorm, ix->half_hi, ix->half_lo,
                                                  ix->enc_meta);
    return icq_check_launch();
}

ICQ_EXPORT int icq_encode(const icq_index *ix, const float *x, int64_t N, uint8_t *codes_out, void *workspace,
                          size_t workspace_bytes, void *stream) {
    if (!ix || N < 0 || N > ICQ_MAX_N) return ICQ_ERR_ARG;
    if (N == 0) return ICQ_OK;
    if (!x || !codes_out) return ICQ_ERR_ARG;
    size_t need = 0;
    (void)icq_encode_workspace_bytes(ix, N, &need);
    if (!workspace || ((uintptr_t)workspace % ICQ_ALIGN) != 0 || workspace_bytes < need) return ICQ_ERR_WORKSPACE;
    return launch_encode<false>(ix, x, N, codes_out, 1, static_cast<float *>(workspace), nullptr, (hipStream_t)stream);
}

ICQ_EXPORT int icq_encode_refine(const icq_index *ix, const float *x, int64_t N, uint8_t *codes, int sweeps,
                                 uint32_t *changed_out, void *workspace, size_t workspace_bytes, void *stream) {
    if (!ix || N < 0 || N > ICQ_MAX_N || sweeps < 0 || sweeps > ICQ_MAX_SWEEPS) return ICQ_ERR_ARG;
    if (N == 0 || sweeps == 0) return ICQ_OK;
    if (!x || !codes) return ICQ_ERR_ARG;
    size_t need = 0;
    (void)icq_encode_workspace_bytes(ix, N, &need);
    if (!workspace || ((uintptr_t)workspace % ICQ_ALIGN) != 0 || workspace_bytes < need) return ICQ_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    if (changed_out) icq_zero_words(changed_out, sweeps, s);
    return launch_encode<true>(ix, x, N, codes, sweeps, static_cast<float *>(workspace), changed_out, s);
}

ICQ_EXPORT int icq_quantization_error(const icq_index *ix, const float *x, int64_t N, const uint8_t *codes,
                                      double *err_out, void *stream) {
    if (!ix || N < 0 || N > ICQ_MAX_N) return ICQ_ERR_ARG;
    if (N == 0) return ICQ_OK;
    if (!x || !codes || !err_out) return ICQ_ERR_ARG;
    quantization_error_kernel<<<(unsigned)((N + 3) / 4), 256, 0, (hipStream_t)stream>>>(x, ix->d, ix->d_pad, ix->cb, ix->K,
                                                                                         codes, N, err_out);
    return icq_check_launch();
}
