// Encoding with the residuals in registers (arxiv 1912.08756; the method -- candidates from half precision with an error
// bound, decided by fp32 scores -- stands in icq_encode.hip): up to 128 dimensions always, up to 512 where launch_encode
// there says so.
//
// A wavefront owns its 32 (few items: 16) vectors alone and sees all 256 codewords, so nothing is exchanged with the rest of
// the block but the codewords' halves, which the four wavefronts stream through LDS together, 32 codewords (a chunk) at a
// time.  Two layouts of a vector:
//  - as owner, lane (og, ol) holds dimensions 32 g + 4 ol + (0 .. 3) of the items og + 8 p: eight lanes read 128 bytes of a
//    row at once.  (Two lanes an item, as the matrix instruction wants it, made gathers of 16 bytes from 64 lines: the
//    address unit takes those one lane a clock, and the update of the residuals took as long as the contraction.)
//  - in the contraction the items are the columns of the matrix instruction, lane (item, sub) holds parts of all slices;
//    the halves get there through 2.5 KiB of LDS, the fp32 values never do.
// The candidates are collected chunk by chunk against the best score so far (less twice the error bound): no score is kept.
// What the running bound admits too many is dropped when a later chunk lifts it by more than that margin.  The residuals are
// kept times a power of two of the block (see sr), so making halves of them is one instruction for two.
//
// What bounds it (10^6 x 128, K = 8): vector issue, 53 % busy with 1002 instructions per wavefront and level (32 items; the
// form before spent 3252 on as many), beside the matrix cores' 27 %; three wavefronts a SIMD overlap the two.
// Contraction and candidates are about half of the instructions (per chunk 16 differences, 16 sign collections, 8
// maxima of three), halves and norms 130, the update 64, second looks 250.  Leaving out single parts gained 3 - 5 % each.
// Before / now: 10^6 x 128, K = 8: 1.03 / 0.84 ms; 262147 x 96, K = 16, two sweeps: 1.74 / 1.21 ms; 5000 x 128, K = 8:
// 0.050 / 0.037; 30000 x 180: 0.130 / 0.058; 15000 x 300: 0.182 / 0.079; 320000 x 32: 0.262 / 0.159 ms.
#include "icq_internal.h"
#include "icq_sort.h"
#include "icq_encode.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2 __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
constexpr int W_THREADS = 256;             // four wavefronts, each with items of its own
// Candidates of an item looked at one by one, beyond that all codewords are scored on the matrix cores; and items of a wavefront
// without a usable list that are taken one after another instead.  Above 128 dimensions a level's codewords come from memory
// for each such item as they do for all of them together.  10^5 items, K = 8, 16 equal codewords each, 8 / 32: 128 dimensions,
// greedy 849 / 705 us, a sweep 1516 / 923; 32 dimensions, greedy 311 / 362, a sweep 592 / 450; 256, greedy 1925 / 2495.  One infinite vector
// in 128 items, a sweep, without / with: 128 dimensions 1130 / 316 us.
constexpr int w_cand(int ns, bool icm) { return ns > 4 || (ns == 1 && !icm) ? 8 : 32; }
constexpr int w_lone(int ns) { return ns <= 4 ? 4 : 0; }
constexpr float W_U = 4.8828125e-4f;       // 2^-11: relative rounding error of a half

// NS: 32-wide slices of the dimensions.  A chunk is 32 codewords of one codebook as halves, all dimensions: 2 NS KiB.
constexpr int w_step(int ns) { return ns > 4 ? 2 : 1; }                                   // chunks contracted together
constexpr int w_stage(int ns) { return ns == 1 ? 8 : ns == 2 ? 4 : 2; }                   // and fetched together
constexpr int w_ring(int ns) { return ns == 8 ? 4 : 2; }                                  // such stages in LDS

// Wavefronts per SIMD that the registers allow with next to no spilling: a spilled register costs more than a missing wavefront
// (128 dimensions, greedy: 106 spilled at two wavefronts 1.9 ms, none 0.94; 51 at three 1.5, none 0.84; 262147 x 96, 16
// codebooks, greedy and two sweeps, three wavefronts: 57 spilled 1.53, 13 1.27, 5 1.21).  Spilled by <items, slices, ICM>: <32, 3, true> 5, <32, 4, false> 9,
// <16, 16, true> 10, <32, 16, false> 63; the others none.
constexpr int w_waves(int it, int ns, bool icm) {
    if (ns <= 4) return ns == 4 && it == 32 && icm ? 2 : 3;
    if (ns <= 8) return it == 16 ? (ns == 8 && icm ? 1 : 2) : (ns == 6 && !icm ? 2 : 1);
    return it == 16 && ns == 12 && !icm ? 2 : 1;
}

// What a wavefront keeps in LDS for itself.
template <int IT, int NS, bool ICM>
struct WaveOwn {
    uint4 piece[4][IT + 8];                // a slice of the halves: [reduction index / 8][item]; of the residuals: 16 dimensions.
                                           // (128 bytes to spare: the rows that owners write together meet different banks)
    float nrm2[IT];                        // ||v||^2
    uint32_t count[IT];                    // candidates
    alignas(8) uint8_t cand[IT][w_cand(NS, ICM)];          // the first of them
};
template <int IT, int NS, bool ICM>
struct WaveShared {
    uint4 ring[w_ring(NS)][w_stage(NS) * NS * 128];        // chunk: [reduction index / 8][codeword]
    WaveOwn<IT, NS, ICM> own[4];
    float cnh[2][ICQ_LUT_W];               // -||c||^2 / 2, scaled: what the accumulators of a level start from
    uint32_t reach[3];                     // largest ||v||^2 of the block's items, as bits, of three levels in turn
    uint32_t wild;                         // whether some item of the block has a norm that is no number
    uint8_t code[][4 * IT];                // [K]
};

// a combination over the 64 / IT lanes of an item (lanes IT apart), in each of them
template <int IT, typename F>
__device__ __forceinline__ uint32_t over_item(uint32_t x, F f) {
    if (IT == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = f(p[0], p[1]);
    }
    const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return f(p[0], p[1]);
}
template <int IT>
__device__ __forceinline__ float item_max(float x) {
    return __uint_as_float(over_item<IT>(__float_as_uint(x), [](uint32_t a, uint32_t b) {
        uint32_t y;                        // (fmaxf would first quieten both: three instructions)
        asm("v_max_f32 %0, %1, %2" : "=v"(y) : "v"(a), "v"(b));
        return y;
    }));
}

// x, from here on: what is derived from it is computed again instead of kept in a register since the kernel's start
__device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

template <int IT> struct Tile;
template <> struct Tile<32> {
    typedef float16v acc;
    static __device__ __forceinline__ acc half(half8 a, half8 b, acc c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ acc full(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <> struct Tile<16> {
    typedef float4v acc;
    static __device__ __forceinline__ acc half(half8 a, half8 b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ acc full(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

// x [N][d]; cb [K*256][d_pad] fp32; halves: see encode_pack_kernel; meta[k] = scale, largest ||c||, largest ||c - c'||.  ICM: `codes`
// is in and out, `changed` (or nullptr) counts per sweep; res [N][d_pad] is scratch.
template <int IT, int NS, bool ICM>
__global__ __launch_bounds__(W_THREADS, w_waves(IT, NS, ICM)) void encode_wave_kernel(
    const float *__restrict__ x, int d, const float *__restrict__ cb, int d_pad, const float *__restrict__ cnorm,
    const uint4 *__restrict__ halves, const float4 *__restrict__ meta, int K, int m, int64_t N, uint8_t *codes, int sweeps,
    float *res, uint32_t *changed) {
    constexpr int P = IT / 8;              // items per owner group of eight lanes
    constexpr int LPI = 64 / IT;           // lanes of an item in the contraction
    constexpr int KS = 4 / LPI;            // matrix instructions a slice takes per tile
    constexpr int AV = IT * IT / 64;       // scores of a tile of IT codewords that a lane holds
    constexpr int CPS = w_step(NS);        // chunks per step
    constexpr int TP = 32 * CPS / IT;      // tiles of a step
    constexpr int CS = AV * TP;            // scores of a step that a lane holds
    constexpr int NW = 256 / IT * AV / 32; // words of candidate bits
    constexpr int SW = 32 / CS;            // steps a word holds
    constexpr int GS = KS * TP == 2 && NS % 2 == 0 && NS > 4 ? 2 : 1;              // slices whose codewords are read from LDS together
    constexpr float ROOT_D = NS == 1 ? 5.66f : NS == 2 ? 8.0f : NS == 3 ? 9.8f : NS == 4 ? 11.32f : NS <= 8 ? 16.0f : NS <= 16 ? 22.63f : 32.0f;     // of the dimensions
    constexpr int EB = 4 * IT;             // items per block
    constexpr int TS = w_stage(NS), RING = w_ring(NS), PARTS = TS * NS / 2;        // 4 KiB each
    constexpr int OG = NS < 16 / P ? NS : 16 / P;          // slices of current codewords loaded together (64 registers)
    constexpr int PG = NS * P * 4 <= 128 ? P : NS * 4 <= 64 ? 2 : 1;     // items whose new codewords are (128 registers)
    typedef typename Tile<IT>::acc acc_t;
    extern __shared__ __attribute__((aligned(16))) unsigned char enc_smem[];
    auto &sh = *reinterpret_cast<WaveShared<IT, NS, ICM> *>(enc_smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto &own = sh.own[wave];
    const int og = lane >> 3, ol = lane & 7;               // as owner: items og + 8 p, dimensions 32 g + 4 ol + (0 .. 3)
    const int64_t i0 = (int64_t)blockIdx.x * EB + wave * IT;               // the wavefront's first item
    const int live = N - i0 < IT ? (N > i0 ? (int)(N - i0) : 0) : IT;      // and how many; rows past the last read it
    const int steps = (m + 32 * CPS - 1) / (32 * CPS), stages = (steps * CPS + TS - 1) / TS;

    // the stream of stages, codebook after codebook (round and round), straight from memory into the ring
    int fk = 0, fs = 0, fslot = 0, slot = 0;
    auto fetch = [&]() __attribute__((always_inline)) {
        const uint4 *s = halves + ((int64_t)fk * 8 + fs * TS) * (NS * 128) + tid;
        uint4 *dst = sh.ring[fslot] + wave * 64;
#pragma unroll
        for (int i = 0; i < PARTS; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(s + i * 256),
                                             (__attribute__((address_space(3))) void *)(dst + i * 256), 16, 0, 0);
        if (++fs == stages) {
            fs = 0;
            fk = fk + 1 == K ? 0 : fk + 1;
        }
        fslot = fslot + 1 == RING ? 0 : fslot + 1;
    };
    // this lane's piece of slice g of a row of d_pad floats (a multiple of 16: the piece is inside or outside as a whole)
    auto load4 = [&](const float *s, int g, float *v, int l8) __attribute__((always_inline)) {
        const int e = g * 32 + l8 * 4;
        const bool in = NS * 32 - 32 > g * 32 && NS <= 4 ? true : e < d_pad;
        const uint4 a = *reinterpret_cast<const uint4 *>(s + (in ? e : 0));
        const uint32_t k = in ? ~0u : 0u;
        v[0] = __uint_as_float(a.x & k);
        v[1] = __uint_as_float(a.y & k);
        v[2] = __uint_as_float(a.z & k);
        v[3] = __uint_as_float(a.w & k);
    };
    auto codeword = [&](int k, uint32_t j) -> const float * { return cb + (((uint32_t)k * ICQ_LUT_W + j) * (uint32_t)d_pad); };
    // sum over the eight lanes of an owner group, in each of them
    auto group_add = [&](float v) __attribute__((always_inline)) -> float {
        v += __uint_as_float(icq_dpp<0xB1, 0xf, 0u>(__float_as_uint(v)));      // quad_perm: lane ^ 1
        v += __uint_as_float(icq_dpp<0x4E, 0xf, 0u>(__float_as_uint(v)));      // lane ^ 2
        v += __uint_as_float(icq_dpp<0x141, 0xf, 0u>(__float_as_uint(v)));     // row_half_mirror: the other four
        return v;
    };

    float r[P][NS][4];
    uint8_t (*code)[EB] = sh.code;
    if (ICM) {
        for (int i = tid; i < K * EB; i += W_THREADS) {
            const int64_t p = (int64_t)blockIdx.x * EB + i % EB;
            code[i / EB][i % EB] = codes[(int64_t)(i / EB) * N + (p < N ? p : N - 1)];
        }
        __syncthreads();
    }
    {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
        // pieces need no alignment; what lies outside the row is masked by bits
        auto load_x = [&](auto piece) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int64_t row = i0 + og + 8 * p < N ? i0 + og + 8 * p : N - 1;
#pragma unroll
                for (int g = 0; g < NS; ++g) {
                    const int e = g * 32 + ol * 4;
                    const u32x4 w = piece(reinterpret_cast<const uint32_t *>(x) + (row * d + (e < d ? e : 0)), e);
#pragma unroll
                    for (int i = 0; i < 4; ++i) r[p][g][i] = __uint_as_float(w[i] & (e + i < d ? ~0u : 0u));
                }
            }
        };
        if (N - i0 >= IT + 1 && (N - i0 - IT) * d >= 4)    // wavefront-uniform: pieces of these rows end inside x
            load_x([&](const uint32_t *s, int) { return *reinterpret_cast<const u32x4 *>(s); });
        else
            load_x([&](const uint32_t *s, int e) {
                u32x4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = s[e + i < d ? i : 0];
                return w;
            });
    }
    if (ICM) {                             // x - sum_k c_k, k ascending
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const float *c = codeword(k, code[k][wave * IT + og + 8 * p]);
#pragma unroll
                for (int g = 0; g < NS; ++g) {
                    float v[4];
                    load4(c, g, v, ol);
#pragma unroll
                    for (int i = 0; i < 4; ++i) r[p][g][i] -= v[i];
                }
            }
    }
    // the largest norm of the block's items (none that is no number: it would take the others' halves from them and has no
    // bound anyway) -> LDS, zero before; n2[p]: ||v||^2 of item og + 8 p
    auto tell_reach = [&](int to, const float (&n2)[P]) __attribute__((always_inline)) {
        uint32_t most = 0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t b = __float_as_uint(n2[p]);
            most = max(most, b < 0x7f800000u ? b : 0u);
        }
        if (ol == 0) atomicMax(&sh.reach[to], most);
    };
    auto hear_reach = [&](int from) __attribute__((always_inline)) -> float {
        return __builtin_amdgcn_sqrtf(__uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)sh.reach[from])));
    };
    float n2[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        n2[p] = 0.0f;
#pragma unroll
        for (int g = 0; g < NS; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) n2[p] = fmaf(r[p][g][i], r[p][g][i], n2[p]);
        n2[p] = group_add(n2[p]);
    }
    if (tid < 3) sh.reach[tid] = 0;
    if (tid == 3) sh.wild = 0;
    __syncthreads();
    tell_reach(2, n2);
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (!(n2[p] < INFINITY)) sh.wild = 1;
    for (int i = 0; i < RING - 1; ++i) fetch();
    __syncthreads();
    // From here on r holds the residuals times sr, a power of two of the block that keeps the halves within their range;
    // it follows the norms when they have left a wide band.  A vector whose norm is no number may have finite components
    // that only sr <= 1 keeps so.
    float4 mt = meta[0];
    const float upper = hear_reach(2) * 1.0001f + (ICM ? mt.y : 0.0f);
    const float sr_max = sh.wild != 0 ? 1.0f : INFINITY;
    float sr = fminf(icq_enc_scale_below(fmaxf(upper, mt.y), 13), sr_max);
    auto rescale = [&](float f) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int g = 0; g < NS; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) r[p][g][i] *= f;
    };
    rescale(sr);
    sh.cnh[0][tid] = -0.5f * (sr * mt.x) * cnorm[tid];     // -inf beyond m
    uint32_t nchanged = 0;

    const int levels = ICM ? K * sweeps : K;
    for (int lev = 0; lev < levels; ++lev) {
        const int k = ICM ? lev % K : lev, kn = k == K - 1 ? 0 : k + 1;
        const float cmax = mt.y, dmax = mt.z, sc = mt.x;
        const float4 mn = meta[kn];
        const float twice = 2.0f / sr;                     // exact
        const float cn = cnorm[kn * ICQ_LUT_W + tid];
        uint32_t old[P];                                   // ICM: the current sub-codes
#pragma unroll
        for (int p = 0; p < P; ++p) old[p] = ICM ? code[k][wave * IT + og + 8 * p] : 0u;
        // ---- v, what the level contracts, as halves: from its owners through LDS to the lanes that multiply it
        const int lane = fresh(tid) & 63, og = lane >> 3, ol = lane & 7;
        const int col = lane % IT, sub = lane / IT;        // in the contraction: item, part of a slice's dimensions
        half8 h[NS * KS];
        float o[ICM ? P : 1][OG][4];
#pragma unroll
        for (int p = 0; p < P; ++p) n2[p] = 0.0f;
#pragma unroll
        for (int g = 0; g < NS; ++g) {
            if (ICM && g % OG == 0) {
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int u = 0; u < OG; ++u)
                        if (g + u < NS) load4(codeword(k, old[p]), g + u, o[p][u], ol);
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                half4 y;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = ICM ? fmaf(o[ICM ? p : 0][g % OG][i], sr, r[p][g][i]) : r[p][g][i];
                    y[i] = (_Float16)v;
                }
                n2[p] = __builtin_amdgcn_fdot2(half2{y[0], y[1]}, half2{y[0], y[1]}, n2[p], false);
                n2[p] = __builtin_amdgcn_fdot2(half2{y[2], y[3]}, half2{y[2], y[3]}, n2[p], false);
                reinterpret_cast<uint2 *>(&own.piece[ol >> 1][og + 8 * p])[ol & 1] = __builtin_bit_cast(uint2, y);
            }
            wave_lds_order();
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) h[g * KS + kk] = __builtin_bit_cast(half8, own.piece[sub * KS + kk][col]);
            wave_lds_order();
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            n2[p] = group_add(n2[p]);
            if (ol == 0) own.nrm2[og + 8 * p] = n2[p];
        }
        tell_reach(lev % 3, n2);
        if (tid == 0) sh.reach[(lev + 1) % 3] = 0;
        wave_lds_order();
        // ---- scores <v, c> - ||c||^2 / 2 in half precision, and candidates: codewords whose score is within twice the
        // error bound of the item's best so far.  |<r,c> - <r',c'>|, scaled; the third term: halves below the normal
        // range (2^-25 each at most); the last: the roundings of the sum.  The norm is the halves' own: 2^-11 off at most,
        // and what halves below the normal range may have lost
        const float rn = __builtin_amdgcn_sqrtf(own.nrm2[col]) * 1.001f + ROOT_D * 6.2e-5f;
        const float E = sc * rn * (W_U * cmax + (1.0f + W_U) * dmax) + ROOT_D * 2.98e-8f * sc * cmax +
                        (float)(NS * 32 + 8) * 1.2e-7f * sc * cmax * (rn + sr * cmax);
        // a bound that is no number (infinities, NaN, components beyond the halves' range) admits nobody
        const bool known = E < INFINITY && col < live;
        const float margin = 2.0f * E + 1e-30f;
        float best = -INFINITY;
        uint32_t bits[NW];                                 // a score above the bound sets its bit; first score in bit 31
#pragma unroll
        for (int w = 0; w < NW; ++w) bits[w] = 0;
        int from = 0;                                      // of the steps before this one even the best score is out
#pragma unroll
        for (int step = 0; step < 8 / CPS; ++step) {
            if (step >= steps) {                           // uniform
                if (step % SW != 0) bits[step / SW] <<= CS & 31;
                continue;
            }
            if (step * CPS % TS == 0) {
                // this thread's part of the stage is in LDS, and what it read of the one before is here; behind the
                // barrier that holds for all threads, and the stage before may be overwritten
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PARTS * (RING - 2)) : "memory");
                fetch();
                if (step > 0 || lev > 0) slot = slot + 1 == RING ? 0 : slot + 1;
            }
            acc_t acc[TP];
#pragma unroll
            for (int t = 0; t < TP; ++t)
#pragma unroll
                for (int w = 0; w < AV / 4; ++w) {
                    const float4v c = *reinterpret_cast<const float4v *>(&sh.cnh[lev & 1][(step * TP + t) * IT + w * 8 + sub * 4]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[t][w * 4 + i] = c[i];
                }
            const uint4 *ring = sh.ring[slot] + step * CPS % TS * (NS * 128) + sub * KS * 32 + col;
            half8 a[2][GS * KS * TP];
            auto read = [&](int gi) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < GS * KS * TP; ++i) {
                    const int t = i % TP, kk = i / TP % KS, g = gi * GS + i / (TP * KS);
                    a[gi & 1][i] = __builtin_bit_cast(half8, ring[(t * IT / 32) * (NS * 128) + (g * 4 + kk) * 32 + t * IT % 32]);
                }
            };
            read(0);
#pragma unroll
            for (int gi = 0; gi < NS / GS; ++gi) {
                if (gi + 1 < NS / GS) read(gi + 1);
                __builtin_amdgcn_sched_barrier(0);         // these reads are under way before the products that do not need them
#pragma unroll
                for (int i = 0; i < GS * KS * TP; ++i)
                    acc[i % TP] = Tile<IT>::half(a[gi & 1][i], h[(gi * GS + i / (TP * KS)) * KS + i / TP % KS], acc[i % TP]);
            }
            // register i of lane l is codeword (i % 4) + 4 (l / IT) + 8 (i / 4) of its tile, item l % IT
            float most = best;
#pragma unroll
            for (int i = 0; i < CS; ++i) most = fmaxf(most, acc[i / AV][i % AV]);
            most = item_max<IT>(most);
            const float bound = most - margin - fabsf(most) * 1e-6f;
            from = best > bound ? from : step;
            best = most;
#pragma unroll
            for (int i = 0; i < CS; ++i)                   // the sign of bound - score
                bits[step / SW] = __builtin_amdgcn_alignbit(bits[step / SW], __float_as_uint(bound - acc[i / AV][i % AV]), 31);
        }
        // the item's list, lane after lane of its own
        bool hard, several;                                // some of the wavefront have more than one; hard: see below
        {
            uint32_t n = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int out = (from - w * SW) * CS;      // leading bits that are out
                bits[w] = !known || out >= 32 ? 0u : out <= 0 ? bits[w] : bits[w] & (0xFFFFFFFFu >> out);
                n += (uint32_t)__builtin_popcount(bits[w]);
            }
            // candidates of the lanes before this one, and of all
            uint32_t before = 0, all = n;
            if (IT == 16) {
                const auto q = __builtin_amdgcn_permlane16_swap(all, all, false, false);
                before += (sub & 1) != 0 ? q[0] : 0u;
                all = q[0] + q[1];
            }
            {
                const auto q = __builtin_amdgcn_permlane32_swap(all, all, false, false);
                before += sub >= LPI / 2 ? q[0] : 0u;
                all = q[0] + q[1];
            }
            if (sub == 0) own.count[col] = all;
            hard = col < live && all - 1u >= (uint32_t)w_cand(NS, ICM);
            several = __builtin_amdgcn_ballot_w64(all > 1) != 0;
            uint8_t *list = own.cand[col];
            for (; n != 0; --n, ++before) {                // mostly once
                uint32_t b = bits[NW - 1], j = (NW - 1) * (IT == 32 ? 64 : 128);
#pragma unroll
                for (int w = NW - 2; w >= 0; --w) {
                    j = bits[w] != 0 ? (uint32_t)(w * (IT == 32 ? 64 : 128)) : j;
                    b = bits[w] != 0 ? bits[w] : b;
                }
                const uint32_t i = (uint32_t)__builtin_clz(b), cut = ~(0x80000000u >> i);
                j += (i & 3u) + ((i >> 2) << (IT == 32 ? 3 : 4)) + (uint32_t)(4 * sub);
                if (before < (uint32_t)w_cand(NS, ICM)) list[before] = (uint8_t)j;
                if (n > 1) {
                    uint32_t done = 0;
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        const uint32_t was = bits[w];
                        bits[w] = done == 0 ? was & cut : was;
                        done |= was;
                    }
                }
            }
        }
        wave_lds_order();
        // ---- items whose candidates say nothing (none or too many): all scores in fp32; a few items one after another, eight
        // codewords at a time by the eight owner groups, more of them on the matrix cores
        {
            uint64_t left = __builtin_amdgcn_ballot_w64(hard) & (IT == 32 ? 0xFFFFFFFFull : 0xFFFFull);
            if (left != 0 && __builtin_popcountll(left) <= w_lone(NS)) {
                const int lane = fresh(tid) & 63, og = lane >> 3, ol = lane & 7;
                constexpr int U = NS <= 1 ? 4 : NS <= 3 ? 2 : 1;           // codewords of a group under way (registers)
                do {
                    const uint32_t item = (uint32_t)__builtin_ctzll(left), p1 = item >> 3;
                    const uint32_t cur = ICM ? code[k][wave * IT + item] : 0u;
                    float v[NS][4];
#pragma unroll
                    for (int g = 0; g < NS; ++g) {
                        float o[4];
                        if (ICM) load4(codeword(k, cur), g, o, ol);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            uint32_t w = __float_as_uint(r[0][g][e]);
#pragma unroll
                            for (int p = 1; p < P; ++p) {
                                const uint32_t is = p1 == (uint32_t)p ? ~0u : 0u;          // by bits, see below
                                w = (w & ~is) | (__float_as_uint(r[p][g][e]) & is);
                            }
                            w = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((item & 7u) * 8u + (uint32_t)ol) * 4, (int)w);
                            v[g][e] = ICM ? fmaf(o[e], sr, __uint_as_float(w)) : __uint_as_float(w);
                        }
                    }
                    float least = INFINITY;
                    uint32_t f = 0;                        // 0 for the current codeword (ICM), else index + 1
                    for (int s = 0; s < m; s += 8 * U) {
                        float y[U][NS][4], cq[U], dot[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            cq[u] = cnorm[k * ICQ_LUT_W + s + 8 * u + og];
#pragma unroll
                            for (int g = 0; g < NS; ++g) load4(codeword(k, (uint32_t)(s + 8 * u + og)), g, y[u][g], ol);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            dot[u] = 0.0f;
#pragma unroll
                            for (int g = 0; g < NS; ++g)
#pragma unroll
                                for (int e = 0; e < 4; ++e) dot[u] = fmaf(v[g][e], y[u][g][e], dot[u]);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint32_t j = (uint32_t)(s + 8 * u + og), fq = ICM && j == cur ? 0u : j + 1u;
                            const float score = cq[u] - twice * group_add(dot[u]);
                            if (score < least || (score == least && fq < f)) {
                                least = score;
                                f = fq;
                            }
                        }
                    }
                    u64 key = least < INFINITY ? ((u64)icq_order_bits(least + 0.0f) << 32) | f : ~0ull;
#pragma unroll
                    for (int o = 8; o < 64; o *= 2) {
                        const u64 other = __shfl_xor(key, o, 64);
                        key = other < key ? other : key;
                    }
                    // no score a number: index 0 (ICM: the current one) stays
                    if (lane == 0) {
                        own.cand[item][0] = (uint8_t)(key == ~0ull || (uint32_t)key == 0u ? cur : (uint32_t)key - 1u);
                        own.count[item] = 1;
                    }
                    left &= left - 1;
                } while (left != 0);
                wave_lds_order();
            } else if (left != 0) {
                const int lane = fresh(tid) & 63, col = lane % IT, sub = lane / IT, og = lane >> 3, ol = lane & 7;
                // least score and the first index that has it (ICM: or the current codeword); no number, no key
                const uint32_t cur = ICM ? code[k][wave * IT + col] : 0u;
                float least = INFINITY;
                uint32_t f = 0;
                bool keep = false;
                // One tile or two at a time; 16 dimensions go from the owners through LDS, lane (item, sub) multiplies those from
                // 16 sub / LPI on.  The codewords of the next 16 are asked for before the products of these.
                constexpr int Q = 16 / LPI, U = IT == 16 || !ICM ? 2 : 1;          // (registers)
                float *F = reinterpret_cast<float *>(own.piece);           // [16 dimensions][IT]
                // ICM: the residuals wait in the workspace while v takes their registers.  Through a buffer that ends with the
                // wavefront's last item, with no branch: where `if (item < live)` stood, the compiler put copies of other values
                // in front of the point at which the lanes of missing items join again, and those lanes were left without them.
                const auto rows = __builtin_amdgcn_make_buffer_rsrc(res + i0 * d_pad, 0, live * d_pad * 4, 0x00027000);
                auto place = [&](int l, int p, int g) -> int {
                    const int e = g * 32 + (l & 7) * 4;
                    return e < d_pad ? (((l >> 3) + 8 * p) * d_pad + e) * 4 : 1 << 30;     // past the buffer: not written, read as zero
                };
                if (ICM) {
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int g = 0; g < NS; ++g) {
                            float o[4];
                            load4(codeword(k, old[p]), g, o, ol);
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint32x4, float4v{r[p][g][0], r[p][g][1], r[p][g][2], r[p][g][3]}),
                                                                   rows, place(lane, p, g), 0, 0);
#pragma unroll
                            for (int i = 0; i < 4; ++i) r[p][g][i] = fmaf(o[i], sr, r[p][g][i]);
                        }
                }
                auto half_slice = [&](int t, int q, float (&c)[U][Q]) __attribute__((always_inline)) {
                    const int e = q * 16 + sub * Q;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float *s = codeword(k, (uint32_t)((t + u) * IT + col)) + (q * 16 < d_pad ? e : 0);
#pragma unroll
                        for (int i = 0; i < Q; i += 4) {
                            const float4v a = *reinterpret_cast<const float4v *>(s + i);
#pragma unroll
                            for (int v = 0; v < 4; ++v) c[u][i + v] = a[v];
                        }
                    }
                };
#pragma nounroll
                for (int t = 0; t < ICQ_LUT_W / IT; t += U) {
                    acc_t full[U];
#pragma unroll
                    for (int v = 0; v < AV; ++v) full[0][v] = full[U - 1][v] = 0.0f;
                    float c[2][U][Q];
                    half_slice(t, 0, c[0]);
#pragma unroll
                    for (int q = 0; q < 2 * NS; ++q) {
                        const int g = q >> 1;
                        if ((ol >> 2) == (q & 1)) {
#pragma unroll
                            for (int p = 0; p < P; ++p) {
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    F[((ol & 3) * 4 + i) * IT + og + 8 * p] = r[p][g][i];
                            }
                        }
                        if (q + 1 < 2 * NS) half_slice(t, q + 1, c[(q + 1) & 1]);
                        wave_lds_order();
                        if (q * 16 < d_pad) {
#pragma unroll
                            for (int i = 0; i < Q; ++i) {
                                const float b = F[(sub * Q + i) * IT + col];
#pragma unroll
                                for (int u = 0; u < U; ++u) full[u] = Tile<IT>::full(c[q & 1][u][i], b, full[u]);
                            }
                        }
                        wave_lds_order();
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        uint32_t at = ~0u;                 // where in the tile it was improved
                        const uint32_t here = cur - (uint32_t)((t + u) * IT + 4 * sub);
#pragma unroll
                        for (int v = 0; v < AV; ++v) {
                            if (v % 4 == 0) asm volatile("" ::: "memory");
                            const uint32_t j = (uint32_t)((v & 3) + 8 * (v >> 2));
                            const float score = cnorm[k * ICQ_LUT_W + (t + u) * IT + 4 * sub + j] - twice * full[u][v];
                            if (ICM) keep = score < least ? j == here : keep || (score == least && j == here);
                            at = score < least ? j : at;
                            least = fminf(score, least);   // not NaN
                        }
                        f = at != ~0u ? (uint32_t)((t + u) * IT + 4 * sub) + at : f;
                    }
                }
                f = keep ? 0u : f + 1u;
                u64 key = least < INFINITY ? ((u64)icq_order_bits(least + 0.0f) << 32) | f : ~0ull;
#pragma unroll
                for (int o = IT; o < 64; o *= 2) {
                    const u64 other = __shfl_xor(key, o, 64);
                    key = other < key ? other : key;
                }
                // no score a number: index 0 (ICM: the current one) stays
                if (ICM) {
                    const int lane = fresh(tid) & 63;
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int g = 0; g < NS; ++g) {
                            const float4v v = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rows, place(lane, p, g), 0, 0));
#pragma unroll
                            for (int i = 0; i < 4; ++i) r[p][g][i] = v[i];
                        }
                }
                if (hard && sub == 0) {
                    own.cand[col][0] = (uint8_t)(key == ~0ull || (uint32_t)key == 0u ? cur : (uint32_t)key - 1u);
                    own.count[col] = 1;
                }
                wave_lds_order();
            }
        }
        // ---- items with several candidates, one of each owner group at a time: the argmin of the candidates' fp32 scores
        uint32_t now[P];
        if (several) {
            const int lane = fresh(tid) & 63, og = lane >> 3, ol = lane & 7;
            uint32_t many = 0;
#pragma unroll
            for (int p = 0; p < P; ++p) many |= own.count[og + 8 * p] > 1 ? 1u << p : 0u;
            while (__builtin_amdgcn_ballot_w64(many != 0) != 0) {
                const uint32_t p1 = many != 0 ? (uint32_t)__builtin_ctz(many) : 0u;
                const uint32_t item = og + 8 * p1, n = many != 0 ? own.count[item] : 0u;   // at most w_cand(NS, ICM)
                uint8_t *list = own.cand[item];
                uint32_t cur = old[0], is[P];
#pragma unroll
                for (int p = 1; p < P; ++p) {
                    is[p] = p1 == (uint32_t)p ? ~0u : 0u;
                    cur = p1 == (uint32_t)p ? old[p] : cur;
                }
                float least = INFINITY;
                uint32_t f = 0, at = 0;                    // f: 0 for the current codeword (ICM), else index + 1
                for (uint32_t i = 0; __builtin_amdgcn_ballot_w64(i < n) != 0; i += 2) {
                    if (i < n) {                           // (an item's eight lanes come here together)
                        const uint32_t q[2] = {list[i], list[i + 1 < n ? i + 1 : i]};
                        const float cq[2] = {cnorm[k * ICQ_LUT_W + q[0]], cnorm[k * ICQ_LUT_W + q[1]]};
                        float dot[2] = {0.0f, 0.0f};
#pragma unroll
                        for (int g = 0; g < NS; ++g) {
                            float y[2][4], o[4];
                            load4(codeword(k, q[0]), g, y[0], ol);
                            load4(codeword(k, q[1]), g, y[1], ol);
                            if (ICM) load4(codeword(k, cur), g, o, ol);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                uint32_t w = __float_as_uint(r[0][g][e]);                  // item p1's, by bits: a select of
#pragma unroll                                                                             // elements may end as an indexed load
                                for (int p = 1; p < P; ++p) w = (w & ~is[p]) | (__float_as_uint(r[p][g][e]) & is[p]);
                                float v = __uint_as_float(w);
                                if (ICM) v = fmaf(o[e], sr, v);
                                dot[0] = fmaf(v, y[0][e], dot[0]);
                                dot[1] = fmaf(v, y[1][e], dot[1]);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const float score = cq[u] - twice * group_add(dot[u]);
                            const uint32_t fq = ICM && q[u] == cur ? 0u : q[u] + 1u;
                            if (score < least || (score == least && fq < f) || (i + u == 0)) {
                                least = score;
                                f = fq;
                                at = q[u];
                            }
                        }
                    }
                }
                if (n != 0 && ol == 0) list[0] = (uint8_t)at;
                many &= many - 1u;
                wave_lds_order();
            }
        }
        // ---- the sub-codes, and the residual that is left
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t q = own.cand[og + 8 * p][0];
            now[p] = own.count[og + 8 * p] != 0 ? q : old[p];
            if (ol == 0) code[k][wave * IT + og + 8 * p] = (uint8_t)now[p];
        }
        if (!ICM && lev + 1 == levels) break;
        float next_sr;
#pragma unroll
        for (int p0 = 0; p0 < P; p0 += PG) {
            float c[ICM ? 1 : PG][NS][4];
            if (!ICM) {
#pragma unroll
                for (int u = 0; u < PG; ++u)
#pragma unroll
                    for (int g = 0; g < NS; ++g) load4(codeword(k, now[p0 + u]), g, c[ICM ? 0 : u][g], ol);
            }
            if (p0 == 0) {                                 // (while those are on their way)
                // the next level's scale: a level leaves residuals no longer than the longest v and its codewords
                const float reach = fmaxf((hear_reach(lev % 3) * 1.001f + ROOT_D * 6.2e-5f) / sr + cmax + (ICM ? mn.y : 0.0f), mn.y);
                next_sr = reach * sr < 32768.0f && (reach * sr >= 4.0f || sr >= sr_max) ? sr : fminf(icq_enc_scale_below(reach, 13), sr_max);
                sh.cnh[(lev + 1) & 1][tid] = -0.5f * (next_sr * mn.x) * cn;
            }
#pragma unroll
            for (int u = 0; u < PG; ++u) {
                const int p = p0 + u;
                if (ICM) {
                    if (now[p] != old[p]) {
                        if (ol == 0 && og + 8 * p < live) ++nchanged;
                        float y[NS][4];
#pragma unroll
                        for (int g = 0; g < NS; ++g) {
                            load4(codeword(k, old[p]), g, y[g], ol);
                            load4(codeword(k, now[p]), g, c[0][g], ol);
                        }
#pragma unroll
                        for (int g = 0; g < NS; ++g)
#pragma unroll
                            for (int i = 0; i < 4; ++i) r[p][g][i] = fmaf(-c[0][g][i], sr, fmaf(y[g][i], sr, r[p][g][i]));
                    }
                } else {
#pragma unroll
                    for (int g = 0; g < NS; ++g)
#pragma unroll
                        for (int i = 0; i < 4; ++i) r[p][g][i] = fmaf(-c[ICM ? 0 : u][g][i], sr, r[p][g][i]);
                }
            }
        }
        if (next_sr != sr) rescale(next_sr / sr);          // block-uniform
        wave_lds_order();                                  // an item's lanes read what one of them wrote
        if (ICM && k == K - 1 && changed) {
            const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(nchanged), 63);
            if (lane == 0 && s != 0) atomicAdd(&changed[lev / K], s);
            nchanged = 0;
        }
        mt = mn;
        sr = next_sr;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the stages asked for in vain
    __syncthreads();
    for (int i = tid; i < K * EB; i += W_THREADS) {
        const int64_t p = (int64_t)blockIdx.x * EB + i % EB;
        if (p < N) codes[(int64_t)(i / EB) * N + p] = code[i / EB][i % EB];
    }
}

}  // namespace

int icq_launch_encode_wave(const icq_index *ix, const float *x, int64_t N, uint8_t *codes, bool icm, int sweeps,
                           float *res, uint32_t *changed, hipStream_t s) {
    auto launch = [&](auto kernel, int it, size_t lds) -> int {
        ICQ_HIP_TRY(icq_allow_lds(reinterpret_cast<const void *>(kernel), (int)lds));
        kernel<<<(unsigned)((N + 4 * it - 1) / (4 * it)), W_THREADS, lds, s>>>(
            x, ix->d, ix->cb, ix->d_pad, ix->cnorm, ix->half_hi, ix->enc_meta, ix->K, ix->m, N, codes, sweeps, res, changed);
        return icq_check_launch();
    };
#define ICQ_ENC_AS(IT, NS, ICM) launch(encode_wave_kernel<IT, NS, ICM>, IT, sizeof(WaveShared<IT, NS, ICM>) + (size_t)ix->K * 4 * IT)
#define ICQ_ENC(IT, NS) return icm ? ICQ_ENC_AS(IT, NS, true) : ICQ_ENC_AS(IT, NS, false)
#define ICQ_ENC_BOTH(NS, FEW) do { if (FEW) { ICQ_ENC(16, NS); } ICQ_ENC(32, NS); } while (0)
    // 16 items a wavefront while such blocks find room beside each other (two per CU; one from 8 slices on): a level's chain of
    // steps is shorter (30000 x 128: 47 against 57 us; 15000 x 256: 61 / 83), but every codeword is read from LDS for half as
    // many items (160000 x 128: 178 / 150; 30000 x 256: 118 / 87).  16 slices, one block per CU either way: whole rounds
    // of blocks are compared, one of 128 items taking 1.95 times one of 64 (512 dimensions; 15000 items: 104 / 185, 50000: 362
    // / 347, 80000: 459 / 512).
    const int64_t cu = ix->num_cu, blocks = (N + 63) / 64;                 // of 64 items
    switch (icq_enc_slices(ix->d_pad)) {
        case 1: ICQ_ENC_BOTH(1, blocks <= 2 * cu);
        case 2: ICQ_ENC_BOTH(2, blocks <= 2 * cu);
        case 3: ICQ_ENC_BOTH(3, blocks <= 2 * cu);
        case 4: ICQ_ENC_BOTH(4, blocks <= 2 * cu);
        case 6:
            if (icm || blocks <= 2 * cu) { ICQ_ENC(16, 6); }
            return ICQ_ENC_AS(32, 6, false);
        case 8: ICQ_ENC_BOTH(8, blocks <= cu);
        case 12:
            if (icm || blocks <= cu) { ICQ_ENC(16, 12); }
            return ICQ_ENC_AS(32, 12, false);
        default:
            if (icm || (blocks + cu - 1) / cu * 20 <= ((blocks + 1) / 2 + cu - 1) / cu * 39) { ICQ_ENC(16, 16); }
            return ICQ_ENC_AS(32, 16, false);
    }
#undef ICQ_ENC_BOTH
#undef ICQ_ENC
#undef ICQ_ENC_AS
}
