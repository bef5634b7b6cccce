// Both stages of the two-step search (arxiv 1912.08756, Eq. 2 and Eq. 1) in one kernel, for an index of few items:
// a small database, or the first tiles of the running search, where every item or every fifth one survives.
//
// A block takes 4096 items at a time for one query (2048 where many queries meet few items: icq_launch_small): their crude distances from the query's tables in LDS, the
// survivors compacted into a list in LDS, and that list's exact distances as keys (order-preserving bits of D, id)
// for the selection.  No candidate list goes through memory, the codes are read from the item records that the
// second stage needs as well, and a list slot in memory is reserved once per 4096 items instead of once per
// wavefront (one query's reservations go to one counter at 11 ns each: with 2048 items a step 10^6 items took 23.6 us, now 20.8; 8192
// a step leave too few blocks, 3e5 items 15.8 / 17.6).  The table reads collide in LDS banks (codes are random, one copy of the tables, about five clocks per 64
// reads); scan_stream_kernel's copies avoid that, but its block of 16384 items and its 128 KB of tables leave most of the
// chip idle here and its lists cost atomics.
// What bounds it: the LDS while survivors are few, the keys' stores when all survive (both sides: icq_small_usable).
// The running search's first two tiles, 128 queries, K = 16, Kf = 4 (scan + distances before, this kernel now): 8192 items,
// all surviving, 60 -> 12 us; 32768 items 26 -> 15 us.
#include "icq_internal.h"
#include "icq_sort.h"

namespace {

constexpr int SM_PER = 4;                            // items per thread and step

// items [N] records of WORDS words; thr [Q], Q = gridDim.y; keys [Q][cap]; count [Q] zero on entry, N <= ICQ_MAX_N
// (a step past it still fits 32 bits).
// Block x takes the items [x * per, (x + 1) * per), per a multiple of the step.
template <int WORDS, int SM_THREADS>
__global__ __launch_bounds__(SM_THREADS) void small_search_kernel(
    const uint8_t *__restrict__ items, uint32_t N, int K, int Kf, const float *__restrict__ lut,
    const float *__restrict__ thr, uint32_t per, u64 *__restrict__ keys, int64_t cap, uint32_t *__restrict__ count) {
    constexpr int SM_STEP = SM_THREADS * SM_PER;
    static_assert(SM_STEP <= 65536, "the list holds 16-bit offsets");
    __shared__ __attribute__((aligned(16))) float T[4 * WORDS * ICQ_LUT_W];      // a table per record byte, zero beyond K
    __shared__ float list_p[SM_STEP];
    __shared__ uint16_t list_i[SM_STEP];
    __shared__ uint32_t s_n, s_at;
    const int tid = threadIdx.x, q = blockIdx.y;
    const uint32_t lane = tid & 63;
    const uint32_t begin = blockIdx.x * per, end = N - begin < per ? N : begin + per;
    {
        const float4 *src = reinterpret_cast<const float4 *>(lut + (int64_t)q * K * ICQ_LUT_W);
        for (int i = tid; i < WORDS * ICQ_LUT_W; i += SM_THREADS)
            reinterpret_cast<float4 *>(T)[i] = i / (ICQ_LUT_W / 4) < K ? src[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    const float t = thr[q];
    const uint32_t *rec = reinterpret_cast<const uint32_t *>(items);
    u64 *out = keys + (int64_t)q * cap;
    for (uint32_t base = begin; base < end; base += SM_STEP) {
        uint32_t w[SM_PER];
#pragma unroll
        for (int j = 0; j < SM_PER; ++j) {
            const uint32_t i = base + j * SM_THREADS + tid;
            w[j] = rec[(size_t)(i < end ? i : end - 1) * WORDS];
        }
        if (tid == 0) s_n = 0;
        __syncthreads();                             // tables there; the list of the step before consumed
        float P[SM_PER];
#pragma unroll
        for (int j = 0; j < SM_PER; ++j) {           // Eq. 2, k ascending; Kf <= 4
            P[j] = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < Kf) P[j] += T[k * ICQ_LUT_W + ((w[j] >> (8 * k)) & 0xffu)];
        }
        uint64_t hit[SM_PER];
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < SM_PER; ++j) {
            hit[j] = __builtin_amdgcn_ballot_w64(P[j] < t && base + j * SM_THREADS + tid < end);
            n += (uint32_t)__builtin_popcountll(hit[j]);
        }
        uint32_t at = 0;
        if (n != 0) {                                // wavefront-uniform
            if (lane == 0) at = atomicAdd(&s_n, n);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
            for (int j = 0; j < SM_PER; ++j) {
                if ((hit[j] >> lane) & 1) {
                    const uint32_t slot = at + (uint32_t)__builtin_popcountll(hit[j] & ((1ull << lane) - 1));
                    list_i[slot] = (uint16_t)(j * SM_THREADS + tid);
                    list_p[slot] = P[j];
                }
                at += (uint32_t)__builtin_popcountll(hit[j]);
            }
        }
        __syncthreads();
        n = s_n;
        if (tid == 0 && n != 0) s_at = atomicAdd(&count[q], n);
        __syncthreads();
        for (uint32_t e = tid; e < n; e += SM_THREADS) {
            const uint32_t id = base + list_i[e];
            float D = list_p[e];
            uint32_t r[WORDS];
#pragma unroll
            for (int v = 0; v < WORDS; ++v) r[v] = rec[(size_t)id * WORDS + v];
#pragma unroll
            for (int k = 0; k < 4 * WORDS; ++k)      // Eq. 1: the terms behind the crude distance's
                if (k >= 4 || k >= Kf) D += T[k * ICQ_LUT_W + ((r[k / 4] >> (8 * (k % 4))) & 0xffu)];
            const u64 slot = (u64)s_at + e;
            if (slot < (u64)cap) out[slot] = ((u64)icq_order_bits(D) << 32) | id;
        }
    }
}

}  // namespace

// Where the line lies: with few survivors the scan with its conflict-free table copies is ahead once there are enough
// (query, item) pairs to fill the chip with it; what it costs with many survivors moves the line (us per search at 1 %
// survivors, K = 16, Kf = 4, lists / this: 1 x 131072 26.0 / 18.5, 8 x 131072 30.0 / 23.9, 128 x 8192 27.3 / 20.7,
// 8 x 200000 30.9 / 27.5, 37 x 65536 29.4 / 31.5, 128 x 32768 29.2 / 31.4, 1000 x 32768 63 / 90; at 20 %: 128 x 8192
// 35.6 / 21.9, 128 x 32768 47.4 / 35.2, 1000 x 32768 117 / 108; all surviving: 128 x 8192 75.5 / 27.3,
// 1000 x 131072 2253 / 900.  Kf = 1, 2, 3: the same line within 20 %.  Those with 2048 items a step; with 4096, lists / this:
// 1 x 2.5e6 33.6 / 29.0, 1 x 4e6 35.4 / 34.2, 4 x 5e5 29.0 / 21.1, 3 x 10^6 28.0 / 25.5, 5 x 10^6 33.6 / 37.0, 8 x 5e5 29.3 / 29.7,
// 100 x 30000 25.3 / 23.9, 700 x 5000 31.5 / 31.7; at 0.1 %: 4 x 7e5 23.0 / 24.5, 28 x 10^5 24.1 / 22.4; at 5 %: 39.7 / 33.5,
// 30.7 / 24.1: next to the line lists may be ahead by 6 % where next to nothing survives.  Against 2048 items a step and a line at
// 1.8e6 pairs, 816 calls of 1.5e6 to 2.9e6 pairs at 0.05 % to all surviving: 0.69 of the time, none 4 % slower).
bool icq_small_usable(const icq_index *ix, int Q, int topk, icq_share share) {
    const double pairs = (double)Q * (double)ix->N;
    return ix->scan_mode == ICQ_SCAN_AUTO && ix->Kf <= 4 && ix->item_stride <= 16 && topk <= 512 &&
           (share == ICQ_SHARE_ALL || pairs <= (share == ICQ_SHARE_MANY ? 5.0e6 : 3.0e6));
}

int icq_launch_small(const icq_index *ix, const float *lut, int Q, const float *thr, unsigned long long *cand_keys,
                     uint32_t *cand_count, int64_t cap, hipStream_t s) {
    // 1024 threads, or 512 where those cover the index in one step (the other half would only wait at the barriers) and the
    // blocks are more than two per CU, the most that run at a time with 1024: then the next ones start earlier.  K = 12, 2 %
    // surviving, 1024 / 512 threads in us: 520 queries over 700, 1300, 2048 items 18.0 / 16.3, 19.8 / 18.0, 20.1 / 18.6; 1000
    // queries 23.5 / 21.3, 26.4 / 24.3, 27.8 / 26.1; 3000 over 700 47.7 / 41.2.  Up to 512 queries the two are within 2 %, and past
    // 2048 items (to 4096) 512 threads take 7 to 15 % longer for 300 to 1000 queries.
    const int threads = ix->N <= 512 * SM_PER && Q > 2 * ix->num_cu ? 512 : 1024;
    const int64_t step = threads * SM_PER;
    // about eight blocks per CU, of which two run at a time; beyond that a block takes more steps with the tables it has loaded
    int64_t chunks = (8ll * ix->num_cu + Q - 1) / Q;
    const int64_t most = (ix->N + step - 1) / step;
    if (chunks > most) chunks = most;
    const uint32_t per = (uint32_t)(((ix->N + chunks - 1) / chunks + step - 1) / step * step);
    const dim3 grid((unsigned)((ix->N + per - 1) / per), (unsigned)Q);
#define ICQ_SM_AS(W, THREADS)                                                                                      \
    small_search_kernel<W, THREADS><<<grid, THREADS, 0, s>>>(ix->items, (uint32_t)ix->N, ix->K, ix->Kf, lut, thr, per, cand_keys, \
                                                             cap, cand_count)
#define ICQ_SM_LAUNCH(W) do { if (threads == 512) ICQ_SM_AS(W, 512); else ICQ_SM_AS(W, 1024); } while (0)
    switch (ix->item_stride) {
        case 4: ICQ_SM_LAUNCH(1); break;
        case 8: ICQ_SM_LAUNCH(2); break;
        default: ICQ_SM_LAUNCH(4); break;
    }
#undef ICQ_SM_LAUNCH
#undef ICQ_SM_AS
    return icq_check_launch();
}
