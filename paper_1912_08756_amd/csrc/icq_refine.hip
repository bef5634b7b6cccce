// Stage 2 of the two-step search (arxiv 1912.08756, Eq. 1 and Sec. 3.4): for
// the survivors of the crude comparison only, finish the K-term table sum
//   D[q][i] = P[q][i] + sum_{k=Kf..K-1} lut[q][k][code_k(i)]
// and keep the per-query list of the topk nearest, ordered by (D, id).
//
// One block handles one slice of one query's candidate list.  The query's
// tables sit in LDS; each thread gathers one survivor's sub-codes (stored
// item-major, one aligned record per item) and forms D, either from the crude
// distance handed over by stage 1 plus the slow terms, or -- when stage 1 listed
// ids only -- as the whole K-term sum in the same order of additions.  Selection keeps a
// running bound: a 64-bit key (order-preserving bits of D, id) enters an LDS
// buffer only if it beats the current topk-th key; when the buffer fills it is
// sorted (bitonic) and cut back to topk, which tightens the bound.
#include "icq_internal.h"
#include "icq_sort.h"

namespace {

constexpr int RF_THREADS = ICQ_SORT_THREADS;   // block_sort runs with the whole block

__device__ __forceinline__ uint32_t order_bits(float x) { return icq_order_bits(x); }
__device__ __forceinline__ float unorder_bits(uint32_t u) { return icq_unorder_bits(u); }

// Sort the buffered keys and keep the best `topk`; returns the kept count.
// Every thread of the block must call it (contains barriers).
__device__ int compact_keys(u64 *keys, uint32_t *s_cnt, u64 *s_bound, int topk) {
    int n = (int)*s_cnt;
    __syncthreads();
    int len = 2;
    while (len < n) len <<= 1;
    for (int i = n + threadIdx.x; i < len; i += RF_THREADS) keys[i] = KEY_PAD;
    __syncthreads();
    block_sort(keys, len);
    int kept = n < topk ? n : topk;
    if (threadIdx.x == 0) {
        *s_cnt = (uint32_t)kept;
        *s_bound = n >= topk ? keys[topk - 1] : KEY_PAD;
    }
    __syncthreads();
    return kept;
}

__device__ __forceinline__ void write_result(const u64 *keys, int kept, int topk,
                                             uint32_t *out_ids, float *out_dist) {
    for (int r = threadIdx.x; r < topk; r += RF_THREADS) {
        if (r < kept) {
            out_ids[r] = (uint32_t)keys[r];
            out_dist[r] = unorder_bits((uint32_t)(keys[r] >> 32));
        } else {
            out_ids[r] = ICQ_PAD_ID;
            out_dist[r] = INFINITY;
        }
    }
}

// grid (Q * splits), block b = q * splits + slice.  LDS: keys[bufn] | tables k0..K-1,
// k0 = Kf when cand_part is given, else 0.
__global__ __launch_bounds__(RF_THREADS) void refine_kernel(
    const uint8_t *__restrict__ items, int stride, int K, int Kf, const float *__restrict__ lut,
    const uint32_t *__restrict__ cand_ids, const float *__restrict__ cand_part,
    const uint32_t *__restrict__ perm, const uint32_t *__restrict__ cand_count, int64_t cap, int topk,
    int bufn, int splits, u64 *__restrict__ keys_out, uint32_t *__restrict__ out_ids,
    float *__restrict__ out_dist) {
    extern __shared__ u64 smem64[];
    __shared__ uint32_t s_cnt;
    __shared__ u64 s_bound;
    u64 *keys = smem64;
    float *T = reinterpret_cast<float *>(keys + bufn);
    const int k0 = cand_part ? Kf : 0;
    const int q = blockIdx.x / splits, sp = blockIdx.x % splits;
    const int tid = threadIdx.x;

    for (int i = tid; i < (K - k0) * ICQ_LUT_W; i += RF_THREADS)
        T[i] = lut[((int64_t)q * K + k0) * ICQ_LUT_W + i];
    if (tid == 0) {
        s_cnt = 0;
        s_bound = KEY_PAD;
    }
    __syncthreads();

    u64 n = cand_count[q];
    if (n > (u64)cap) n = (u64)cap;
    const u64 lo = n * (u64)sp / (u64)splits, hi = n * (u64)(sp + 1) / (u64)splits;
    const uint32_t *ids = cand_ids + (int64_t)q * cap;
    const float *part = cand_part ? cand_part + (int64_t)q * cap : nullptr;
    const int w0 = k0 / 4;   // first record word that holds a needed sub-code

    for (u64 base = lo; base < hi; base += RF_THREADS) {
        const u64 idx = base + tid;
        if (idx < hi) {
            const uint32_t id = ids[idx];
            float D = part ? part[idx] : 0.0f;
            const uint32_t *rec = reinterpret_cast<const uint32_t *>(items + (size_t)id * stride);
            for (int w = w0; w * 4 < K; ++w) {
                const uint32_t word = rec[w];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = w * 4 + j;
                    if (k >= k0 && k < K) {
                        const float v = T[(k - k0) * ICQ_LUT_W + ((word >> (8 * j)) & 0xffu)];
                        D = (k == 0) ? v : D + v;
                    }
                }
            }
            const u64 key = ((u64)order_bits(D) << 32) | (perm ? perm[id] : id);
            if (key < s_bound) {
                uint32_t slot = atomicAdd(&s_cnt, 1u);
                keys[slot] = key;
            }
        }
        __syncthreads();
        const int filled = (int)s_cnt;
        __syncthreads();   // every thread has read the count before anyone appends again
        if (filled > bufn - RF_THREADS) compact_keys(keys, &s_cnt, &s_bound, topk);
    }
    const int kept = compact_keys(keys, &s_cnt, &s_bound, topk);
    if (splits == 1) {
        write_result(keys, kept, topk, out_ids + (int64_t)q * topk, out_dist + (int64_t)q * topk);
    } else {
        u64 *dst = keys_out + ((int64_t)q * splits + sp) * topk;
        for (int r = tid; r < topk; r += RF_THREADS) dst[r] = r < kept ? keys[r] : KEY_PAD;
    }
}

// grid (Q): merge the per-slice lists of one query.  LDS: keys[len], len >= splits*topk.
__global__ __launch_bounds__(RF_THREADS) void merge_kernel(const u64 *__restrict__ keys_in,
                                                           int splits, int topk, int len,
                                                           uint32_t *__restrict__ out_ids,
                                                           float *__restrict__ out_dist) {
    extern __shared__ u64 smem64[];
    u64 *keys = smem64;
    const int q = blockIdx.x;
    const int n = splits * topk;
    for (int i = threadIdx.x; i < len; i += RF_THREADS)
        keys[i] = i < n ? keys_in[(int64_t)q * n + i] : KEY_PAD;
    __syncthreads();
    block_sort(keys, len);
    // pads sort last; count the real keys among the first topk
    for (int r = threadIdx.x; r < topk; r += RF_THREADS) {
        const u64 key = keys[r];
        if (key != KEY_PAD) {
            out_ids[(int64_t)q * topk + r] = (uint32_t)key;
            out_dist[(int64_t)q * topk + r] = unorder_bits((uint32_t)(key >> 32));
        } else {
            out_ids[(int64_t)q * topk + r] = ICQ_PAD_ID;
            out_dist[(int64_t)q * topk + r] = INFINITY;
        }
    }
}

int bufn_for(int topk) { return topk <= 256 ? 2048 : 4096; }

// ------------------------------------------------------------------ distances, then bounded select
// Stage 2 runs as two kernels.
//   refine_dist_kernel: flat over all candidates of all queries, many small blocks at
//     full occupancy.  A block owns RD_BLOCK consecutive candidates of one query,
//     keeps that query's tables in LDS (one table per record byte; tables that do not
//     take part are zero, so the sum has no conditions) and writes one 64-bit key
//     (order-preserving bits of D, item id) per candidate.
//   select_kernel (icq_select.hip): the topk smallest of a query's keys.
constexpr int RD_PER = 8;                            // candidates per thread and step
constexpr int RD_STEP = RF_THREADS * RD_PER;         // 2048
constexpr int RD_BLOCK = 2 * RD_STEP;                // candidates per block

template <int WORDS>
__global__ __launch_bounds__(RF_THREADS) void refine_dist_kernel(
    const uint8_t *__restrict__ items, int K, int Kf, const float *__restrict__ lut,
    const uint32_t *__restrict__ cand_ids, const float *__restrict__ cand_part,
    const uint32_t *__restrict__ cand_count, int64_t cap, int blocks_per_query, u64 *__restrict__ keys,
    uint32_t *__restrict__ ticket) {
    __shared__ float T[4 * WORDS * ICQ_LUT_W];
    constexpr int RW = WORDS;                         // words per item record
    // Blocks are numbered piece-major: blocks that run together take the same stretch of every
    // query's list.  The lists follow the scan order, so those stretches hold ids from the same
    // regions of the item records, and a record line fetched for one query is still cached when
    // the other queries' candidates in it are gathered.
    const int nq = gridDim.x / blocks_per_query;
    const int q = blockIdx.x % nq;
    const u64 c0 = (u64)(blockIdx.x / nq) * RD_BLOCK;
    const int tid = threadIdx.x;
    u64 n = cand_count[q];
    if (n > (u64)cap) n = (u64)cap;
    if (ticket && c0 == 0 && tid == 0) ticket[q] = 0; // for the selection that follows
    if (c0 >= n) return;                              // block-uniform
    const int k0 = cand_part ? Kf : 0;
    const uint32_t *ids = cand_ids + (int64_t)q * cap;
    const float *part = cand_part ? cand_part + (int64_t)q * cap : nullptr;
    u64 *out = keys + (int64_t)q * cap;

    // Loads are unconditional with the index clamped to the last candidate: without
    // branches around them they all go out back to back and are waited for once.
    uint32_t id[2][RD_PER], rec[2][RD_PER][RW];
    float D[2][RD_PER];
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
        for (int j = 0; j < RD_PER; ++j) {
            const u64 i = c0 + (u64)st * RD_STEP + j * RF_THREADS + tid;
            const u64 ic = i < n ? i : n - 1;
            id[st][j] = ids[ic];
            D[st][j] = part ? part[ic] : 0.0f;
        }
    }
    {   // tables -> LDS
        const float4 *src = reinterpret_cast<const float4 *>(lut + (int64_t)q * K * ICQ_LUT_W);
        float4 *dst = reinterpret_cast<float4 *>(T);
        constexpr int N4 = 4 * WORDS * (ICQ_LUT_W / 4);
        float4 v[(N4 + RF_THREADS - 1) / RF_THREADS];
#pragma unroll
        for (int r = 0; r < (N4 + RF_THREADS - 1) / RF_THREADS; ++r) {
            const int i = r * RF_THREADS + tid;
            const int k = i / (ICQ_LUT_W / 4);
            v[r] = (i < N4 && k >= k0 && k < K) ? src[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int r = 0; r < (N4 + RF_THREADS - 1) / RF_THREADS; ++r) {
            const int i = r * RF_THREADS + tid;
            if (i < N4) dst[i] = v[r];
        }
    }
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
        for (int j = 0; j < RD_PER; ++j) {
            const uint32_t *p = reinterpret_cast<const uint32_t *>(items + (size_t)id[st][j] * (RW * 4));
            if (RW == 1) {
                rec[st][j][0] = p[0];
            } else if (RW == 2) {
                const uint2 v = *reinterpret_cast<const uint2 *>(p);
                rec[st][j][0] = v.x;
                rec[st][j][1 % RW] = v.y;
            } else {
#pragma unroll
                for (int w4 = 0; w4 < RW / 4; ++w4) {
                    const uint4 v = reinterpret_cast<const uint4 *>(p)[w4];
                    rec[st][j][(4 * w4) % RW] = v.x;
                    rec[st][j][(4 * w4 + 1) % RW] = v.y;
                    rec[st][j][(4 * w4 + 2) % RW] = v.z;
                    rec[st][j][(4 * w4 + 3) % RW] = v.w;
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
        for (int j = 0; j < RD_PER; ++j) {
            float d = D[st][j];
#pragma unroll
            for (int w = 0; w < WORDS; ++w) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    d += T[(w * 4 + b) * ICQ_LUT_W + ((rec[st][j][w] >> (8 * b)) & 0xffu)];
            }
            const u64 i = c0 + (u64)st * RD_STEP + j * RF_THREADS + tid;
            if (i < n) out[i] = ((u64)order_bits(d) << 32) | id[st][j];
        }
    }
}

// ------------------------------------------------------------------ stage 2 from hit bits
// icq_search with the item-by-item stage 1: stage 1 leaves one hit bit per scan position and query,
// and these kernels turn them into distances and keys.  The positions are cut into chunks of 32768
// (4 KB of hit bits per query, 512 KB of 16-byte item records).  A block belongs to ONE query --
// its tables stay in LDS for the block's whole life -- and walks a window of a few chunks, its
// four wavefronts a chunk at a time each and each on its own (no barrier after the tables are
// in place).  Workgroups go round the 8 XCDs in turn, each XCD has a cache of its own (block x of
// the grid is on XCD x % 8), and they start in the order of their numbers: the blocks are
// numbered window by window, within a window query by query, then XCD -- so the blocks of ALL
// queries of the batch that walk the same window run on the same XCD at about the same time,
// the chip holds the blocks of two windows at once, and that XCD has a few chunks' records in its
// cache at a time.  An item that survives for several queries of the batch -- or shares its cache
// line with one that does -- is then fetched from memory once: with 1 % survivors and 128
// queries that is ten uses per 128-byte line.  Per chunk and wavefront: the query's 256 words of hit
// bits (16 words per lane, a chunk ahead), the set bits expanded into a position list in the
// wavefront's part of LDS, then per position the record gather, the table reads and the key, as in
// refine_dist_kernel.
// Where a bound of the topk-th distance is known (refine_bounded_kernel) only what reaches it gets a key, else
// (refine_mask_kernel: small indexes) every survivor; ties at the bound are kept, the selection decides.
constexpr int RM_THREADS = 256;
constexpr int RM_WAVES = RM_THREADS / 64;
constexpr uint32_t RM_CHUNK = 32768;                  // positions per chunk; a multiple of the scan kernel's block step
constexpr int RM_WORDS = RM_CHUNK / 32 / 64;          // 32-bit words of hit bits per lane and chunk
constexpr int RM_PER = 4;                             // records a lane gathers together
constexpr int RM_LIST = 512;                          // positions a wavefront expands per round
static_assert(RM_LIST % (64 * RM_PER) == 0, "a round of the list is whole steps of gathers");
static_assert(RM_CHUNK <= 65536, "the position lists hold 16-bit offsets into the chunk");

// The hit bits mark a superset of the survivors (the 16-bit pre-filter of stage 1: indexes this small keep hit bits for calls of many queries
// only); an item is a survivor when the first Kf terms of its sum -- the crude distance of Eq. 2, the same fp32 additions
// stage 1 makes item by item -- are below thr[q].  Only survivors are counted and get keys.
template <int WORDS>
__global__ __launch_bounds__(RM_THREADS) void refine_mask_kernel(
    const uint8_t *__restrict__ items, int K, const float *__restrict__ lut, const uint32_t *__restrict__ masks,
    size_t mask_words, uint32_t nsel, int window, int xs_shift, int Q,
    u64 *__restrict__ keys, uint32_t *__restrict__ key_count,
    int64_t cap, uint32_t *__restrict__ cand_count, const float *__restrict__ thr, int Kf) {
    __shared__ __attribute__((aligned(16))) float T[4 * WORDS * ICQ_LUT_W];
    __shared__ uint16_t cand_all[RM_WAVES][RM_LIST];  // positions inside the chunk (RM_CHUNK <= 65536)
    __shared__ uint32_t sum_all, done_all;            // survivors of the block, wavefronts that have added theirs
    constexpr int RW = WORDS;
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint16_t *cand = cand_all[wave];
    // block -> (window, query, XCD): chunks i = (win * window + j) * 8 + xcd, j = 0 .. window - 1; wavefront
    // w takes j = w, w + 4, ..  (An index of few chunks is cut 2^xs_shift < 8 ways instead, so
    // that a block still has a window's worth of chunks for the tables it loads.)
    const uint32_t xcd = blockIdx.x & ((1u << xs_shift) - 1u), rest = blockIdx.x >> xs_shift;
    const uint32_t q = rest % (uint32_t)Q, win = rest / (uint32_t)Q;
    auto chunk_of = [&](uint32_t j) -> uint32_t {
        const uint32_t i = ((win * (uint32_t)window + j) << xs_shift) + xcd;
        return j >= (uint32_t)window || i >= nsel ? 0xFFFFFFFFu : i;
    };
    if (chunk_of(0) == 0xFFFFFFFFu) return;           // block-uniform: nothing for this block
    // Word r of this lane covers the 32 positions from c * RM_CHUNK + (r * 64 + lane) * 32: neighbouring
    // words sit in neighbouring lanes, so a dense stretch of hits is shared out among many lanes.
    // The next chunk's hit bits travel while the current one is worked on.
    const uint32_t *mq = masks + (size_t)q * mask_words + lane;
    uint32_t j = (uint32_t)wave;
    uint32_t c = chunk_of(j);
    uint32_t nxt[RM_WORDS];
    {
        const uint32_t c0 = c != 0xFFFFFFFFu ? c : 0u;
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) nxt[r] = __builtin_nontemporal_load(mq + (size_t)c0 * (RM_CHUNK / 32) + r * 64);
    }
    {   // the query's tables -> LDS, one table per record byte, zero beyond K
        const float4 *src = reinterpret_cast<const float4 *>(lut + (int64_t)q * K * ICQ_LUT_W);
        float4 *dst = reinterpret_cast<float4 *>(T);
        constexpr int N4 = 4 * WORDS * (ICQ_LUT_W / 4);
        float4 v[N4 / RM_THREADS];
#pragma unroll
        for (int u = 0; u < N4 / RM_THREADS; ++u) {
            const int i = u * RM_THREADS + tid;
            v[u] = i / (ICQ_LUT_W / 4) < K ? src[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int u = 0; u < N4 / RM_THREADS; ++u) dst[u * RM_THREADS + tid] = v[u];
    }
    const float tq = thr[q];
    u64 *kout = keys + (int64_t)q * cap;
    if (tid == 0) sum_all = done_all = 0;
    __syncthreads();                                  // the only barrier: from here on every wavefront is on its own
    uint32_t lane_survivors = 0;                      // counted per lane, summed at the end
    while (c != 0xFFFFFFFFu) {
        uint32_t w[RM_WORDS];
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) w[r] = nxt[r];
        j += RM_WAVES;
        const uint32_t cn = chunk_of(j);
        if (cn != 0xFFFFFFFFu) {
#pragma unroll
            for (int r = 0; r < RM_WORDS; ++r) nxt[r] = __builtin_nontemporal_load(mq + (size_t)cn * (RM_CHUNK / 32) + r * 64);
        }
        uint32_t mine = 0;
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) mine += (uint32_t)__builtin_popcount(w[r]);
        const uint32_t incl = wave_scan_add(mine);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        const uint32_t off = incl - mine;
        const uint32_t cbase = c * RM_CHUNK, p0 = lane * 32u;
        for (uint32_t lo = 0; lo < total; lo += RM_LIST) {      // wavefront-uniform; one round unless the chunk is dense
            wave_lds_order();                         // the last round's reads are done
            if (off + mine > lo && off < lo + RM_LIST) {
                uint32_t idx = off - lo;              // wraps below the window: fails the test until it is inside
#pragma unroll
                for (int r = 0; r < RM_WORDS; ++r) {
                    uint32_t m = w[r];
                    while (m != 0) {
                        const uint32_t bit = (uint32_t)__builtin_ctz(m);
                        m &= m - 1;
                        if (idx < (uint32_t)RM_LIST) cand[idx] = (uint16_t)(p0 + (uint32_t)r * 2048u + bit);
                        ++idx;
                    }
                }
            }
            wave_lds_order();
            const uint32_t n = total - lo < (uint32_t)RM_LIST ? total - lo : (uint32_t)RM_LIST;
            for (uint32_t base = 0; base < n; base += 64 * RM_PER) {
                uint32_t id[RM_PER], rec[RM_PER][RW];
#pragma unroll
                for (int u = 0; u < RM_PER; ++u) {
                    const uint32_t i = base + (uint32_t)u * 64u + lane;
                    id[u] = cbase + cand[i < n ? i : n - 1];
                }
#pragma unroll
                for (int u = 0; u < RM_PER; ++u) {
                    const uint32_t *p = reinterpret_cast<const uint32_t *>(items + (size_t)id[u] * (RW * 4));
                    if (RW == 1) {
                        rec[u][0] = p[0];
                    } else if (RW == 2) {
                        const uint2 v = *reinterpret_cast<const uint2 *>(p);
                        rec[u][0] = v.x;
                        rec[u][1 % RW] = v.y;
                    } else {
                        const uint4 v = *reinterpret_cast<const uint4 *>(p);
                        rec[u][0] = v.x;
                        rec[u][1 % RW] = v.y;
                        rec[u][2 % RW] = v.z;
                        rec[u][3 % RW] = v.w;
                    }
                }
                u64 key[RM_PER];
                uint64_t mk[RM_PER];
                uint32_t mycnt = 0;
#pragma unroll
                for (int u = 0; u < RM_PER; ++u) {
                    // all table reads of the record first (a read waited for before the next is asked for is a
                    // chain of 4 * WORDS LDS round trips), then the sum: k ascending like every other kernel, the
                    // first term standing for 0 + itself (no table holds -0)
                    float tv[4 * WORDS];
#pragma unroll
                    for (int x = 0; x < WORDS; ++x) {
#pragma unroll
                        for (int b = 0; b < 4; ++b) tv[x * 4 + b] = T[(x * 4 + b) * ICQ_LUT_W + ((rec[u][x] >> (8 * b)) & 0xffu)];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    float d = tv[0];
                    float crude = d;                  // the sum after its first Kf terms (Kf <= 4: inside the first word)
#pragma unroll
                    for (int i = 1; i < 4 * WORDS; ++i) {
                        d += tv[i];
                        if (i < 4) crude = i < Kf ? d : crude;
                    }
                    const uint32_t ob = icq_order_bits(d);
                    const bool keep = base + (uint32_t)u * 64u + lane < n && crude < tq;
                    lane_survivors += keep ? 1u : 0u;
                    mk[u] = __builtin_amdgcn_ballot_w64(keep);
                    mycnt += (uint32_t)__builtin_popcountll(mk[u]);
                    key[u] = (u64)ob << 32;
                }
                if (mycnt == 0) continue;             // wavefront-uniform
                uint32_t slot0 = 0;
                if (lane == 0) slot0 = atomicAdd(&key_count[q], mycnt);
                slot0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot0);
#pragma unroll
                for (int u = 0; u < RM_PER; ++u) {
                    if ((mk[u] >> lane) & 1ull) {
                        const uint64_t slot = (uint64_t)__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(mk[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk[u], slot0));
                        if (slot < (uint64_t)cap) kout[slot] = key[u] | id[u];
                    }
                    slot0 += (uint32_t)__builtin_popcountll(mk[u]);
                }
            }
        }
        c = cn;
    }
    const uint32_t survivors = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(lane_survivors), 63);
    // one addition per block: thousands of wavefronts of one query at one counter would take 11 ns each.  The last of the four
    // to come here makes it.
    if (lane == 0) {
        atomicAdd(&sum_all, survivors);
        __threadfence_block();
        if (atomicAdd(&done_all, 1u) == RM_WAVES - 1) {
            const uint32_t sum = atomicAdd(&sum_all, 0u);
            if (sum != 0) atomicAdd(&cand_count[q], sum);
        }
    }
}

// ---- the same with a bound on the result at hand
// Where a finite upper bound of the topk-th distance is known before stage 2 (icq_bound.hip, or the list of the tiles
// before), a survivor can be dropped as soon as its sum and the smallest that the tables left can add are beyond it.  With K > 8 and
// codebooks that shrink, the first eight terms do that for nearly all (10^8 items, K = 16, 1 % survivors, shrinking by 0.8: all
// but 1.3 %).  So the first half of a 16-byte record is gathered for every survivor -- over the pair ordering the halves lie
// in planes of their own, and a window of chunks is half as many bytes for the XCD's cache -- and the second half only for
// what is left, collected 64 at a time.  Where the second half's codebooks are as large as the others that is
// next to everything (by 0.9: 93 %, of one size: all), and a half record more, its tables read from memory, costs twice what the whole
// record would: such an index keeps its records whole (icq_group2.hip has the line and both sides), and all tables are in the LDS.
// Records of 16 bytes in id order come in one line, and whole (2e7, 64 queries, shrinking by 0.8 / of one size, with the second half waiting in the
// queue 331 / 1182, whole 322 / 373; 1e7, four, Kf = 2 50.5 / 105, 49.7 / 56).  K <= 8: the whole distance is known at once.
// A wavefront's positions go through a stack in LDS that outlives the chunk, so that the gathers always come 256 or 512 at a time.
// A word's lowest hit bit goes there straight; what is left of words with several (one in seven at 1 %) is collected 64
// words at a time first: with a loop over every word's bits the expansion was more than half of all vector instructions.
// What bounds it: 10^8 items, 128 queries, 1 %: 4.0 GB fetched (1.6 of hit bits) in 0.77 ms, where the kernel that gathered
// whole records took 0.92 + 0.09 ms for 5.9 GB; vector issue at half of its rate.  The fetched bytes grow with the window and
// with everything that lets the queries' wavefronts drift apart (one block per query and XCD for the whole index: 1.5 ms),
// and a wavefront lives through three chunks only, so that work at its end weighs: asking for the records of a batch before
// the last one is worked off, words instead of positions in the stack, half chunks and more wavefronts were all slower
// (0.85 to 1.0 ms).  512 gathers at a time, for indexes of many chunks, 0.74 ms (2e7 items, 64 queries, whole calls 187 / 183 us,
// 1e8, 20 queries 388 / 371; 1e7, 200 queries 247 / 254; 1e6, 1000 queries 266 / 280; 1e8, 1 query 119 / 122; 640 and more at a time are slower).
constexpr int RB_MORE = 128;                          // words with hit bits left
constexpr int RB_QUEUE = 128;                         // survivors to be finished

struct RbRest { uint32_t pos, sum; };                 // a survivor in the queue: position, bits of the sum so far

// WHOLE: records are gathered whole; else (16 bytes over the pair ordering) the halves lie in planes of their own, `items`
// and `tail`.
template <int WORDS, bool WHOLE, bool EXACT, int PER>
__global__ __launch_bounds__(RM_THREADS, 5) void refine_bounded_kernel(
    const uint8_t *__restrict__ items, const uint8_t *__restrict__ tail, int K, const float *__restrict__ lut,
    const uint32_t *__restrict__ masks, size_t mask_words, const uint32_t *__restrict__ perm, uint32_t nsel, int window,
    int xs_shift, int Q, const float *__restrict__ bound_dist, int topk, u64 *__restrict__ keys,
    uint32_t *__restrict__ key_count, int64_t cap, uint32_t *__restrict__ cand_count, const float *__restrict__ thr, int Kf) {
    constexpr bool HALF = WORDS == 4 && !WHOLE;       // a second half is left
    constexpr int FW = HALF ? 2 : WORDS;              // words of a record that are fetched
    constexpr int FT = 4 * FW;                        // their tables
    constexpr uint32_t BATCH = 64 * PER;              // survivors gathered together
    constexpr uint32_t LIST = BATCH + 64;             // positions a wavefront holds
    __shared__ __attribute__((aligned(16))) float T[FT * ICQ_LUT_W];
    __shared__ uint32_t list_all[RM_WAVES][LIST];
    __shared__ uint2 more_all[RM_WAVES][RB_MORE];     // hit bits, first position of the word
    __shared__ RbRest queue_all[RM_WAVES][RB_QUEUE];
    __shared__ float tmin[8];                         // smallest entry of each table of the second half
    __shared__ uint32_t sum_all, done_all;
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t *list = list_all[wave];
    uint2 *more = more_all[wave];
    RbRest *queue = queue_all[wave];
    // block -> (window, query, XCD) as in refine_mask_kernel
    const uint32_t xcd = blockIdx.x & ((1u << xs_shift) - 1u), rest = blockIdx.x >> xs_shift;
    const uint32_t q = rest % (uint32_t)Q, win = rest / (uint32_t)Q;
    auto chunk_of = [&](uint32_t j) -> uint32_t {
        const uint32_t i = ((win * (uint32_t)window + j) << xs_shift) + xcd;
        return j >= (uint32_t)window || i >= nsel ? 0xFFFFFFFFu : i;
    };
    if (chunk_of(0) == 0xFFFFFFFFu) return;           // block-uniform: nothing for this block
    const uint32_t *mq = masks + (size_t)q * mask_words + lane;
    uint32_t j = (uint32_t)wave, c = chunk_of(j);
    uint32_t w[RM_WORDS];
#pragma unroll
    for (int r = 0; r < RM_WORDS; ++r) w[r] = __builtin_nontemporal_load(mq + (c != 0xFFFFFFFFu ? c * (RM_CHUNK / 32) : 0u) + r * 64);
    const float *Tq = lut + (int64_t)q * K * ICQ_LUT_W;
    {
        const float4 *src = reinterpret_cast<const float4 *>(Tq);
        float4 *dst = reinterpret_cast<float4 *>(T);
#pragma unroll
        for (int u = 0; u < FT / 4; ++u) {            // tables per wavefront
            const int i = u * RM_THREADS + tid;
            dst[i] = u * 4 + wave < K ? src[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        if (HALF) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = 8 + u * 4 + wave;       // table k, whole
                const float4 v = k < K ? src[k * (ICQ_LUT_W / 4) + (int)lane] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                const float m = wave_min_f32(fminf(fminf(v.x, v.y), fminf(v.z, v.w)));
                if (lane == 0) tmin[u * 4 + wave] = m;
            }
        }
    }
    const float bound_f = bound_dist[(int64_t)q * topk + topk - 1];
    uint32_t bound = icq_order_bits(bound_f);
    const bool open = bound >= 0xFF800000u;           // infinite or not a number
    if (open) bound = 0xFFFFFFFFu;
    const float tq = EXACT ? thr[q] : 0.0f;
    if (tid == 0) sum_all = done_all = 0;
    __syncthreads();                                  // the only barrier: from here on every wavefront is on its own
    // A sum of eight terms above `most` cannot come to the bound: the eight additions that follow give no less than the same
    // ones of the tables' smallest entries would (rounding is monotone), which is (sum + those entries) (1 +- 8 * 2^-24); 1e-5
    // covers that and the roundings here.  Open bounds and tables without a number drop nothing.
    float most = INFINITY;
    if (HALF && !open) {
        float s = 0.0f, a = fabsf(bound_f);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            s += tmin[k];
            a += fabsf(tmin[k]);
        }
        most = (bound_f - s) + 1e-5f * a;
    }
    uint32_t lane_survivors = 0;
    u64 *kout = keys + (int64_t)q * cap;
    uint32_t n = 0, nm = 0, nq = 0;                   // positions, words with bits left, survivors in the queue (wavefront-uniform)
    // the queue's last `cnt` (at most 64): the remaining terms, and a key for what reaches the bound
    auto finish = [&](uint32_t cnt) __attribute__((always_inline)) {
        wave_lds_order();
        const bool in = lane < cnt;
        const RbRest e = queue[nq - cnt + (in ? lane : 0u)];
        nq -= cnt;
        float d = __uint_as_float(e.sum);
        if (HALF) {
            const uint2 r = reinterpret_cast<const uint2 *>(tail)[e.pos];
            float tv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t code = ((i < 4 ? r.x : r.y) >> (8 * (i & 3))) & 0xffu;
                tv[i] = 8 + i < K ? Tq[(8 + i) * ICQ_LUT_W + code] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) d += tv[i];
        }
        const uint32_t ob = icq_order_bits(d);
        const bool keep = in && ob <= bound;
        const uint64_t mk = __builtin_amdgcn_ballot_w64(keep);
        if (mk == 0) return;                          // wavefront-uniform
        uint32_t slot0 = 0;
        if (lane == 0) slot0 = atomicAdd(&key_count[q], (uint32_t)__builtin_popcountll(mk));
        slot0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot0);
        if (keep) {
            const uint64_t slot = (uint64_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, slot0));
            if (slot < (uint64_t)cap) kout[slot] = ((u64)ob << 32) | (perm ? perm[e.pos] : e.pos);
        }
    };
    // the list's last `cnt` (at most BATCH)
    auto batch = [&](uint32_t cnt) __attribute__((always_inline)) {
        wave_lds_order();
        uint32_t pos[PER], rec[PER][FW];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const uint32_t i = (uint32_t)u * 64u + lane;
            pos[u] = list[n - cnt + (i < cnt ? i : cnt - 1)];
        }
        n -= cnt;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (FW == 1) {
                rec[u][0] = reinterpret_cast<const uint32_t *>(items)[pos[u]];
            } else if (FW == 2) {
                const uint2 x = reinterpret_cast<const uint2 *>(items)[pos[u]];
                rec[u][0] = x.x;
                rec[u][1 % FW] = x.y;
            } else {
                const uint4 x = reinterpret_cast<const uint4 *>(items)[pos[u]];
                rec[u][0] = x.x;
                rec[u][1 % FW] = x.y;
                rec[u][2 % FW] = x.z;
                rec[u][3 % FW] = x.w;
            }
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            // all table reads of the (half) record first, then the sum: k ascending like every other kernel, the first term
            // standing for 0 + itself (no table holds -0)
            float tv[FT];
#pragma unroll
            for (int x = 0; x < FT; ++x) tv[x] = T[x * ICQ_LUT_W + ((rec[u][x / 4] >> (8 * (x % 4))) & 0xffu)];
            __builtin_amdgcn_sched_barrier(0);
            float d = tv[0], crude = d;               // crude: the sum of the first Kf terms (Kf <= 4)
#pragma unroll
            for (int i = 1; i < FT; ++i) {
                d += tv[i];
                if (EXACT && i < 4) crude = i < Kf ? d : crude;
            }
            bool keep = (uint32_t)u * 64u + lane < cnt;
            if (EXACT) keep = keep && crude < tq;
            lane_survivors += keep ? 1u : 0u;
            keep = keep && (HALF ? !(d > most) : icq_order_bits(d) <= bound);
            const uint64_t mk = __builtin_amdgcn_ballot_w64(keep);
            if (mk == 0) continue;                    // wavefront-uniform
            if (keep)
                queue[__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, nq))] = {pos[u], __float_as_uint(d)};
            nq += (uint32_t)__builtin_popcountll(mk);
            if (nq >= 64u) finish(64u);
        }
    };
    // the lowest hit bit of every lane's word m (positions from `at`) -> list; returns the others
    auto emit = [&](uint32_t m, uint32_t at) __attribute__((always_inline)) -> uint32_t {
        const uint64_t mk = __builtin_amdgcn_ballot_w64(m != 0);
        if (m != 0)
            list[__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, n))] = at + (uint32_t)__builtin_ctz(m);
        n += (uint32_t)__builtin_popcountll(mk);
        if (n > BATCH) batch(BATCH);
        return m & (m - 1);
    };
    // the last `cnt` words (at most 64) with bits left
    auto drain = [&](uint32_t cnt) __attribute__((always_inline)) {
        wave_lds_order();
        uint2 e = more[nm - cnt + (lane < cnt ? lane : 0u)];
        nm -= cnt;
        if (lane >= cnt) e.x = 0;
        while (__builtin_amdgcn_ballot_w64(e.x != 0) != 0) e.x = emit(e.x, e.y);
    };
    while (c != 0xFFFFFFFFu) {
        uint32_t v[RM_WORDS];
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) v[r] = w[r];
        const uint32_t at = c * RM_CHUNK + lane * 32u;
        j += RM_WAVES;
        c = chunk_of(j);
        if (c != 0xFFFFFFFFu) {
#pragma unroll
            for (int r = 0; r < RM_WORDS; ++r) w[r] = __builtin_nontemporal_load(mq + (size_t)c * (RM_CHUNK / 32) + r * 64);
        }
#pragma nounroll                                       // (the register of word r by index: unrolled it is 20000 instructions)
        for (int r = 0; r < RM_WORDS; ++r) {
            const uint32_t left = emit(v[r], at + (uint32_t)r * 2048u);
            const uint64_t mk = __builtin_amdgcn_ballot_w64(left != 0);
            if (mk == 0) continue;                    // wavefront-uniform
            if (left != 0)
                more[__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, nm))] =
                    make_uint2(left, at + (uint32_t)r * 2048u);
            nm += (uint32_t)__builtin_popcountll(mk);
            if (nm >= 64u) drain(64u);
        }
    }
    if (nm != 0) drain(nm);
    while (n != 0) batch(n < BATCH ? n : BATCH);
    if (nq != 0) finish(nq);
    const uint32_t survivors = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(lane_survivors), 63);
    // one addition per block, as above
    if (lane == 0) {
        atomicAdd(&sum_all, survivors);
        __threadfence_block();
        if (atomicAdd(&done_all, 1u) == RM_WAVES - 1) {
            const uint32_t sum = atomicAdd(&sum_all, 0u);
            if (sum != 0) atomicAdd(&cand_count[q], sum);
        }
    }
}

}  // namespace

// Item records of at most 16 bytes take the bounded-stream kernel; wider records
// (K > 16) the generic streaming kernel.
bool icq_selects(const icq_index *ix, int topk) { return ix->item_stride <= 16 && topk <= 512; }

// Parts a query's work is cut into: the selection of the keys, or (wider records, longer results) the slices of
// the generic kernel's candidate list.
int icq_stage2_splits(const icq_index *ix, int Q, int64_t cap, int topk) {
    if (Q <= 0) return 1;
    if (icq_selects(ix, topk)) return icq_select_splits(ix, Q, cap, topk);
    int64_t s = (4LL * ix->num_cu + Q - 1) / Q;
    int64_t by_len = cap / 2048 + 1;            // do not slice short lists
    int64_t by_merge = 4096 / topk;             // merge buffer holds splits*topk keys
    if (s > by_len) s = by_len;
    if (s > by_merge) s = by_merge;
    if (s > 64) s = 64;
    if (s < 1) s = 1;
    return (int)s;
}

int icq_launch_refine(const icq_index *ix, const float *lut, int Q, const uint32_t *cand_ids,
                      const float *cand_part, int list_kind,
                      const uint32_t *cand_count, int64_t cap, int topk, int splits, u64 *keys,
                      uint32_t *ticket, uint32_t *out_ids, float *out_dist, hipStream_t s) {
    if (Q == 0 || list_kind == ICQ_LIST_DONE) return ICQ_OK;
    const uint8_t *items = list_kind == ICQ_LIST_POSITIONS ? ix->items_grouped : ix->items;
    const uint32_t *perm = list_kind == ICQ_LIST_POSITIONS ? ix->perm : nullptr;
    const unsigned grid = (unsigned)Q * (unsigned)splits;
    const size_t tab = sizeof(float) * (size_t)(cand_part ? ix->Ks : ix->K) * ICQ_LUT_W;
    if (icq_selects(ix, topk)) {
        // distances for every candidate (flat), then the per-query select over the keys
        int64_t len = cap < ix->N ? cap : ix->N;
        const int bpq = len > 0 ? (int)((len + RD_BLOCK - 1) / RD_BLOCK) : 1;
        const unsigned dgrid = (unsigned)Q * (unsigned)bpq;
        if (list_kind != ICQ_LIST_KEYS) {
            auto launch = [&](auto kernel) {
                kernel<<<dgrid, RF_THREADS, 0, s>>>(items, ix->K, ix->Kf, lut, cand_ids, cand_part, cand_count, cap, bpq, keys,
                                                    ticket);
            };
            switch (ix->item_stride) {
                case 4: launch(refine_dist_kernel<1>); break;
                case 8: launch(refine_dist_kernel<2>); break;
                default: launch(refine_dist_kernel<4>); break;
            }
            if (icq_check_launch() != ICQ_OK) return ICQ_ERR_HIP;
        }
        return icq_launch_select(keys, cand_count, cap, Q, topk, splits, ticket, out_ids,
                                 out_dist, s);
    }
    const int bufn = bufn_for(topk);
    const size_t lds = sizeof(u64) * bufn + tab;
    ICQ_HIP_TRY(icq_allow_lds(reinterpret_cast<const void *>(&refine_kernel), 98304));
    refine_kernel<<<grid, RF_THREADS, lds, s>>>(items, ix->item_stride, ix->K, ix->Kf, lut, cand_ids, cand_part, perm,
                                                cand_count, cap, topk, bufn, splits, keys, out_ids, out_dist);
    if (icq_check_launch() != ICQ_OK) return ICQ_ERR_HIP;
    if (splits == 1) return ICQ_OK;
    // join the slices' lists, KEY_PAD where one is short (splits * topk <= 4096)
    if (topk <= 512)
        return icq_launch_select(keys, nullptr, (int64_t)splits * topk, Q, topk, 1, nullptr, out_ids, out_dist, s);
    int len = 2;
    while (len < splits * topk) len <<= 1;
    merge_kernel<<<Q, RF_THREADS, sizeof(u64) * len, s>>>(keys, splits, topk, len, out_ids, out_dist);
    return icq_check_launch();
}

ICQ_EXPORT int icq_refine(const icq_index *ix, const float *lut, int Q, const uint32_t *cand_ids,
                          const float *cand_part, const uint32_t *cand_count, int64_t cap, int topk,
                          uint32_t *out_ids, float *out_dist, void *workspace,
                          size_t workspace_bytes, void *stream) {
    if (!ix || Q < 0 || Q > ICQ_MAX_Q || cap < 1 || topk < 1 || topk > ICQ_MAX_TOPK)
        return ICQ_ERR_ARG;
    if (Q == 0) return ICQ_OK;
    if (!lut || !cand_ids || !cand_count || !out_ids || !out_dist) return ICQ_ERR_ARG;
    if ((double)Q * (double)cap >= 1099511627776.0) return ICQ_ERR_ARG;
    icq_ws_layout L = icq_layout(ix, Q, cap, topk, false, false);
    if (L.total > 0 &&
        (!workspace || ((uintptr_t)workspace % ICQ_ALIGN) != 0 || workspace_bytes < L.total))
        return ICQ_ERR_WORKSPACE;
    u64 *keys = reinterpret_cast<u64 *>(static_cast<char *>(workspace) + L.keys_off);
    return icq_launch_refine(ix, lut, Q, cand_ids, cand_part, ICQ_LIST_IDS, cand_count, cap, topk,
                             L.splits, keys, L.tickets ? reinterpret_cast<uint32_t *>(static_cast<char *>(workspace) + L.ticket_off) : nullptr,
                             out_ids, out_dist, (hipStream_t)stream);
}

// From 2^22 items on; with the pre-filters (eight or sixteen queries per pass of stage 1) and enough queries to fill the
// chunk walk already from 2^19 (1000 queries, K = 16: lists are ahead up to 3e5 items, hit bits from 6e5).  Below that the item
// records stay in the caches whatever the order of the gathers, and candidate lists with the flat distance kernel are quicker.
bool icq_masks_usable(const icq_index *ix, int Q, int topk) {
    const bool large = ix->N >= (1ll << 22) || (ix->N >= (1ll << 19) && Q >= 32 && icq_scan_q16_usable(ix, Q));
    return ix->Kf <= 4 && !icq_group_usable(ix, Q) && icq_selects(ix, topk) && large &&
           ix->N + 16ll * 65536 < (1ll << 31);
}

int64_t icq_mask_scan_end(const icq_index *ix, bool pairs) {
    const int64_t npos = pairs ? ix->g2_npos : ix->N;
    return (npos + RM_CHUNK - 1) / RM_CHUNK * RM_CHUNK;
}

int icq_launch_refine_masks(const icq_index *ix, const float *lut, int Q, const uint16_t *masks, size_t mask_stride,
                            int64_t scan_end, bool pairs, int64_t cap, int topk, int splits, u64 *keys, uint32_t *key_count,
                            uint32_t *ticket, uint32_t *cand_count, const float *thr, bool superset, const float *bound_dist,
                            uint32_t *out_ids, float *out_dist, hipStream_t s) {
    if (Q == 0) return ICQ_OK;
    const bool halves = pairs && ix->g2_halves;
    const uint8_t *items = pairs ? ix->items_grouped : ix->items;
    const uint32_t *perm = pairs ? ix->perm : nullptr;
    const uint32_t chunks = (uint32_t)(scan_end / RM_CHUNK);
    const uint64_t visits = (uint64_t)chunks * (uint64_t)Q;
    // From 128 chunks on (2^22 items), and over the pair ordering, a bound is worth its launch of 8 to 12 us (20 to 40 for hundreds of queries).  Whole calls, us, one
    // unfiltered launch (up to 130 chunks; beyond, behind one over every 65th chunk) / bounded: K = 16: 7.8e5 items, 37 queries
    // 43 / 47; 1e6, 1000 queries (id order) 330 / 333; 4.3e6, 1 / 3 / 8 queries 44 / 39, 56 / 43, 76 / 52; 1e7, 16 queries, 30 % 765 / 146;
    // 2e7, 64 queries 340 / 198; 1e8, 1 / 128 queries 161 / 104, 1797 / 1536; K = 12, Kf = 3, 1e7, 100 queries, 10 % 873 / 305;
    // K = 8, Kf = 2, 1e7, 1 query 49 / 35, 1.3e7, 4 queries 83 / 47.
    if (pairs || chunks >= 128) {
        const int rc = icq_launch_near_bound(ix, lut, Q, thr, topk, masks, mask_stride, scan_end, pairs, cap, bound_dist, out_dist, s);
        if (rc != ICQ_OK) return rc;
        bound_dist = out_dist;
    }
    // Chunks per block: few, so that the blocks in flight (two windows' worth when the queries fill the chip) keep to a few
    // chunks per XCD, but enough to be worth the tables a block loads.  Bounded: up to three per wavefront while that leaves a
    // block for every place on the chip (1e8 items, 128 queries, windows of 4 / 8 / 12 / 16 / 24: 1675 / 1545 / 1536 / 1541 / 1570 us;
    // 1 query 104 / 109 / 115 / 119; 2e6, 80 queries 81 / 73 / 77; 3e7, 20 queries - / 144 / 149; 1e7, 60 queries 119 / 117 / 118; 1e8 in
    // id order, 128 queries 2641 / 2589 / 2790).  Unfiltered: one per wavefront while that is
    // all the parallelism there is, else full windows, and the chunks cut fewer than 8 ways when 8 windows' worth do not
    // exist: 16 MB of records stay in the caches wherever the blocks run.
    // (with thousands of queries a window's blocks no longer run at the same time, and the 8-way cut that
    // keeps a chunk's records in ONE L2 is worth more than the longer windows: 1e4 queries, 1e6 items,
    // 8-byte records: 0.80 ms with it, 0.83 without)
    struct plan { int window, xs_shift; unsigned grid; };
    auto plan_for = [&](int window) -> plan {
        int xs_shift = 3;
        if (bound_dist) {
            // Few windows: four ways where the last of eight would leave a sixth of the wavefronts without a chunk (2e6 items, 200
            // queries, windows of 8 cut 8 / 4 / 1 ways 117 / 105 / 116 us; 1e6, 1000 queries, of 12, 4 / 1 ways 265 / 278)
            const uint32_t places = (chunks + ((uint32_t)window << 3) - 1) / ((uint32_t)window << 3) * ((uint32_t)window << 3);
            if (places * 5u > chunks * 6u) xs_shift = 2;
            while (xs_shift > 0 && ((uint32_t)window << (xs_shift - 1)) >= chunks) --xs_shift;
        } else {
            while (Q <= 2048 && xs_shift > 0 && ((uint32_t)window << xs_shift) > chunks) --xs_shift;
        }
        const int most = (int)((chunks + (1u << xs_shift) - 1) >> xs_shift);
        if (window > most) window = most > 0 ? most : 1;
        const unsigned per_win = (unsigned)window << xs_shift;
        return {window, xs_shift, ((chunks + per_win - 1) / per_win * (unsigned)Q) << xs_shift};
    };
    const size_t mask_words = mask_stride / 2;
    const uint32_t *m32 = reinterpret_cast<const uint32_t *>(masks);
    if (bound_dist) {
        const uint8_t *tail = halves ? reinterpret_cast<const uint8_t *>(ix->g2_halves + ix->g2_npad) : nullptr;
        auto go = [&](auto kernel, const uint8_t *from, int window) {
            const plan p = plan_for(window);
            kernel<<<p.grid, RM_THREADS, 0, s>>>(from, tail, ix->K, lut, m32, mask_words, perm, chunks, p.window, p.xs_shift, Q,
                                                 bound_dist, topk, keys, key_count, cap, cand_count, thr, ix->Kf);
        };
        const int window = visits < 5000u ? 4 : visits < 40000u || !pairs ? 8 : 12;
#define ICQ_RB(W, WHOLE, FROM, WIN)                                                               \
    do {                                                                                         \
        if (superset) go(refine_bounded_kernel<W, WHOLE, true, RM_PER>, FROM, WIN);              \
        else go(refine_bounded_kernel<W, WHOLE, false, RM_PER>, FROM, WIN);                      \
    } while (0)
        if (ix->item_stride == 4) ICQ_RB(1, true, items, window);
        else if (ix->item_stride == 8) ICQ_RB(2, true, items, window);
        else if (!halves) {
            // (whole records leave the caches sooner, so the windows are shorter: codebooks shrinking by 0.9, 1e8 items, 128 queries, windows of
            // 8 / 12 / 16: 1827 / 1962 / 1996 us; of one size, 1e7, 16 queries, 30 %, 4 / 8: 303 / 329; 2e7, 64 queries 293 / 298)
            ICQ_RB(4, true, items, !pairs ? window : visits < 40000u ? 4 : 8);
        } else {
            const uint8_t *first = reinterpret_cast<const uint8_t *>(ix->g2_halves);
            // (a wavefront's gathers at a time: see the kernel; fewer than six queries have no superset, and so many chunks only beyond 1.6e8 items)
            if (superset && chunks >= 600 && visits >= 30000u) go(refine_bounded_kernel<4, false, true, 8>, first, window);
            else ICQ_RB(4, false, first, window);
        }
#undef ICQ_RB
    } else {
        auto go = [&](auto kernel) {
            const plan p = plan_for(visits <= 16384u ? 4 : 16);
            kernel<<<p.grid, RM_THREADS, 0, s>>>(items, ix->K, lut, m32, mask_words, chunks, p.window, p.xs_shift, Q, keys, key_count, cap,
                                                 cand_count, thr, ix->Kf);
        };
        if (ix->item_stride == 4) go(refine_mask_kernel<1>);
        else if (ix->item_stride == 8) go(refine_mask_kernel<2>);
        else go(refine_mask_kernel<4>);
    }
    if (icq_check_launch() != ICQ_OK) return ICQ_ERR_HIP;
    return icq_launch_select(keys, key_count, cap, Q, topk, splits, ticket, out_ids, out_dist, s);
}
