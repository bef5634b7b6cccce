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
// and this kernel turns them into distances and keys.  The positions are cut into chunks of 32768
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
// bits (one 128-bit load per lane, two chunks ahead), a prefix of their popcounts, the set bits
// expanded into a position list in the wavefront's part of LDS, then per position the record
// gather, the K table reads and the key, as in refine_dist_kernel.
// (A wavefront may take half or a quarter of a chunk, see icq_launch_refine_masks; what follows says chunk for either.)
// Every 65th chunk (or every 65th quarter of one, seed_parts = 4) is done in a first launch, unfiltered
// (!FILTER); the select kernel's topk-th
// distance of those keys then bounds what the others add in a second launch (FILTER: keys
// above it are dropped; ties at it are kept, the final select decides).  The final lists are
// unchanged -- at least topk keys at or below the bound are already there -- and the key lists
// shrink to a few per cent.  Survivors are counted from the popcounts, added up per block.
constexpr int RM_THREADS = 256;
constexpr int RM_WAVES = RM_THREADS / 64;
constexpr uint32_t RM_CHUNK = 32768;                  // positions per chunk; a multiple of the scan kernel's block step
constexpr int RM_FULL = RM_CHUNK / 32 / 64;           // 32-bit words of hit bits per lane and chunk (pieces of chunks: fewer)
constexpr int RM_PER = 4;                             // records a lane gathers together
constexpr int RM_LIST = 512;                          // positions a wavefront expands per round
constexpr int RM_QPB = 1;                             // queries per block (two: 1.39 against 1.25 ms at N = 1e8, 128 queries)
constexpr int RM_SEED_EVERY = 65;                     // odd: the first launch's chunks are spread over all XCDs
constexpr uint32_t RM_SEED_PARTS = 4;                 // of whole chunks the first launch may take quarters
static_assert(RM_LIST % (64 * RM_PER) == 0, "a round of the list is whole steps of gathers");
static_assert(RM_CHUNK <= 65536, "the position lists hold 16-bit offsets into the chunk");

// QPB queries per block: their tables sit in LDS side by side and every chunk is worked through for one
// query after the other, so the later ones find the chunk's records in the cache for certain.
// EXACT: the hit bits mark a superset of the survivors (the 16-bit pre-filter of stage 1); an item is a
// survivor when the first Kf terms of its sum -- the crude distance of Eq. 2, the same fp32 additions
// stage 1 makes item by item -- are below thr[q].  Only survivors are counted and get keys.
// The filtered launch is held to the registers of five wavefronts per SIMD (the exact comparison's few
// more would cost the fifth: 1.17 -> 1.29 ms for the stage at N = 1e8).
template <int WORDS, bool FILTER, int QPB, bool EXACT, int RM_WORDS>
__global__ __launch_bounds__(RM_THREADS, FILTER ? 5 : 1) void refine_mask_kernel(
    const uint8_t *__restrict__ items, int K, const float *__restrict__ lut, const uint32_t *__restrict__ masks,
    size_t mask_words, const uint32_t *__restrict__ perm, uint32_t nsel, uint32_t seed_every, uint32_t seed_parts, int window, int xs_shift, int Q,
    const float *__restrict__ kth_dist, int topk, u64 *__restrict__ keys, uint32_t *__restrict__ key_count,
    int64_t cap, uint32_t *__restrict__ cand_count, const float *__restrict__ thr, int Kf) {
    __shared__ __attribute__((aligned(16))) float T_all[QPB][4 * WORDS * ICQ_LUT_W];
    __shared__ uint16_t cand_all[RM_WAVES][RM_LIST];  // positions inside the chunk (RM_CHUNK <= 65536)
    __shared__ uint32_t sum_all[QPB], done_all[QPB];  // survivors of the block, wavefronts that have added theirs
    constexpr int RW = WORDS;
    constexpr uint32_t PIECE = RM_WORDS * 2048;       // positions
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint16_t *cand = cand_all[wave];
    // block -> (window, query group, XCD): chunks i = (win * window + j) * 8 + xcd, j = 0 .. window - 1, of this
    // launch's; wavefront w takes j = w, w + 4, ..  (An index of few chunks is cut 2^xs_shift < 8 ways instead, so
    // that a block still has a window's worth of chunks for the tables it loads.)
    const uint32_t ngroups = ((uint32_t)Q + QPB - 1) / QPB;
    const uint32_t xcd = blockIdx.x & ((1u << xs_shift) - 1u), rest = blockIdx.x >> xs_shift;
    const uint32_t q0 = (rest % ngroups) * QPB, win = rest / ngroups;
    const uint32_t nq = (uint32_t)Q - q0 < (uint32_t)QPB ? (uint32_t)Q - q0 : (uint32_t)QPB;
    auto chunk_of = [&](uint32_t j) -> uint32_t {
        const uint32_t i = ((win * (uint32_t)window + j) << xs_shift) + xcd;
        if (j >= (uint32_t)window || i >= nsel) return 0xFFFFFFFFu;
        if (!FILTER) return i * seed_every;
        return seed_parts == 1u ? i + i / (RM_SEED_EVERY - 1u) + 1u : i;   // all but every 65th : all
    };
    if (chunk_of(0) == 0xFFFFFFFFu) return;           // block-uniform: nothing for this block
    // Word r of this lane covers the 32 positions from c * PIECE + (r * 64 + lane) * 32: neighbouring
    // words sit in neighbouring lanes, so a dense stretch of hits is shared out among many lanes.
    // The wavefront's work is the sequence (chunk j, query qq), qq fastest; the next one's hit bits travel
    // while the current one is worked on.
    const uint32_t *mq = masks + (size_t)q0 * mask_words + lane;
    uint32_t j = (uint32_t)wave, qq = 0;
    uint32_t c = chunk_of(j);
    uint32_t nxt[RM_WORDS];
    {
        const uint32_t c0 = c != 0xFFFFFFFFu ? c : 0u;
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) nxt[r] = __builtin_nontemporal_load(mq + (size_t)c0 * (PIECE / 32) + r * 64);
    }
    // the queries' tables -> LDS, one table per record byte, zero beyond K
#pragma unroll
    for (int g = 0; g < QPB; ++g) {
        const uint32_t qg = q0 + ((uint32_t)g < nq ? (uint32_t)g : 0u);
        const float4 *src = reinterpret_cast<const float4 *>(lut + (int64_t)qg * K * ICQ_LUT_W);
        float4 *dst = reinterpret_cast<float4 *>(T_all[g]);
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
    uint32_t bound_all[QPB];
#pragma unroll
    for (int g = 0; g < QPB; ++g) {
        bound_all[g] = 0xFFFFFFFFu;
        if (FILTER) {
            const uint32_t qg = q0 + ((uint32_t)g < nq ? (uint32_t)g : 0u);
            const uint32_t ob = icq_order_bits(kth_dist[(int64_t)qg * topk + topk - 1]);
            if (ob < 0xFF800000u) bound_all[g] = ob;  // a finite topk-th distance; else the list is still open
        }
    }
    if (tid < QPB) sum_all[tid] = done_all[tid] = 0;
    __syncthreads();                                  // the only barrier: from here on every wavefront is on its own
    uint32_t survivors[QPB];                          // of this wavefront's chunks (wavefront-uniform)
    uint32_t lane_survivors[QPB];                     // EXACT: counted per lane, summed at the end
#pragma unroll
    for (int g = 0; g < QPB; ++g) survivors[g] = lane_survivors[g] = 0;
    while (c != 0xFFFFFFFFu) {
        uint32_t w[RM_WORDS];
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) w[r] = nxt[r];
        if (FILTER && RM_WORDS == RM_FULL && seed_parts > 1u) {       // the quarter that the first launch has done is out
            const uint32_t at = c * RM_SEED_PARTS % RM_SEED_EVERY, done = at == 0u ? 0u : RM_SEED_EVERY - at;
            if (done < RM_SEED_PARTS) {               // wavefront-uniform
#pragma unroll
                for (int r = 0; r < RM_WORDS; ++r) w[r] = (uint32_t)r / (RM_FULL / RM_SEED_PARTS) == done ? 0u : w[r];
            }
        }
        // next piece of work: the next query of this chunk, else the wavefront's next chunk
        uint32_t qn = qq + 1, jn = j, cn = c;
        if (qn >= nq) {
            qn = 0;
            jn = j + RM_WAVES;
            cn = chunk_of(jn);
        }
        if (cn != 0xFFFFFFFFu) {
            const uint32_t *mn = mq + (size_t)qn * mask_words + (size_t)cn * (PIECE / 32);
#pragma unroll
            for (int r = 0; r < RM_WORDS; ++r) nxt[r] = __builtin_nontemporal_load(mn + r * 64);
        }
        const uint32_t q = q0 + qq;
        const float tq = EXACT ? thr[q] : 0.0f;
        const float *T = T_all[QPB == 1 ? 0 : qq];
        uint32_t bound = bound_all[0];
#pragma unroll
        for (int g = 1; g < QPB; ++g) bound = qq == (uint32_t)g ? bound_all[g] : bound;
        u64 *kout = keys + (int64_t)q * cap;
        uint32_t mine = 0;
#pragma unroll
        for (int r = 0; r < RM_WORDS; ++r) mine += (uint32_t)__builtin_popcount(w[r]);
        const uint32_t incl = wave_scan_add(mine);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        const uint32_t off = incl - mine;
        if (!EXACT) {
#pragma unroll
            for (int g = 0; g < QPB; ++g) survivors[g] += qq == (uint32_t)g ? total : 0u;
        }
        // unfiltered: every survivor of the chunk gets a key, so their slots are reserved at once (the atomic's
        // answer travels while the positions are expanded)
        uint32_t chunk_slot = 0;
        if (!FILTER && !EXACT && total != 0) {
            if (lane == 0) chunk_slot = atomicAdd(&key_count[q], total);
        }
        const uint32_t cbase = c * PIECE, p0 = lane * 32u;
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
                        if (EXACT && i < 4) crude = i < Kf ? d : crude;
                    }
                    const uint32_t ob = icq_order_bits(d);
                    bool keep = base + (uint32_t)u * 64u + lane < n;
                    if (EXACT) {
                        keep = keep && crude < tq;
#pragma unroll
                        for (int g = 0; g < QPB; ++g) lane_survivors[g] += (qq == (uint32_t)g && keep) ? 1u : 0u;
                    }
                    keep = keep && ob <= bound;
                    mk[u] = __builtin_amdgcn_ballot_w64(keep);
                    mycnt += (uint32_t)__builtin_popcountll(mk[u]);
                    key[u] = (u64)ob << 32;
                }
                if (mycnt == 0) continue;             // wavefront-uniform
                uint32_t slot0 = 0;
                if (FILTER || EXACT) {
                    if (lane == 0) slot0 = atomicAdd(&key_count[q], mycnt);
                    slot0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot0);
                } else {
                    slot0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)chunk_slot) + lo + base;
                }
#pragma unroll
                for (int u = 0; u < RM_PER; ++u) {
                    if ((mk[u] >> lane) & 1ull) {
                        const uint64_t slot = (uint64_t)__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(mk[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk[u], slot0));
                        if (slot < (uint64_t)cap) kout[slot] = key[u] | (perm ? perm[id[u]] : id[u]);
                    }
                    slot0 += (uint32_t)__builtin_popcountll(mk[u]);
                }
            }
        }
        qq = qn;
        j = jn;
        c = cn;
    }
    if (EXACT) {
#pragma unroll
        for (int g = 0; g < QPB; ++g)
            survivors[g] = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(lane_survivors[g]), 63);
    }
    // one addition per block: thousands of wavefronts of one query at one counter would take 11 ns each.  The last of the four
    // to come here makes it.
#pragma unroll
    for (int g = 0; g < QPB; ++g) {
        if (lane != 0) continue;
        atomicAdd(&sum_all[g], survivors[g]);
        __threadfence_block();
        if (atomicAdd(&done_all[g], 1u) != RM_WAVES - 1) continue;
        const uint32_t sum = atomicAdd(&sum_all[g], 0u);
        if ((uint32_t)g < nq && sum != 0) atomicAdd(&cand_count[q0 + g], sum);
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
        return icq_launch_select(keys, const_cast<uint32_t *>(cand_count), cap, Q, topk, splits, false, ticket, out_ids,
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
        return icq_launch_select(keys, nullptr, (int64_t)splits * topk, Q, topk, 1, false, nullptr, out_ids, out_dist, s);
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

// From about four million items on: below that the item records stay in the caches whatever the
// order of the gathers, and candidate lists with the flat distance kernel are quicker (N = 1e6,
// K = 16, 1000 queries: 0.15 against 0.24 ms for stage 2).
bool icq_masks_usable(const icq_index *ix, int Q, int topk) {
    // from 2^22 items on; with the 16-bit pre-filter (eight queries per pass of stage 1) and enough queries to
    // fill the chunk walk already from 2^19 (1000 queries, K = 16: lists are ahead up to 3e5 items, hit bits from 6e5)
    const bool large = ix->N >= (1ll << 22) || (ix->N >= (1ll << 19) && Q >= 32 && icq_scan_q16_usable(ix, Q));
    return ix->Kf <= 4 && !icq_group_usable(ix, Q) && icq_selects(ix, topk) && large &&
           ix->N + 16ll * 65536 < (1ll << 31);
}

int64_t icq_mask_scan_end(const icq_index *ix) {
    const int64_t npos = icq_g2_usable(ix) ? ix->g2_npos : ix->N;
    return (npos + RM_CHUNK - 1) / RM_CHUNK * RM_CHUNK;
}

int icq_launch_refine_masks(const icq_index *ix, const float *lut, int Q, const uint16_t *masks, size_t mask_stride,
                            int64_t scan_end, int64_t cap, int topk, int splits, u64 *keys, uint32_t *key_count,
                            uint32_t *ticket, uint32_t *cand_count, const float *thr, uint32_t *out_ids, float *out_dist,
                            hipStream_t s) {
    if (Q == 0) return ICQ_OK;
    const bool g2 = icq_g2_usable(ix);
    const uint8_t *items = g2 ? ix->items_grouped : ix->items;
    const uint32_t *perm = g2 ? ix->perm : nullptr;
    // few chunks: one unfiltered launch over all of them (a bound would save less than its second launch costs)
    const uint32_t seed_every = scan_end / RM_CHUNK < 2 * RM_SEED_EVERY ? 1u : (uint32_t)RM_SEED_EVERY;
    // A wavefront takes a chunk at a time, or half or a quarter of one.  What a call spends its time on depends on what survives:
    // with little, on each piece's chain of steps and each block's tables, so that smaller pieces cost; with much, on the first
    // launch, whose few wavefronts then hold long lists, and on records that leave the caches before the other queries'
    // blocks come to them, so that smaller pieces and windows gain.  Whole chunks with a first launch of quarters and windows of
    // four chunks lose to larger pieces at no share; smaller pieces stand where they do not lose at a low share either.  Whole
    // calls, us, at 0.05 / 1 / 5 / 30 % (K = 16, Kf = 4; whole chunks in both launches, windows of 16, 12 from eight queries on | halves
    // in both, windows of 8 | quarters, windows of 8 | this):
    //   4.3e6 items, 1 query     44/102/317/2300 |  34/46/82/335   |  33/44/58/146     quarters
    //   4.3e6, 3 queries        48/109/353/2339  |  45/56/107/330  |  46/62/88/183     halves
    //   4.3e6, 8                57/106/302/1709  |  64/85/165/514  |  70/98/148/289    whole  53/74/156/509
    //   9e6, 16                 100/162/375/1575 | 114/172/335/708 | 129/221/335/570   whole  97/152/342/734
    //   2e7, 5                  80/158/395       |  84/127/207     |  85/123/167       halves
    //   2e7, 64                 228/409/742/3756 | 254/413/645/2258| 266/439/607/1751  whole  222/399/665/3399
    //   6e7, 8                  152/322/617/2274 | 133/248/373/1244| 152/243/356/859   halves
    //   1e8, 1                  90/205/540/3472  |  90/166/260/753 |  87/184/252/473   halves
    //   1e8, 64                 669/1220/2318    | 649/1088/1985   | 714/1178/2068     halves
    // Codes not ordered by their first two (K = 8, Kf = 2): 9e6, 1 query 45/67/209/2055 | 37/41/67/248 | 42/45/63/142; 1.3e7, 4
    // queries 63/91/233/1933 | 75/81/174/428 | 108/114/173 | whole 58/80/167/380.
    const uint64_t whole = (uint64_t)(scan_end / RM_CHUNK), pairs = whole * (uint64_t)Q;
    int words = RM_FULL;
    if (seed_every != 1u) {
        if (pairs <= 320) words = RM_FULL / 4;
        else if (pairs <= 700 || (g2 && Q < 8 && whole >= 600) || (g2 && whole >= 1700 && pairs <= 200000)) words = RM_FULL / 2;
    }
    // (the largest calls have wavefronts enough for whole ones: 1e8 items, 128 queries 1802 us, with quarters 1823)
    const uint32_t seed_parts = seed_every != 1u && words == RM_FULL && pairs <= 200000 ? RM_SEED_PARTS : 1u;
    const int seed_words = words / (int)seed_parts;
    const uint32_t chunks = (uint32_t)(scan_end / (2048 * words)), seed_chunks = (uint32_t)(scan_end / (2048 * seed_words));
    const uint32_t nseed = (seed_chunks + seed_every - 1) / seed_every;
    const uint32_t nmain = seed_every == 1u ? 0u : seed_parts == 1u ? chunks - nseed : chunks;
    auto select = [&](bool more) -> int {
        return icq_launch_select(keys, key_count, cap, Q, topk, splits, more, ticket, out_ids, out_dist, s);
    };
    // Pieces per block: few, so that the blocks in flight (two windows' worth when the queries fill the
    // chip) keep to a few chunks per XCD.  With few queries one per wavefront.
    // An unfiltered launch with little work for the chip (the first part of a large index: one chunk per
    // wavefront is all the parallelism there is) is spread over as many blocks as possible; one that is the
    // whole stage (a small index, many queries) takes full windows, and the chunks are cut fewer than 8
    // ways when 8 windows' worth do not exist: 16 MB of records stay in the caches wherever the blocks run.
    auto plan_for = [&](uint32_t nsel, bool filtered, int *xs_shift) -> int {
        // whole chunks: 4, with more blocks than the chip holds for long 12 or 8 (at N = 1e8, 128 queries, pair ordering:
        // 16 / 12 / 8 / 6 / 4: 1.105 / 1.090 / 1.109 / 1.18 / 1.31 ms; whole calls at 1 %, windows of 4 / 12: 2e7 items, 128 queries
        // 512 / 529 us, 3e7, 200 queries (K = 8) 804 / 769)
        int w = words != RM_FULL ? 8 : pairs <= 131072u ? 4 : g2 ? 12 : 8;
        if ((uint64_t)nsel * (uint64_t)Q <= 16384u && (!filtered || Q < 8)) w = 4;
        else if (!filtered) w = 16 * RM_FULL / seed_words;
        // (with thousands of queries a window's blocks no longer run at the same time, and the 8-way cut that
        // keeps a chunk's records in ONE L2 is worth more than the longer windows: 1e4 queries, 1e6 items,
        // 8-byte records: 0.80 ms with it, 0.83 without)
        int shift = 3;
        while (Q <= 2048 && shift > 0 && ((uint32_t)w << shift) > nsel) --shift;
        *xs_shift = shift;
        const int most = (int)((nsel + (1u << shift) - 1) >> shift);
        return w < most ? w : (most > 0 ? most : 1);
    };
    const size_t mask_words = mask_stride / 2;
    const uint32_t *m32 = reinterpret_cast<const uint32_t *>(masks);
#define ICQ_RM_LAUNCH(W, FILTER, NSEL)                                                                       \
    do {                                                                                                     \
        int xs_shift = 3;                                                                                    \
        const int window = plan_for(NSEL, FILTER, &xs_shift);                                                \
        const unsigned per_win = (unsigned)window << xs_shift;                                               \
        const unsigned nwin = ((NSEL) + per_win - 1) / per_win;                                              \
        const unsigned ngroups = ((unsigned)Q + RM_QPB - 1) / RM_QPB;                                        \
        auto go = [&](auto kernel) {                                                                         \
            kernel<<<(nwin * ngroups) << xs_shift, RM_THREADS, 0, s>>>(                                      \
                items, ix->K, lut, m32, mask_words, perm, (NSEL), seed_every, seed_parts, window, xs_shift, Q, out_dist, topk,     \
                keys, key_count, cap, cand_count, thr, ix->Kf);                                              \
        };                                                                                                   \
        const int piece = FILTER ? words : seed_words;                                                       \
        if (piece == RM_FULL / 4) { if (thr) go(refine_mask_kernel<W, FILTER, RM_QPB, true, RM_FULL / 4>); else go(refine_mask_kernel<W, FILTER, RM_QPB, false, RM_FULL / 4>); } \
        else if (piece == RM_FULL / 2) { if (thr) go(refine_mask_kernel<W, FILTER, RM_QPB, true, RM_FULL / 2>); else go(refine_mask_kernel<W, FILTER, RM_QPB, false, RM_FULL / 2>); } \
        else { if (thr) go(refine_mask_kernel<W, FILTER, RM_QPB, true, RM_FULL>); else go(refine_mask_kernel<W, FILTER, RM_QPB, false, RM_FULL>); }         \
    } while (0)
    switch (ix->item_stride) {
        case 4: ICQ_RM_LAUNCH(1, false, nseed); break;
        case 8: ICQ_RM_LAUNCH(2, false, nseed); break;
        default: ICQ_RM_LAUNCH(4, false, nseed); break;
    }
    if (icq_check_launch() != ICQ_OK) return ICQ_ERR_HIP;
    if (nmain == 0) return select(false);
    int rc = select(true);
    if (rc != ICQ_OK) return rc;
    switch (ix->item_stride) {
        case 4: ICQ_RM_LAUNCH(1, true, nmain); break;
        case 8: ICQ_RM_LAUNCH(2, true, nmain); break;
        default: ICQ_RM_LAUNCH(4, true, nmain); break;
    }
#undef ICQ_RM_LAUNCH
    if (icq_check_launch() != ICQ_OK) return ICQ_ERR_HIP;
    return select(false);
}
