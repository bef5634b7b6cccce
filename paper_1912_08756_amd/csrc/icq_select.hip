// The nearest-neighbour list of arxiv 1912.08756, Sec. 3.4, out of keys: the topk smallest of a
// query's 64-bit keys (order-preserving bits of D, item id), ascending.  The keys are either the
// survivors' (count[q] of them) or the ascending lists that several blocks left for one query.
//
// One block per query.  Every thread takes the smallest key of its share (or of two shares); the
// topk-th smallest of those minima (one histogram pass) bounds the topk-th smallest key from above,
// because at least topk keys are at or below it -- and hardly more are: with 10^4 keys, 1024 threads
// and topk = 100 some 110.  Those are collected into LDS and ranked by counting.  The keys stay in
// registers between the two looks while there are at most PER per thread (8192 with 1024 threads),
// else they are read again from the caches.  Where equal distances let hundreds through, the ids decide as well.
//
// What bounds it is latency: three dependent trips to memory (count, keys, results) and a dozen
// barriers; 128 queries of 15000 keys also take the time their keys need to come from another
// chiplet's cache.  One query of 10^4 keys: 11 us, where a wavefront per slice (17 us) and a kernel
// that joined 25 sorted slices (103 us) did the same before; 40 slices joined by binary searches took
// 20 + 198 us, now 16.
//
// A query with very many keys is cut into up to `splits` parts, as many as its count asks for; each
// part leaves its ascending list in place of its keys and the last block to finish selects again from those.
#include "icq_internal.h"
#include "icq_sort.h"

#include <math.h>

namespace {

constexpr int SEL_LIST = 1024;     // keys the LDS list holds; topk <= 512
constexpr int SEL_PART = 16384;    // keys of a part, once a query's keys are cut into parts (SEL_ALONE)
constexpr int SEL_RANK = 256;      // up to so many keys are ranked by counting, more are sorted

template <int T>
struct SelShared {
    IcqKthSharedT<T> kth;
    uint32_t cnt, minima, below, last;
    uint32_t rank[SEL_RANK];
};

// The topk smallest keys of in[0..n) (KEY_PAD entries are skipped) -> list[0..kept) ascending;
// returns kept = min(topk, number of keys).  PER: keys per thread held in registers; MIN: shares of a thread, a minimum each.  LISTS: n is a multiple of topk, and
// each run of topk keys starts `stride` after the one before.  Every thread of the block calls.
template <int T, int PER, int MIN, bool LISTS>
__device__ int block_select(SelShared<T> &sh, u64 *list, const u64 *in, u64 n, u64 stride, int topk) {
    auto key = [&](u64 i) { return LISTS ? in[(uint32_t)i / (uint32_t)topk * stride + (uint32_t)i % (uint32_t)topk] : in[i]; };
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u;
    const int wave = tid >> 6;
    if (n == 0) return 0;
    u64 r[PER];
    auto load = [&](u64 base) {        // unconditional, clamped: all of a thread's loads are in flight together
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const u64 i = base + (u64)j * T + tid;
            r[j] = key(i < n ? i : n - 1);
        }
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (base + (u64)j * T + tid >= n) r[j] = KEY_PAD;
    };
    const bool once = n <= (u64)PER * T;
    u64 least[MIN];                    // the smallest keys of this thread's shares
#pragma unroll
    for (int u = 0; u < MIN; ++u) least[u] = KEY_PAD;
    for (u64 base = 0; base < n; base += (u64)PER * T) {
        load(base);
#pragma unroll
        for (int j = 0; j < PER; ++j) least[j % MIN] = r[j] < least[j % MIN] ? r[j] : least[j % MIN];
    }
    uint32_t high[MIN], low[MIN], any = 0;
#pragma unroll
    for (int u = 0; u < MIN; ++u) {
        high[u] = (uint32_t)(least[u] >> 32);
        low[u] = (uint32_t)least[u];
        if (least[u] != KEY_PAD) any |= 1u << u;
    }
    if (tid == 0) sh.cnt = sh.minima = sh.below = 0;
    __syncthreads();
    // the lanes' flagged minima, as one count per wavefront
    auto count = [&](uint32_t flags, uint32_t *to) {
        uint32_t n = 0;
#pragma unroll
        for (int u = 0; u < MIN; ++u) n += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((flags >> u) & 1u));
        if (lane == 0) atomicAdd(to, n);
    };
    count(any, &sh.minima);
    __syncthreads();
    const bool bounded = n > (u64)topk && sh.minima >= (uint32_t)topk;
    u64 limit = KEY_PAD - 1;           // the largest key that is collected
    if (bounded) {
        const u64 top = ((u64)block_kth<MIN>(sh.kth, high, any, (uint32_t)topk, false, tid, lane, wave) << 32) | 0xFFFFFFFFu;
        limit = top < limit ? top : limit;
    }
    auto collect = [&]() {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const bool keep = r[j] <= limit;
            const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
            if (mask == 0) continue;                       // wavefront-uniform
            uint32_t slot = 0;
            if (lane == 0) slot = atomicAdd(&sh.cnt, (uint32_t)__builtin_popcountll(mask));
            slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
            slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, slot));
            if (keep && slot < (uint32_t)SEL_LIST) list[slot] = r[j];
        }
    };
    uint32_t cnt;
    for (bool exact = false;; exact = true) {
        if (once) {
            collect();
        } else {
            for (u64 base = 0; base < n; base += (u64)PER * T) {
                load(base);
                collect();
            }
        }
        __syncthreads();
        cnt = sh.cnt;
        if (cnt <= (uint32_t)SEL_LIST || exact || !bounded) break;     // block-uniform
        // Masses of equal distances, or a histogram bin wide enough to hold hundreds of keys: the topk-th smallest of the
        // minima as whole keys, the id deciding among equal distances, bounds as well and lets through about as few as
        // distinct distances would.  icq_refine of one query, 16 different distances among 20000 / 120000 candidates,
        // topk = 100: 30 / 71 us (in parts 31), where the digit passes below, taken at once, made it 70 / 316.
        const uint32_t kth = block_kth<MIN>(sh.kth, high, any, (uint32_t)topk, true, tid, lane, wave);
        uint32_t under = 0, at = 0;
#pragma unroll
        for (int u = 0; u < MIN; ++u) {
            if (((any >> u) & 1u) && high[u] < kth) under |= 1u << u;
            if (((any >> u) & 1u) && high[u] == kth) at |= 1u << u;
        }
        count(under, &sh.below);
        if (tid == 0) sh.cnt = 0;
        __syncthreads();
        limit = ((u64)kth << 32) | block_kth<MIN>(sh.kth, low, at, (uint32_t)topk - sh.below, true, tid, lane, wave);
    }
    if (cnt > (uint32_t)SEL_RANK && cnt <= (uint32_t)SEL_LIST && cnt > (uint32_t)topk) {
        // a fat histogram bin, or ties: cut the list exactly at the topk-th smallest distance and, where too many keys have
        // that one for the ranks, at the topk-th smallest key
        constexpr int LPT = SEL_LIST / T;
        u64 e[LPT];
        uint32_t v[LPT], id[LPT], ok = 0;
#pragma unroll
        for (int u = 0; u < LPT; ++u) {
            const uint32_t i = (uint32_t)u * T + tid;
            e[u] = list[i];
            v[u] = (uint32_t)(e[u] >> 32);
            id[u] = (uint32_t)e[u];
            if (i < cnt) ok |= 1u << u;
        }
        const uint32_t cut = block_kth<LPT>(sh.kth, v, ok, (uint32_t)topk, true, tid, lane, wave);
        if (tid == 0) sh.cnt = sh.below = 0;
        __syncthreads();                                   // the list has been read, the counters are zero
        uint32_t tie = 0, below = 0, upto = 0;
#pragma unroll
        for (int u = 0; u < LPT; ++u) {
            const bool in = (ok >> u) & 1u;
            if (in && v[u] == cut) tie |= 1u << u;
            below += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(in && v[u] < cut));
            upto += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(in && v[u] <= cut));
        }
        if (lane == 0) {
            atomicAdd(&sh.below, below);
            atomicAdd(&sh.cnt, upto);
        }
        __syncthreads();
        uint32_t last_id = 0xFFFFFFFFu;
        if (sh.cnt > (uint32_t)SEL_RANK && topk <= SEL_RANK)       // block-uniform
            last_id = block_kth<LPT>(sh.kth, id, tie, (uint32_t)topk - sh.below, true, tid, lane, wave);
        __syncthreads();
        if (tid == 0) sh.cnt = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < LPT; ++u)
            if (((ok >> u) & 1u) && (v[u] < cut || (v[u] == cut && id[u] <= last_id))) list[atomicAdd(&sh.cnt, 1u)] = e[u];
        __syncthreads();
        cnt = sh.cnt;
    }
    if (cnt > (uint32_t)SEL_LIST) {
        // Few threads hold most of the smallest keys (or any at all), or a key is there many times: exact radix select
        // over whole keys, 8 bits at a time, re-reading the keys for every digit.  More than topk keys are there.
        u64 prefix = 0;
        uint32_t kr = (uint32_t)topk;
        for (int shift = 56; shift >= 0; shift -= 8) {
            __syncthreads();
            if (tid < 256) sh.kth.hist[tid] = 0;
            __syncthreads();
            for (u64 i = tid; i < n; i += T) {
                const u64 k = key(i);
                if (k != KEY_PAD && (shift == 56 || (k >> (shift + 8)) == prefix))
                    atomicAdd(&sh.kth.hist[(uint32_t)(k >> shift) & 255u], 1u);
            }
            __syncthreads();
            // every wavefront locates the bin by itself (4 bins per lane)
            uint32_t h[4], mine = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                h[b] = sh.kth.hist[lane * 4 + b];
                mine += h[b];
            }
            const uint32_t incl = wave_scan_add(mine);
            const int L = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl >= kr));
            uint32_t run = incl - mine, my_bin = 0, my_below = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (run < kr && run + h[b] >= kr) {
                    my_bin = lane * 4 + b;
                    my_below = run;
                }
                run += h[b];
            }
            prefix = (prefix << 8) | (uint32_t)__builtin_amdgcn_readlane((int)my_bin, L);
            kr -= (uint32_t)__builtin_amdgcn_readlane((int)my_below, L);
        }
        // the keys below the cut, then copies of it (a caller's list may name an item twice) up to topk
        __syncthreads();
        if (tid == 0) sh.cnt = 0;
        __syncthreads();
        for (u64 i = tid; i < n; i += T) {
            const u64 k = key(i);
            if (k < prefix) list[atomicAdd(&sh.cnt, 1u)] = k;
        }
        __syncthreads();
        for (uint32_t i = sh.cnt + (uint32_t)tid; i < (uint32_t)topk; i += T) list[i] = prefix;
        __syncthreads();
        cnt = (uint32_t)topk;
    }
    const int kept = (int)cnt < topk ? (int)cnt : topk;
    if (cnt <= (uint32_t)SEL_RANK) {
        // rank = number of keys before one's own (equal keys: by place); W threads side by side, T / W
        // groups of them share the counting
        const uint32_t W = cnt <= 64 ? 64u : cnt <= 128 ? 128u : 256u;
        const uint32_t i = (uint32_t)tid & (W - 1u), part = (uint32_t)tid / W, parts = (uint32_t)T / W;
        const uint32_t per = (cnt + parts - 1) / parts, j0 = part * per, j1 = j0 + per < cnt ? j0 + per : cnt;
        const u64 mine = i < cnt ? list[i] : KEY_PAD;
        if (tid < SEL_RANK) sh.rank[tid] = 0;
        __syncthreads();
        uint32_t rank = 0;
        for (uint32_t j = j0; j < j1; ++j) {
            const u64 k = list[j];                         // one address for all lanes
            rank += (k < mine || (k == mine && j < i)) ? 1u : 0u;
        }
        if (i < cnt && rank != 0) atomicAdd(&sh.rank[i], rank);
        __syncthreads();                                   // the list has been read
        if (tid < (int)cnt) list[sh.rank[tid]] = mine;     // tid < cnt <= W: i == tid
    } else {
        // bitonic sort of up to SEL_LIST keys in LDS by the whole block
        int len = 512;
        while (len < (int)cnt) len <<= 1;
        for (int i = (int)cnt + tid; i < len; i += T) list[i] = KEY_PAD;
        for (int k = 2; k <= len; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                __syncthreads();
                for (int i = tid; i < len / 2; i += T) {
                    const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1)), hi = lo | j;
                    const u64 x = list[lo], y = list[hi];
                    if ((x > y) == ((lo & k) == 0)) {
                        list[lo] = y;
                        list[hi] = x;
                    }
                }
            }
        }
    }
    __syncthreads();
    return kept;
}

// Grid: Q * splits blocks.  count != nullptr: count[q] keys (at most cap) at keys_in + q * cap, worked off
// by one of the query's blocks, or if they are more than `alone` by one per SEL_PART keys; count == nullptr: cap keys,
// splits == 1.
template <int T, int PER, int MIN>
__global__ __launch_bounds__(T) void select_kernel(u64 *keys_in, const uint32_t *count, int64_t cap, int topk, int splits,
                                                   uint32_t alone, uint32_t *ticket,
                                                   uint32_t *__restrict__ out_ids, float *__restrict__ out_dist) {
    __shared__ SelShared<T> sh;
    __shared__ __attribute__((aligned(16))) u64 list[SEL_LIST];
    const int q = blockIdx.x / splits, sp = blockIdx.x % splits;
    const int tid = threadIdx.x;
    u64 n = (u64)cap;
    int used = 1;
    if (count) {
        n = count[q];
        if (n > (u64)cap) n = (u64)cap;
        const u64 want = (n + (u64)SEL_PART - 1) / (u64)SEL_PART;
        used = n <= (u64)alone ? 1 : want > (u64)splits ? splits : (int)want;
    }
    if (sp >= used) return;                                // block-uniform
    u64 *mine = keys_in + (int64_t)q * cap;
    const u64 per = used == 1 ? n : (n + (u64)used - 1) / (u64)used, lo = (u64)sp * per;
    int kept = block_select<T, PER, MIN, false>(sh, list, mine + lo, n - lo < per ? n - lo : per, 0, topk);
    if (used > 1) {
        for (int i = tid; i < topk; i += T) mine[lo + i] = i < kept ? list[i] : KEY_PAD;     // parts are longer than topk
        // One thread makes the block's list visible to the device and the other blocks' visible to the block: a fence
        // writes back and invalidates the chiplet's L2, and one per wavefront was sixteen of each.  Every wavefront
        // waits for its own stores first: the barrier alone need not order them before another wavefront's fence.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            __threadfence();
            sh.last = atomicAdd(&ticket[q], 1u) == (uint32_t)(used - 1) ? 1u : 0u;
            __threadfence();
        }
        __syncthreads();
        if (sh.last == 0) return;                          // block-uniform
        kept = block_select<T, PER, MIN, true>(sh, list, mine, (u64)used * topk, per, topk);
    }
    for (int i = tid; i < topk; i += T) {
        const bool have = i < kept;
        const u64 k = list[have ? i : 0];
        out_ids[(int64_t)q * topk + i] = have ? (uint32_t)k : ICQ_PAD_ID;
        out_dist[(int64_t)q * topk + i] = have ? icq_unorder_bits((uint32_t)(k >> 32)) : INFINITY;
    }
}

// One block per query: `parts` ascending lists of topk keys, KEY_PAD behind the last, no key twice, SEL_LIST keys at most.
// A key's row is the number of keys below it: a binary search in each other list.
constexpr int JOIN_THREADS = 256;
__global__ __launch_bounds__(JOIN_THREADS) void join_kernel(const u64 *__restrict__ lists, int parts, int topk,
                                                            uint32_t *__restrict__ out_ids, float *__restrict__ out_dist) {
    __shared__ u64 keys[SEL_LIST];
    __shared__ int s_real;
    const int q = blockIdx.x, tid = threadIdx.x, n = parts * topk;
    if (tid == 0) s_real = 0;
    for (int i = tid; i < n; i += JOIN_THREADS) keys[i] = lists[(int64_t)q * n + i];
    __syncthreads();
    int real = 0;
    for (int i = tid; i < n; i += JOIN_THREADS) {
        const u64 k = keys[i];
        if (k == KEY_PAD) continue;
        ++real;
        const int own = i / topk;
        int row = i - own * topk;
        for (int p = 0; p < parts; ++p) {
            if (p == own) continue;
            const u64 *list = keys + p * topk;
            int lo = 0, hi = topk;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (list[mid] < k) lo = mid + 1;
                else hi = mid;
            }
            row += lo;
        }
        if (row < topk) {
            out_ids[(int64_t)q * topk + row] = (uint32_t)k;
            out_dist[(int64_t)q * topk + row] = icq_unorder_bits((uint32_t)(k >> 32));
        }
    }
    real = (int)wave_scan_add((uint32_t)real);
    if ((tid & 63) == 63 && real != 0) atomicAdd(&s_real, real);
    __syncthreads();
    for (int i = s_real + tid; i < topk; i += JOIN_THREADS) {
        out_ids[(int64_t)q * topk + i] = ICQ_PAD_ID;
        out_dist[(int64_t)q * topk + i] = INFINITY;
    }
}

template <int T, int PER, int MIN>
int launch_select(u64 *keys, const uint32_t *count, int64_t cap, int Q, int topk, int splits, uint32_t alone, uint32_t *ticket,
                  uint32_t *out_ids, float *out_dist, hipStream_t s) {
    select_kernel<T, PER, MIN><<<(unsigned)Q * (unsigned)splits, T, 0, s>>>(keys, count, cap, topk, splits, alone, ticket, out_ids,
                                                                       out_dist);
    return icq_check_launch();
}

}  // namespace

// Keys a block takes alone.  Joining parts takes 10 us (25 where lists of more than 256 keys are sorted), a block a
// microsecond per 4000 keys: icq_refine of one query, topk = 100, 40000 / 120000 candidates in one part 22 / 43 us, in
// parts of SEL_PART 22 / 23 us; topk = 512, 120000 candidates: 58 / 64 us.  (128 queries of 20000 / 80000, one part
// 46 / 147, several 58 / 158 us: they fill the chip as they are.)  The line by queries lies where the ticket each of them
// needs no longer fits the 256 bytes that the counters take anyway.
static uint32_t select_alone(int Q, int topk) {
    return topk <= 256 && 3 * sizeof(uint32_t) * (size_t)Q <= ICQ_ALIGN ? 40960 : 131072;
}

// Parts a query's keys may be cut into: more than one only where the queries leave the chip mostly idle.
int icq_select_splits(const icq_index *ix, int Q, int64_t cap, int topk) {
    if (Q <= 0 || cap <= (int64_t)select_alone(Q, topk)) return 1;
    int64_t s = ix->num_cu / Q;
    const int64_t by_len = cap / SEL_PART + 1;
    const int64_t by_merge = 4096 / topk;       // the parts' lists fit one block's registers again
    if (s > by_len) s = by_len;
    if (s > by_merge) s = by_merge;
    if (s > 32) s = 32;
    return s < 1 ? 1 : (int)s;
}

int icq_launch_select(unsigned long long *keys, const uint32_t *count, int64_t cap, int Q, int topk, int splits, uint32_t *ticket,
                      uint32_t *out_ids, float *out_dist, hipStream_t s) {
    if (Q == 0) return ICQ_OK;
    // 1024 threads while every query's block finds a CU to itself or to share with one other; else 512 threads, of which
    // a CU runs four blocks (1000 queries of 10^4 keys: 34 us against 45), with two minima each where one each would
    // bound the list badly (icq_refine, 2000 queries of 3000 candidates, topk = 512: 1024 threads 167 us, 512 with one
    // minimum 143, with two 91), and 256 threads for lists whose keys all fit (2000 queries of 200, topk = 100: 27 / 21 us,
    // of 1000, topk = 400: 67 / 44 us).  Eight keys per thread in registers: sixteen gain nothing on lists that fit and
    // hold twice the registers on those that do not.
    const uint32_t alone = select_alone(Q, topk);
#define ICQ_SEL(T, PER, MIN) launch_select<T, PER, MIN>(keys, count, cap, Q, topk, splits, alone, ticket, out_ids, out_dist, s)
    if (count && (int64_t)Q * splits <= 512) return ICQ_SEL(1024, 8, 1);
    if (Q > 512 && cap <= SEL_LIST) return ICQ_SEL(256, 4, 2);
    if (topk > 256) return ICQ_SEL(512, 8, 2);
    return ICQ_SEL(512, 8, 1);
#undef ICQ_SEL
}

int icq_launch_join(const unsigned long long *lists, int Q, int parts, int topk, uint32_t *out_ids, float *out_dist, hipStream_t s) {
    if (Q == 0) return ICQ_OK;
    // Two to four lists are joined by rank, more by selection (grouped icq_search, N = 10^6, K = 8, selection / ranks:
    // 500 queries, 2 lists of 100: 40.6 / 37.2 us; 180, 3 lists: 34.8 / 33.7; 130, 4 lists: 36.4 / 36.4; 100, 6 lists:
    // 33.7 / 38.1; 64, 8 lists: 33.3 / 44.5 us).
    if (parts <= 4) {
        join_kernel<<<(unsigned)Q, JOIN_THREADS, 0, s>>>(lists, parts, topk, out_ids, out_dist);
        return icq_check_launch();
    }
    return icq_launch_select(const_cast<unsigned long long *>(lists), nullptr, (int64_t)parts * topk, Q, topk, 1, nullptr,
                             out_ids, out_dist, s);
}
