// A bound on the result before stage 2 (arxiv 1912.08756, Sec. 3.4: the distance of the furthest element of the
// nearest-neighbour list).  Any topk items that pass the crude comparison bound the topk-th smallest distance from above,
// and the nearer they are the better: the index keeps its items in runs of equal first two fast sub-codes (Kf <= 2: the
// tuples; Kf = 3, 4: the pairs), and where the first codebooks weigh most the runs whose two table entries add up to least
// hold most of a query's neighbours.
//
// One block per query.  The pairs looked at are the four smallest entries of the first table with all of the second; a
// weighted selection (run lengths) among them takes the smallest sums that hold `target` items, the items get the exact
// comparison, every thread keeps the smallest distance of either half of its share, and the topk-th smallest of those
// minima is the bound.  10^8 items, K = 16, topk = 100, codebooks shrinking by 0.8: one or two of the 65536 runs, 2000
// items, give a bound that a few hundred items reach.
//
// How good that bound is depends on the codebooks and on the codes: where the first two tables say little (codebooks of one
// size: 10^5 items reach it at 10^8), or the nearest runs are empty or do not survive (no bound at all), stage 2 would
// write far more keys than the list it has room for.  So there are three looks at the survivors themselves, each for the queries
// that the one before leaves open, by the keys that stage 2 would write:
//   a glance that costs next to nothing -- a few threads take the first hit of every 64 of 128 scan positions, which stands for
//   the hits of its 64, and its record travels beside the others;
//   (more than `limit`, what the caller's lists hold and no more than NB_KEYS:) a sample in which every hit of 65536
//   positions weighs the same, 32 at a place where the index is large: survivors come in runs, and hits that stand for a
//   run mislead;
//   (more again:) stretches of 2048 positions, spread over up to 1/32 of the index, with so many survivors
//   that about `limit` reach the topk-th of them, 128 topk of them at most: that one is the bound then.
// (A separate pass over every 65th part of the index, all survivors' keys written and selected, did the same for 97 us at
// 10^8 items and 128 queries, and left a bound that 65 topk items reach.)  Most keys of a query, 1e8 items, 128 queries, a million
// survivors each, without the looks / with them: first two codebooks a third of the next 1080000 / 22000, codebooks of one size
// 119000 / 115000 (a few queries escape the glance), nearest runs empty 805000 / 111000; 2e7, 64 queries: 217000 / 20500, 27000 / 22500,
// 151000 / 99000.  The bound takes 12 us then as before, 50 with the closer look.
// What bounds it is latency: four trips to memory in a chain and a dozen barriers (1e8 items, 128 queries: 12 us, of which 2 are the
// glance's).
#include "icq_internal.h"
#include "icq_sort.h"

#include <math.h>

namespace {

// (256 / 512 / 1024 threads and 1024 / 2048 items: 1e8 items, one query, 105 / 101 / 103 us, with 2048 items 102 at 512; 1e6, 1000
// queries 275 / 261 / 268, 266; 1e7, two queries, Kf = 2: 39 / 35 / 37, 37)
constexpr int NB_THREADS = 512;
constexpr int NB_PER = 4;              // items a thread fetches together
constexpr int NB_PAIRS = 4 * ICQ_LUT_W;
constexpr uint32_t NB_KEYS = 16384;    // keys a query may leave for the selection before a better bound is worth its look
constexpr int NB_SLOTS = 320;          // the closer look: positions a wavefront collects (four blocks a CU with it, three with 512)
constexpr uint32_t NB_SAMPLE = 2 * NB_THREADS;   // survivors of the sample at most
constexpr int NB_AHEAD = 4;            // the closer look: stretches whose hit bits are asked for together

// FORM: 0 the pairs of Kf = 3, 4 (icq_group2.hip), else the tuples of Kf = FORM.  masks: hit bits over the pair ordering
// (pairs) or over item ids.  given (may be nullptr): a bound known already, given[q][topk - 1], that takes the place
// of the nearest runs'.
template <int WORDS, int FORM>
__global__ __launch_bounds__(NB_THREADS, 8) void near_bound_kernel(
    const uint8_t *__restrict__ items, const uint2 *__restrict__ halves, size_t plane, const uint8_t *__restrict__ by_id, const float *__restrict__ lut, int K,
    int Kf, const float *__restrict__ thr, const uint32_t *__restrict__ run_begin, const uint32_t *__restrict__ run_end,
    uint32_t target, uint32_t most, int topk, const uint32_t *__restrict__ masks, size_t mask_words, uint32_t place, bool pairs,
    uint32_t limit, bool room, const float *given, float *out_dist) {
    constexpr int WAVES = NB_THREADS / 64, PAIRS = NB_PAIRS / NB_THREADS, TABLES = 4 * WORDS;
    __shared__ __attribute__((aligned(16))) float T[TABLES * ICQ_LUT_W];
    __shared__ uint32_t run_pos[NB_PAIRS], run_off[NB_PAIRS + 1];        // the runs taken: first position - offset, offset
    __shared__ uint32_t slots[WAVES][NB_SLOTS];
    static_assert(WAVES * NB_SLOTS >= 5 * NB_THREADS, "the sample's hit bits lie there before");
    uint32_t *held = &slots[0][0];                       // [NB_THREADS] hits before the thread's in its wavefront, [4][NB_THREADS] words
    __shared__ uint32_t wsum[WAVES][2], hsum[WAVES];
    __shared__ uint32_t s_found[2], s_seen[2];
    __shared__ float tmin[4];
    __shared__ IcqKthSharedT<NB_THREADS> kth;
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = blockIdx.x;
    const float t = thr[q];
    const uint32_t *mq = masks + (size_t)q * mask_words;
    // the glance: four words of the 4 * share of each of its threads, apart where a run is longer than a word.  Few threads: each of
    // their reads is a line and a page of its own (whole calls, one / two / eight wavefronts: 1e6 items, 1000 queries 224 / 234 / 235 us;
    // two / eight: 2e7, 64 queries 187 / 193, 1e8, one query 105 / 110)
    const uint32_t part = place >= 64u ? 2u : 3u;       // of the wavefronts, a 2^part-th
    const bool glances = (uint32_t)wave < (uint32_t)WAVES >> part;
    const uint32_t share = place << part, step = place >= 64u ? share : 1u;
    uint32_t glance[2][WORDS], stands[2] = {0u, 0u};
    uint32_t bits[4];
    if (glances) {                                                           // wavefront-uniform
#pragma unroll
        for (int u = 0; u < 4; ++u) bits[u] = mq[(uint32_t)tid * share * 4u + (uint32_t)u * step];
    }
    {
        const float4 *src = reinterpret_cast<const float4 *>(lut + (int64_t)q * K * ICQ_LUT_W);
        constexpr int N4 = TABLES * (ICQ_LUT_W / 4);
#pragma unroll
        for (int i = 0; i < N4; i += NB_THREADS) {
            const int e = i + tid;
            if (e < N4) reinterpret_cast<float4 *>(T)[e] = e / (ICQ_LUT_W / 4) < K ? src[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    if (tid < 2) s_found[tid] = s_seen[tid] = 0;
    // a record by its position in the runs (grouped) or its id
    auto record = [&](bool grouped, uint32_t pos, uint32_t (&rec)[WORDS]) __attribute__((always_inline)) {
        const uint8_t *base = grouped ? items : by_id;
        if (WORDS == 4) {
            // over the pairs: two planes where the walk reads those
            const bool planes = FORM == 0 && grouped && halves;
            const uint2 *at = planes ? halves : reinterpret_cast<const uint2 *>(base);
            const uint2 x = at[planes ? (size_t)pos : (size_t)pos * 2], y = at[planes ? plane + pos : (size_t)pos * 2 + 1];
            rec[0] = x.x;
            rec[1 % WORDS] = x.y;
            rec[2 % WORDS] = y.x;
            rec[3 % WORDS] = y.y;
        } else if (WORDS == 2) {
            const uint2 x = reinterpret_cast<const uint2 *>(base)[pos];
            rec[0] = x.x;
            rec[1 % WORDS] = x.y;
        } else {
            rec[0] = reinterpret_cast<const uint32_t *>(base)[pos];
        }
    };
    // its distance, and the crude one (Kf <= 4 terms)
    auto measure = [&](const uint32_t (&rec)[WORDS], float &crude) __attribute__((always_inline)) -> float {
        float d = T[rec[0] & 0xffu];
        crude = d;
#pragma unroll
        for (int i = 1; i < TABLES; ++i) {
            d += T[i * ICQ_LUT_W + ((rec[i / 4] >> (8 * (i % 4))) & 0xffu)];
            if (i < 4) crude = i < Kf ? d : crude;
        }
        return d;
    };
    if (glances) {                                                           // wavefront-uniform
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t x = bits[2 * u], y = bits[2 * u + 1], w = 2u * (uint32_t)u + (x != 0 ? 0u : 1u);
            uint32_t pos = 0;                                                // no hit: position 0, which there is, for nothing
            if ((x | y) != 0)
                pos = ((uint32_t)tid * share * 4u + w * step) * 32u + (uint32_t)__builtin_ctz(x != 0 ? x : y);
            stands[u] = (uint32_t)(__builtin_popcount(x) + __builtin_popcount(y));
            record(pairs, pos, glance[u]);
        }
    }
    __syncthreads();
    if (wave < Kf) {                                                         // Kf <= 4 <= WAVES
        const float4 x = reinterpret_cast<const float4 *>(T)[wave * (ICQ_LUT_W / 4) + (int)lane];
        const float m = wave_min_f32(fminf(fminf(x.x, x.y), fminf(x.z, x.w)));
        if (lane == 0) tmin[wave] = m;
    }
    // sums of two numbers over the block: before this thread, and all
    auto scan = [&](uint32_t a, uint32_t b, uint32_t &ex_a, uint32_t &ex_b, uint32_t &tot_a, uint32_t &tot_b) {
        const uint32_t ia = wave_scan_add(a), ib = wave_scan_add(b);
        __syncthreads();
        if (lane == 63) { wsum[wave][0] = ia; wsum[wave][1] = ib; }
        __syncthreads();
        uint32_t pa = 0, pb = 0, ta = 0, tb = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t x = wsum[w][0], y = wsum[w][1];
            if (w < wave) { pa += x; pb += y; }
            ta += x; tb += y;
        }
        ex_a = pa + ia - a; ex_b = pb + ib - b;
        tot_a = ta; tot_b = tb;
    };
    // the topk-th smallest of the smallest distances in `least` (those flagged in `any`), +inf if they are fewer; no item is in two
    auto kth_of = [&](const uint32_t (&least)[2], uint32_t any, uint32_t &s_found) __attribute__((always_inline)) -> float {
        const uint32_t have = (uint32_t)(__builtin_popcountll(__builtin_amdgcn_ballot_w64(any & 1u)) +
                                         __builtin_popcountll(__builtin_amdgcn_ballot_w64(any & 2u)));
        if (lane == 0) atomicAdd(&s_found, have);
        __syncthreads();
        if (s_found < (uint32_t)topk) return INFINITY;                       // block-uniform
        return icq_unorder_bits(block_kth<2, NB_THREADS>(kth, least, any, (uint32_t)topk, false, tid, lane, wave));
    };
    float bound = given ? given[(int64_t)q * topk + topk - 1] : INFINITY;
    if (!(bound < INFINITY)) {                                               // block-uniform
        bound = INFINITY;
        // this thread's pairs: the four smallest entries of the first table (every wavefront finds them by itself; equal to
        // their low byte: the smaller code first) with every entry of the second one
        uint32_t v[PAIRS], n[PAIRS], first[PAIRS], valid = 0;
        {
            uint32_t key[4], row[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t c = (uint32_t)u * 64u + lane;
                key[u] = (icq_order_bits(T[c]) & 0xFFFFFF00u) | c;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t a = key[0] < key[1] ? key[0] : key[1], b = key[2] < key[3] ? key[2] : key[3];
                const uint32_t m = wave_min_u32(a < b ? a : b);
                row[r] = m & 0xFFu;
#pragma unroll
                for (int u = 0; u < 4; ++u) key[u] = key[u] == m ? 0xFFFFFFFFu : key[u];
            }
#pragma unroll
            for (int u = 0; u < PAIRS; ++u) {
                const uint32_t i = (uint32_t)u * NB_THREADS + (uint32_t)tid, c = i & (ICQ_LUT_W - 1), r = i / ICQ_LUT_W;   // r: wavefront-uniform
                const uint32_t c0 = FORM == 1 ? c : r == 0 ? row[0] : r == 1 ? row[1] : r == 2 ? row[2] : row[3];
                const uint32_t slot = FORM == 0 ? icq_g2_slot_of_pair(c0 | (c << 8)) : FORM == 1 ? c0 : c0 * 256u + c;
                first[u] = run_begin[slot];
                n[u] = FORM != 1 || i < (uint32_t)ICQ_LUT_W ? run_end[slot] - first[u] : 0u;
                v[u] = icq_order_bits(FORM == 1 ? T[c0] : T[c0] + T[ICQ_LUT_W + c]);
                if (n[u] != 0) valid |= 1u << u;
            }
        }
        // items of all pairs, of the pairs up to the cut
        auto sum = [&](uint32_t flags) {
            uint32_t x = 0;
#pragma unroll
            for (int u = 0; u < PAIRS; ++u) x += (flags >> u) & 1u ? n[u] : 0u;
            return x;
        };
        uint32_t off, at, total, runs;                   // (its barriers also put tmin in place)
        scan(sum(valid), (uint32_t)__builtin_popcount(valid), off, at, total, runs);
        if (total > target) {                                                // block-uniform
            const uint32_t cut = block_kth_impl<PAIRS, true, NB_THREADS>(kth, v, n, valid, target, false, tid, lane, wave);
#pragma unroll
            for (int u = 0; u < PAIRS; ++u)
                if (v[u] > cut) valid &= ~(1u << u);
            scan(sum(valid), (uint32_t)__builtin_popcount(valid), off, at, total, runs);
        }
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
            if (((valid >> u) & 1u) == 0) continue;
            run_pos[at] = first[u] - off;
            run_off[at++] = off;
            off += n[u];
        }
        float smallest = tmin[0];                        // rounding is monotone: no crude distance is below this sum
        for (int k = 1; k < Kf; ++k) smallest += tmin[k];
        if (tid == 0) run_off[runs] = total;
        if (total > most) total = most;
        __syncthreads();
        if (smallest < t) {                                                  // block-uniform
            uint32_t least[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, any = 0;
            for (uint32_t base = 0; base < total; base += NB_THREADS * NB_PER) {
                uint32_t rec[NB_PER][WORDS];
#pragma unroll
                for (int u = 0; u < NB_PER; ++u) {
                    uint32_t i = base + (uint32_t)u * NB_THREADS + (uint32_t)tid;
                    i = i < total ? i : total - 1;
                    uint32_t lo = 0, hi = runs;                              // the last run that starts at or before item i
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (run_off[mid] <= i) lo = mid;
                        else hi = mid;
                    }
                    record(true, run_pos[lo] + i, rec[u]);
                }
#pragma unroll
                for (int u = 0; u < NB_PER; ++u) {
                    float crude;
                    const float d = measure(rec[u], crude);
                    if (base + (uint32_t)u * NB_THREADS + (uint32_t)tid < total && crude < t) {
                        const uint32_t ob = icq_order_bits(d);
                        least[u % 2] = ob < least[u % 2] ? ob : least[u % 2];
                        any |= 1u << (u % 2);
                    }
                }
            }
            bound = kth_of(least, any, s_found[0]);
        }
    }
    auto reaches = [&](float d) -> bool { return !(bound < INFINITY) || icq_order_bits(d) <= icq_order_bits(bound); };
    // the glance: a position looked at stands for `share`; two more hits for what it leaves open
    if (glances) {                                                           // wavefront-uniform
        uint32_t r = 0, c = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float crude;
            const float d = measure(glance[u], crude);
            if (!(crude < t) || stands[u] == 0) continue;
            c += stands[u];
            r += reaches(d) ? stands[u] | 1u << 20 : 0u;                     // (64 hits of 1024 at most, and their number above)
        }
        r = wave_scan_add(r);
        c = wave_scan_add(c);
        if (lane == 63) {
            atomicAdd(&s_seen[0], r);
            atomicAdd(&s_seen[1], c);
        }
    }
    __syncthreads();
    uint32_t reach = s_seen[0] & 0xFFFFFu, seen = s_seen[1];
    const uint32_t ones = s_seen[0] >> 20;
    float each = (float)share;                                               // survivors that one of those seen stands for
    // (a hit that stands for 64 may mislead: where it is only a matter of time four must agree; where the caller's room is short
    // there is always a second look)
    bool closer = !room || (((float)reach + 2.0f) * each > (float)limit && ones >= 4u);      // block-uniform, as is what follows
    if (closer && !(((float)reach + 2.0f) * each > 4.0f * (float)limit && ones >= 8u)) {     // (else there is no doubt)
        // every stride-th hit of four words of each thread's 4 * place
        const uint32_t apart = place >= 64u ? place : 1u;
        uint32_t hits = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t x = mq[(uint32_t)tid * place * 4u + (uint32_t)u * apart];
            hits += (uint32_t)__builtin_popcount(x);
            held[(u + 1) * NB_THREADS + tid] = x;
        }
        const uint32_t upto = wave_scan_add(hits);
        if (lane == 63) hsum[wave] = upto;
        held[tid] = upto - hits;
        __syncthreads();
        uint32_t marked = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) marked += hsum[w];
        const uint32_t stride = marked > NB_SAMPLE ? (marked + NB_SAMPLE - 1) / NB_SAMPLE : 1u, count = (marked + stride - 1) / stride;
        uint32_t r = 0, c = 0;
        if (count != 0) {
            uint32_t rec[2][WORDS];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // hit j's wavefront, thread, word and bit (a thread that expands its own bits keeps its wavefront waiting: up to 128
                // turns where survivors come in runs)
                const uint32_t i = (uint32_t)u * NB_THREADS + (uint32_t)tid;
                uint32_t j = (i < count ? i : count - 1) * stride, at = 0;
#pragma unroll
                for (int w = 0; w < WAVES - 1; ++w) {
                    if (at == (uint32_t)w * 64u && j >= hsum[w]) {
                        j -= hsum[w];
                        at += 64u;
                    }
                }
#pragma unroll
                for (uint32_t half = 32; half != 0; half >>= 1)
                    if (held[at + half] <= j) at += half;                    // the last thread that starts at or before it
                j -= held[at];
                uint32_t x = held[NB_THREADS + at], word = 0, bit = 0;
#pragma unroll
                for (uint32_t k = 1; k < 4; ++k) {
                    const uint32_t next = held[(k + 1) * NB_THREADS + at], n = (uint32_t)__builtin_popcount(x);
                    if (word == k - 1 && j >= n) {
                        j -= n;
                        x = next;
                        word = k;
                    }
                }
#pragma unroll
                for (uint32_t half = 16; half != 0; half >>= 1) {
                    const uint32_t n = (uint32_t)__builtin_popcount(x & ((1u << half) - 1u));
                    if (j >= n) {
                        j -= n;
                        x >>= half;
                        bit += half;
                    }
                }
                record(pairs, (at * place * 4u + word * apart) * 32u + bit, rec[u]);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float crude;
                const float d = measure(rec[u], crude);
                if ((uint32_t)u * NB_THREADS + (uint32_t)tid >= count || !(crude < t)) continue;
                c += 1u;
                r += reaches(d) ? 1u : 0u;
            }
        }
        uint32_t ex;
        scan(r, c, ex, ex, reach, seen);
        each = (float)stride * (float)place;
        closer = ((float)reach + 2.0f) * each > (float)limit;
    }
    if (closer) {
        // survivors wanted, stretches of 64 words per wavefront that hold them: 1/32 of the index, 16 for a small one
        // (half the limit where a key is finished 64 at a time in a chain: stage 2 with first halves only)
        float want = (halves && pairs ? 2.0f : 1.0f) * (float)topk * (float)seen * each / (float)limit;
        want = fminf(fmaxf(want, 8.0f * (float)topk), 128.0f * (float)topk);
        const uint32_t space = place / 8u > 16u ? place / 8u : 16u;          // of 4 * place, 32 at least
        const float need = seen != 0 ? want * 4.0f * (float)place / ((float)seen * each) : (float)space;
        const uint32_t rows = (uint32_t)__builtin_amdgcn_readfirstlane((int)(need < (float)space ? (uint32_t)need + 1u : space));
        uint32_t least[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, any = 0, have = 0;   // have: positions collected (wavefront-uniform)
        uint32_t *list = slots[wave];
        auto work = [&](uint32_t cnt) __attribute__((always_inline)) {       // the last cnt of the list, at most 64 * NB_PER
            wave_lds_order();
            uint32_t rec[NB_PER][WORDS];
#pragma unroll
            for (int u = 0; u < NB_PER; ++u) {
                const uint32_t i = (uint32_t)u * 64u + lane;
                record(pairs, list[have - cnt + (i < cnt ? i : cnt - 1)], rec[u]);
            }
            have -= cnt;
#pragma unroll
            for (int u = 0; u < NB_PER; ++u) {
                float crude;
                const float x = measure(rec[u], crude);
                if ((uint32_t)u * 64u + lane < cnt && crude < t) {
                    const uint32_t ob = icq_order_bits(x);
                    least[u % 2] = ob < least[u % 2] ? ob : least[u % 2];
                    any |= 1u << (u % 2);
                }
            }
            wave_lds_order();
        };
        static_assert(NB_SLOTS >= 64 * NB_PER + 64, "a full list and one more hit per lane");
        // stretches apart, times 2^32: at least one, since rows <= 4 place
        const uint64_t spacing = ((uint64_t)(place * 32u) << 32) / (rows * WAVES);
        uint32_t next[NB_AHEAD], next_at[NB_AHEAD];
        auto ask = [&](uint32_t r) __attribute__((always_inline)) {          // for the words of rows r .. r + NB_AHEAD - 1
#pragma unroll
            for (int u = 0; u < NB_AHEAD; ++u) {
                const uint32_t i = r + (uint32_t)u < rows ? r + (uint32_t)u : rows - 1;
                next_at[u] = (uint32_t)(((uint64_t)(i * WAVES + (uint32_t)wave) * spacing) >> 32) * 64u;
                next[u] = mq[next_at[u] + lane];
            }
        };
        ask(0);
        for (uint32_t r = 0; r < rows; r += NB_AHEAD) {                      // wavefronts on their own
            uint32_t w[NB_AHEAD], at[NB_AHEAD];
#pragma unroll
            for (int u = 0; u < NB_AHEAD; ++u) {
                w[u] = next[u];
                at[u] = next_at[u];
            }
            if (r + NB_AHEAD < rows) ask(r + NB_AHEAD);
#pragma unroll
            for (int u = 0; u < NB_AHEAD; ++u) {
                if (r + (uint32_t)u >= rows) break;
                for (uint32_t x = w[u];;) {                                  // one hit per lane and turn
                    const uint64_t mk = __builtin_amdgcn_ballot_w64(x != 0);
                    if (mk == 0) break;
                    if (x != 0)
                        list[__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, have))] =
                            (at[u] + lane) * 32u + (uint32_t)__builtin_ctz(x);
                    have += (uint32_t)__builtin_popcountll(mk);
                    x &= x - 1;
                    if (have > NB_SLOTS - 64) work(64 * NB_PER);
                }
            }
        }
        while (have != 0) work(have < 64u * NB_PER ? have : 64u * NB_PER);
        const float kth_seen = kth_of(least, any, s_found[1]);
        if (kth_seen < bound) bound = kth_seen;
    }
    if (tid == 0) out_dist[(int64_t)q * topk + topk - 1] = bound;
}

}  // namespace

// out_dist[q][topk - 1] = an upper bound of query q's topk-th smallest distance among the survivors that `masks` marks (a
// superset does), +inf for none; such that about `cap` survivors reach it at most, where the survivors' sample can
// see to that.
int icq_launch_near_bound(const icq_index *ix, const float *lut, int Q, const float *thr, int topk, const uint16_t *masks,
                          size_t mask_stride, int64_t scan_end, bool pairs, int64_t cap, const float *given, float *out_dist,
                          hipStream_t s) {
    const uint32_t target = 8u * (uint32_t)topk > 1024u ? 8u * (uint32_t)topk : 1024u;
    // a key is a line of ids read and one of keys written: fewer of them pay where there are hundreds of queries
    const int64_t pays = (2 << 20) / (int64_t)Q, keys = pays > NB_KEYS ? NB_KEYS : pays > 2048 ? pays : 2048;
    const bool room = cap / 2 >= keys;                                       // half of it: a sample may mislead
    const uint32_t limit = room ? (uint32_t)keys : (uint32_t)(cap / 2);
    const uint32_t place = (uint32_t)(scan_end / 128 / NB_THREADS);          // scan_end: 2^19 at least
    const int words = ix->item_stride / 4;
    auto go = [&](auto kernel) {
        kernel<<<(unsigned)Q, NB_THREADS, 0, s>>>(ix->items_grouped, ix->g2_halves, (size_t)ix->g2_npad, ix->items, lut, ix->K, ix->Kf, thr,
                                                  ix->group_start, ix->group_cursor, target, 2 * target, topk,
                                                  reinterpret_cast<const uint32_t *>(masks), mask_stride / 2, place, pairs, limit,
                                                  room, given, out_dist);
    };
#define ICQ_NB(FORM)                                                   \
    do {                                                               \
        if (words == 1) go(near_bound_kernel<1, FORM>);                \
        else if (words == 2) go(near_bound_kernel<2, FORM>);           \
        else go(near_bound_kernel<4, FORM>);                           \
    } while (0)
    if (ix->Kf > 2) ICQ_NB(0);
    else if (ix->Kf == 1) ICQ_NB(1);
    else ICQ_NB(2);
#undef ICQ_NB
    return icq_check_launch();
}
