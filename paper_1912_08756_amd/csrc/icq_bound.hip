// A bound on the result before stage 2 (arxiv 1912.08756, Sec. 3.4: the distance of the furthest element of the
// nearest-neighbour list).  Any topk items that pass the crude comparison bound the topk-th smallest distance from above,
// and the nearer they are the better: the index keeps its items in runs of equal first two fast sub-codes (Kf <= 2: the
// tuples; Kf = 3, 4: the pairs), and the runs whose two table entries add up to least hold most of a query's neighbours.
// 10^8 items, K = 16, topk = 100: one or two of the 65536 runs, 2000 items, give a bound that a few hundred items reach, in 12 us; an
// unfiltered walk over every 65th part of the index took 97 us for one that 6500 reach.
//
// One block per query.  The pairs looked at are the four smallest entries of the first table with all of the second; a
// weighted selection (run lengths) among them takes the smallest sums that hold `target` items, the items get the exact
// comparison, every thread keeps the smallest distance of either half of its share, and the topk-th smallest of those
// minima is the bound.  Where fewer than topk pass, items spread over the whole index are looked at instead (the nearest
// runs may be empty, or hold none of the survivors), and where those do not do either the bound is +inf.
// What bounds it is latency: four trips to memory in a chain and a dozen barriers; then the LDS, 16 table entries an item
// (24000 items: 37 us).
#include "icq_internal.h"
#include "icq_sort.h"

#include <math.h>

namespace {

// (256 / 512 / 1024 threads and 1024 / 2048 items: 1e8 items, one query, 105 / 101 / 103 us, with 2048 items 102 at 512; 1e6, 1000
// queries 275 / 261 / 268, 266; 1e7, two queries, Kf = 2: 39 / 35 / 37, 37)
constexpr int NB_THREADS = 512;
constexpr int NB_PER = 4;              // items a thread fetches together
constexpr int NB_PAIRS = 4 * ICQ_LUT_W;
constexpr uint32_t NB_SPREAD = 16384;  // items of the second look

// FORM: 0 the pairs of Kf = 3, 4 (icq_group2.hip), else the tuples of Kf = FORM.
template <int WORDS, int FORM>
__global__ __launch_bounds__(NB_THREADS) void near_bound_kernel(
    const uint8_t *__restrict__ items, size_t plane, const uint8_t *__restrict__ by_id, uint32_t N,
    const float *__restrict__ lut, int K, int Kf, const float *__restrict__ thr, const uint32_t *__restrict__ run_begin, const uint32_t *__restrict__ run_end, uint32_t target, uint32_t most, int topk,
    float *__restrict__ out_dist) {
    constexpr int WAVES = NB_THREADS / 64, PAIRS = NB_PAIRS / NB_THREADS;
    __shared__ __attribute__((aligned(16))) float T[4 * WORDS * ICQ_LUT_W];
    __shared__ uint32_t run_pos[NB_PAIRS], run_off[NB_PAIRS + 1];        // the runs taken: first position - offset, offset
    __shared__ uint32_t wsum[WAVES][2];
    __shared__ uint32_t s_found;
    __shared__ float tmin[4];
    __shared__ IcqKthSharedT<NB_THREADS> kth;
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = blockIdx.x;
    const float t = thr[q];
    {
        const float4 *src = reinterpret_cast<const float4 *>(lut + (int64_t)q * K * ICQ_LUT_W);
        constexpr int N4 = 4 * WORDS * (ICQ_LUT_W / 4);
#pragma unroll
        for (int i = 0; i < N4; i += NB_THREADS) {
            const int e = i + tid;
            if (e < N4) reinterpret_cast<float4 *>(T)[e] = e / (ICQ_LUT_W / 4) < K ? src[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    if (tid == 0) s_found = 0;
    __syncthreads();
    if (wave < Kf) {                                                         // Kf <= 4 <= WAVES
        const float4 x = reinterpret_cast<const float4 *>(T)[wave * (ICQ_LUT_W / 4) + (int)lane];
        const float m = wave_min_f32(fminf(fminf(x.x, x.y), fminf(x.z, x.w)));
        if (lane == 0) tmin[wave] = m;
    }
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
    auto sum = [&](uint32_t flags) {
        uint32_t x = 0;
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) x += (flags >> u) & 1u ? n[u] : 0u;
        return x;
    };
    uint32_t off, at, total, runs;                       // (its barriers also put tmin in place)
    scan(sum(valid), (uint32_t)__builtin_popcount(valid), off, at, total, runs);
    if (total > target) {                                                    // block-uniform
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
    float smallest = tmin[0];                            // rounding is monotone: no crude distance is below this sum
    for (int k = 1; k < Kf; ++k) smallest += tmin[k];
    float bound = INFINITY;
    if (tid == 0) run_off[runs] = total;
    if (total > most) total = most;
#pragma nounroll
    for (int look = smallest < t ? 0 : 2; look < 2; ++look) {                // block-uniform
        if (look == 1) total = N < NB_SPREAD ? N : NB_SPREAD;
        __syncthreads();
        if (tid == 0) s_found = 0;
        uint32_t least[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, any = 0;
        for (uint32_t base = 0; base < total; base += NB_THREADS * NB_PER) {
            uint32_t rec[NB_PER][WORDS];
#pragma unroll
            for (int u = 0; u < NB_PER; ++u) {
                uint32_t i = base + (uint32_t)u * NB_THREADS + (uint32_t)tid;
                i = i < total ? i : total - 1;
                const uint8_t *from = items;
                uint32_t pos;
                if (look == 0) {
                    uint32_t lo = 0, hi = runs;                              // the last run that starts at or before item i
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (run_off[mid] <= i) lo = mid;
                        else hi = mid;
                    }
                    pos = run_pos[lo] + i;
                } else {
                    pos = (uint32_t)((uint64_t)i * N / total);               // distinct: total <= N
                    from = by_id;
                }
                const uint32_t *p = reinterpret_cast<const uint32_t *>(from + (size_t)pos * (WORDS * 4));
                if (FORM == 0 && WORDS == 4 && look == 0) {                  // two planes
                    const uint2 x = reinterpret_cast<const uint2 *>(items)[pos], y = reinterpret_cast<const uint2 *>(items)[plane + pos];
                    rec[u][0] = x.x;
                    rec[u][1 % WORDS] = x.y;
                    rec[u][2 % WORDS] = y.x;
                    rec[u][3 % WORDS] = y.y;
                } else if (WORDS == 1) {
                    rec[u][0] = p[0];
                } else if (WORDS == 2) {
                    const uint2 x = *reinterpret_cast<const uint2 *>(p);
                    rec[u][0] = x.x;
                    rec[u][1 % WORDS] = x.y;
                } else {
                    const uint4 x = *reinterpret_cast<const uint4 *>(p);
                    rec[u][0] = x.x;
                    rec[u][1 % WORDS] = x.y;
                    rec[u][2 % WORDS] = x.z;
                    rec[u][3 % WORDS] = x.w;
                }
            }
#pragma unroll
            for (int u = 0; u < NB_PER; ++u) {
                float d = T[rec[u][0] & 0xffu], crude = d;
#pragma unroll
                for (int i = 1; i < 4 * WORDS; ++i) {
                    d += T[i * ICQ_LUT_W + ((rec[u][i / 4] >> (8 * (i % 4))) & 0xffu)];
                    if (i < 4) crude = i < Kf ? d : crude;
                }
                if (base + (uint32_t)u * NB_THREADS + (uint32_t)tid < total && crude < t) {
                    const uint32_t ob = icq_order_bits(d);
                    least[u % 2] = ob < least[u % 2] ? ob : least[u % 2];
                    any |= 1u << (u % 2);
                }
            }
        }
        const uint32_t have = (uint32_t)(__builtin_popcountll(__builtin_amdgcn_ballot_w64(any & 1u)) +
                                         __builtin_popcountll(__builtin_amdgcn_ballot_w64(any & 2u)));
        __syncthreads();                                                     // s_found is zero
        if (lane == 0) atomicAdd(&s_found, have);
        __syncthreads();
        if (s_found < (uint32_t)topk) continue;                              // block-uniform
        bound = icq_unorder_bits(block_kth<2, NB_THREADS>(kth, least, any, (uint32_t)topk, false, tid, lane, wave));
        break;
    }
    if (tid == 0) out_dist[(int64_t)q * topk + topk - 1] = bound;
}

}  // namespace

// out_dist[q][topk - 1] = an upper bound of query q's topk-th smallest distance among the survivors, +inf for none.
int icq_launch_near_bound(const icq_index *ix, const float *lut, int Q, const float *thr, int topk, float *out_dist, hipStream_t s) {
    const uint32_t target = 8u * (uint32_t)topk > 1024u ? 8u * (uint32_t)topk : 1024u;
    const int words = ix->item_stride / 4;
    auto go = [&](auto kernel) {
        kernel<<<(unsigned)Q, NB_THREADS, 0, s>>>(ix->items_grouped, (size_t)ix->g2_npad, ix->items, (uint32_t)ix->N, lut, ix->K, ix->Kf,
                                                  thr, ix->group_start, ix->group_cursor, target, 2 * target, topk, out_dist);
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
