// Stage 1 of the two-step search (arxiv 1912.08756, Eq. 2) over the pair ordering as a conservative pre-filter in 8-bit
// integers, sixteen queries at a time: what icq_scan16.hip says of the 16-bit form -- a superset of the survivors, the
// exact comparison where the record is in hand -- holds here with half the work per (query, position), for some more items
// let through.
//
// With s a query's unit and m_k its tables' smallest entries, a streamed table is replaced by
//     e_k[c] = min(CAP, floor((T_k[c] - m_k) / s))            (8-bit, CAP = 63 for two streamed tables, 127 for one)
// and the pair's part of the sum, formed once per 16 positions in steps of s / 256 (16-bit, saturating), becomes one byte
//     p = min(128, max(0, floor(128 - 1/8 + (T_0 + T_1 - m_0 - m_1) / s - (t - sum_k m_k) / s))),
// the rounding of the fp32 sums covered by the eighth of a unit (s >= |t| * 2^-16 keeps it below a thirtieth).  An item passes
// when p + e_2 (+ e_3) < 128: every term is rounded down, a streamed entry that stops at CAP is rounded down as well, and
// 128 + 2 * 63 and 128 + 127 fit a byte.  So four queries' sums share a 32-bit word and ONE plain addition adds them with no
// carry between them, a 16-byte LDS read brings sixteen queries' entries, and bit 7 of a byte is clear exactly when the item
// passes; it is collected by a shift and a bit-field insert.  The unit is what lets the largest entry of the streamed tables
// reach CAP, or if that is finer a hundredth of the threshold's distance from the tables' minimum (an eightieth with two streamed tables:
// an entry that stops at CAP is then four fifths of that distance.  With a hundredth it is 0.63, and where the streamed
// codebooks are the larger ones, the first two 0.3 of them, 1.2 to 2.7 times as many items pass as survive, with an eightieth 1.12 to
// 1.21, at shares of 10 to 0.1 %; 1e8 items, 128 queries, whole calls 2345 / 1919 us, 2e7, 64 379 / 299.  Codebooks that shrink or are of one size: within 0.02).
// At 10^8 items, Kf = 4, 1 % survivors, codebooks shrinking by 0.8 the bits mark 8 % more items than survive (16-bit: 0.8 %),
// which costs stage 2 less than a tenth of what stage 1 gains.  A query near the items has entries far below the others in every table (its own codewords); in the first
// two tables they only saturate p.
// What bounds it (10^8 items, 128 queries, 16-bit / 8-bit: 780 / 600 us): vector issue at three quarters of its rate
// (331 instructions per 1024 positions and pass) beside 1.6 GB of hit bits written (without the stores: 468 us; stores of two bytes, of four after a swap between
// neighbouring lanes, ordinary or non-temporal ones, rows of other lengths: the same time).
#include "icq_internal.h"
#include "icq_sort.h"

#include <math.h>

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int Q8_THREADS = 1024;
constexpr int Q8_WAVES = Q8_THREADS / 64;
constexpr int Q8_B = 16;                 // queries per pass
constexpr int Q8_C = 16;                 // copies of a streamed table's entry (lane l reads copy l % 16)
constexpr int Q8_PART = 4;               // positions whose table reads are issued together, while the ones before are added up

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// KF streamed rows (Kf - 2).  Grid: x = ranges of scan positions, y = groups of sixteen queries.  masks [q * mask_stride +
// p / 16] receives the hit bits of positions p .. p + 15 (bit j = position p + j) for every position of the block's range
// below scan_end, zeros beyond the last item.  Rows come in eights (the caller sizes the bits for whole groups of eight
// queries); what a row past the last query receives is read by nobody.
template <int KF>
__global__ __launch_bounds__(Q8_THREADS) void scan_pairs_q8_kernel(
    const uint8_t *rows, int64_t npad, uint32_t N, const float *__restrict__ lut, int K, int m, const float *__restrict__ thr,
    int Q, uint32_t items_per_block, const uint32_t *__restrict__ info, uint16_t *__restrict__ masks, size_t mask_stride,
    uint32_t scan_end) {
    // the streamed tables sit at LDS address 0 (no static arrays in this kernel; the launcher checks that), as in icq_scan16.hip
    extern __shared__ __attribute__((aligned(16))) uint4 q8_smem[];
    constexpr int KFAST = KF + 2;
    constexpr int CAP = KF == 2 ? 63 : 127;
    uint4 *tab = q8_smem;                                            // [KF][256][Q8_C]
    uint4 *t01 = tab + KF * ICQ_LUT_W * Q8_C;                        // [2][256][2]: eight 16-bit entries each
    uint4 *once = t01 + 2 * ICQ_LUT_W * 2;                           // [KF][256]: the streamed entries before they are copied
    float (*s_min)[Q8_B] = reinterpret_cast<float (*)[Q8_B]>(once + KF * ICQ_LUT_W);        // [KFAST]
    float (*s_max)[Q8_B] = s_min + KFAST;                            // [KFAST]: largest entry of a codeword
    float *s_inv = &s_max[KFAST][0];                                 // [Q8_B] 1 / s
    uint32_t *s_off = reinterpret_cast<uint32_t *>(s_inv + Q8_B);    // [Q8_B] added to the first table's entries
    uint32_t *s_sub = s_off + Q8_B;                                  // [Q8_B] taken off the pair's sum
    const int tid = threadIdx.x;
    const uint32_t lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qbase = blockIdx.y * Q8_B;

    const uint32_t begin = blockIdx.x * items_per_block;
    uint32_t end = begin + items_per_block;
    if (end > N || end < begin) end = N;
    uint32_t walk_end = begin + items_per_block;
    if (walk_end > scan_end || walk_end < begin) walk_end = scan_end;
    constexpr uint32_t step = (uint32_t)Q8_WAVES * 1024u;
    const uint32_t nsteps = walk_end > begin ? (walk_end - begin + step - 1) / step : 0;

    uint4 w[2][KF];
    uint32_t ci[2];
    // 1024 positions at g; past the block's range the block's first positions are read instead
    // (unused, in bounds: the rows are padded by more than a block step)
    auto load = [&](uint32_t g, uint4 (&w)[KF], uint32_t &ci) {
        const uint32_t gs = (g < end && g >= begin) ? g : begin;
        ci = info[(gs >> 4) + lane];
#pragma unroll
        for (int k = 0; k < KF; ++k) w[k] = *reinterpret_cast<const uint4 *>(rows + (int64_t)k * npad + gs + lane * 16);
    };
    uint32_t g = begin + wave * 1024u;
    load(g, w[0], ci[0]);                                            // in flight while the tables are prepared

    // slots past the last query repeat it, or where no query is left for the second eight, the first eight (their rows too:
    // rows of hit bits come in eights)
    const int wrap = qbase + Q8_B / 2 < Q ? Q8_B - 1 : Q8_B / 2 - 1;
    auto slot = [&](int b) -> int { return qbase + (b & wrap) < Q ? qbase + (b & wrap) : Q - 1; };
    auto row_of = [&](int b, int k) -> const float * { return lut + ((int64_t)slot(b) * K + k) * ICQ_LUT_W; };
    for (int combo = wave; combo < Q8_B * KFAST; combo += Q8_WAVES) {
        const int b = combo % Q8_B, k = combo / Q8_B;
        const float *r = row_of(b, k);
        float lo = INFINITY, hi = INFINITY;                              // hi: of the negatives
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float v = r[u * 64 + lane];
            lo = fminf(lo, v);
            hi = fminf(hi, u * 64 + (int)lane < m ? -v : INFINITY);
        }
        lo = wave_min_f32(lo);
        hi = -wave_min_f32(hi);
        if (lane == 0) {
            s_min[k][b] = lo;
            s_max[k][b] = hi;
        }
    }
    __syncthreads();
    if (tid < Q8_B) {
        const float t = thr[slot(tid)];
        float L = s_min[0][tid];                                     // the order of the additions of Eq. 2
        float range = 0.0f;
#pragma unroll
        for (int k = 1; k < KFAST; ++k) {
            L += s_min[k][tid];
            if (k >= 2) range = fmaxf(range, s_max[k][tid] - s_min[k][tid]);
        }
        float inv = 0.0f;
        uint32_t off = 0xFFFFu, sub = 0;                             // nothing can pass: t <= L, t = -inf or NaN
        if (t == INFINITY) {
            off = 0;                                                 // everything passes: p = 0, and all quotients are 0
            sub = 0xFFFFu;
        } else if (t > L) {
            const float gap = t - L;
            float s = fminf(range / (float)CAP, gap * (KF == 2 ? 1.0f / 80.0f : 1.0f / 100.0f));
            s = fmaxf(fmaxf(s, gap / 255.0f), fmaxf(fabsf(t) * 1.52587890625e-5f, 1e-30f));
            if (s < INFINITY) {
                inv = 1.0f / s;
                // the pair's sum starts at 128 - 1/8 units less the threshold's, in steps of s / 256
                const int g256 = (int)fminf(floorf(gap * inv * 256.0f), 65535.0f) - (128 * 256 - 32);
                off = g256 < 0 ? (uint32_t)-g256 : 0u;
                sub = g256 > 0 ? (uint32_t)g256 : 0u;
            } else {                                                 // the tables reach beyond the numbers: everything passes
                off = 0;
                sub = 0xFFFFu;
            }
        }
        s_inv[tid] = inv;
        s_off[tid] = off;
        s_sub[tid] = sub;
    }
    __syncthreads();
    // never above the true quotient (x - base) / s: floor, minus a step for the rounding of the product; a NaN (inf * 0) ends as 0
    auto fine = [&](float x, float base, float inv256) -> uint32_t {
        return (uint32_t)fminf(fmaxf(floorf((x - base) * inv256) - 1.0f, 0.0f), 65535.0f);
    };
    if (tid < 2 * ICQ_LUT_W) {
        const int k = tid / ICQ_LUT_W, c = tid % ICQ_LUT_W;
        uint32_t h[Q8_B];
#pragma unroll
        for (int b = 0; b < Q8_B; ++b) {
            h[b] = fine(row_of(b, k)[c], s_min[k][b], s_inv[b] * 256.0f);
            if (k == 0) h[b] = h[b] + s_off[b] < 65535u ? h[b] + s_off[b] : 65535u;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            t01[tid * 2 + u] = make_uint4(h[8 * u] | (h[8 * u + 1] << 16), h[8 * u + 2] | (h[8 * u + 3] << 16),
                                          h[8 * u + 4] | (h[8 * u + 5] << 16), h[8 * u + 6] | (h[8 * u + 7] << 16));
    } else if (tid - 2 * ICQ_LUT_W < KF * ICQ_LUT_W) {
        const int e = tid - 2 * ICQ_LUT_W, k = 2 + e / ICQ_LUT_W, c = e % ICQ_LUT_W;
        uint32_t h[Q8_B];
#pragma unroll
        for (int b = 0; b < Q8_B; ++b) {
            // a step of 1/256 below the quotient, then whole units
            const uint32_t v = fine(row_of(b, k)[c], s_min[k][b], s_inv[b] * 256.0f) >> 8;
            h[b] = v < (uint32_t)CAP ? v : (uint32_t)CAP;
        }
        once[e] = make_uint4(h[0] | (h[1] << 8) | (h[2] << 16) | (h[3] << 24), h[4] | (h[5] << 8) | (h[6] << 16) | (h[7] << 24),
                             h[8] | (h[9] << 8) | (h[10] << 16) | (h[11] << 24), h[12] | (h[13] << 8) | (h[14] << 16) | (h[15] << 24));
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KF * ICQ_LUT_W * Q8_C / Q8_THREADS; ++j) {
        const int p = j * Q8_THREADS + tid;
        tab[p] = once[p / Q8_C];
    }
    uint32_t sub[Q8_B / 2];                                          // wavefront-uniform
#pragma unroll
    for (int j = 0; j < Q8_B / 2; ++j) sub[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(s_sub[2 * j] | (s_sub[2 * j + 1] << 16)));
    __syncthreads();

    // a table address from bytes, as in icq_scan16.hip: byte 0 = this lane's copy (times 16), byte 1 = the sub-code, byte 2 = the table
    const uint32_t lane_bytes = (lane & (Q8_C - 1)) * 16u | 0x100u;  // byte 1 = 1: the source of "table 1"
    uint32_t top_bits;                                               // in a register: an instruction with a literal issues slower
    asm volatile("v_mov_b32 %0, 0x80808080" : "=v"(top_bits));
    // even lanes: (own, other's) low halves; odd lanes: (other's, own) high halves
    const uint32_t swap_sel = lane & 1u ? 0x03020706u : 0x05040100u;
    const uint32_t store_at = (lane & 1u) * (uint32_t)(mask_stride * 2) + (lane >> 1) * 4u;     // bytes: a row is at most 2^28
    uint32_t half_top;
    asm volatile("v_mov_b32 %0, 0x80008000" : "=v"(half_top));
    // MISS bits of the 1024 positions at g: lo[d], hi[d]: positions 0 .. 7 and 8 .. 15 of the lane, byte b = query 4 d + b
    auto misses = [&](const uint4 (&w)[KF], uint32_t ci, uint32_t (&lo)[Q8_B / 4], uint32_t (&hi)[Q8_B / 4]) -> bool {
        uint32_t p[Q8_B / 4];
        {
            const uint4 *a = t01 + (ci & 0xffu) * 2, *c = t01 + (ICQ_LUT_W + ((ci >> 8) & 0xffu)) * 2;
            const uint4 a0 = a[0], a1 = a[1], c0 = c[0], c1 = c[1];
            uint32_t x[Q8_B / 2] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const uint32_t y[Q8_B / 2] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
            for (int j = 0; j < Q8_B / 2; ++j) {
                asm("v_pk_add_u16 %0, %0, %1 clamp\n\tv_pk_sub_u16 %0, %0, %2 clamp\n\tv_pk_min_u16 %0, %0, %3"
                    : "+&v"(x[j]) : "v"(y[j]), "s"(sub[j]), "v"(half_top));
            }
#pragma unroll
            for (int d = 0; d < Q8_B / 4; ++d) p[d] = __builtin_amdgcn_perm(x[2 * d + 1], x[2 * d], 0x07050301u);
        }
        // the streamed tables add at least 0: where every sum has reached 128 in every lane there is no hit among the
        // wavefront's 1024 positions
        if (__builtin_amdgcn_ballot_w64((~(p[0] & p[1] & p[2] & p[3]) & 0x80808080u) != 0u) == 0) return false;
        // positions h .. h + Q8_PART - 1 of the lane: addresses and reads
        auto fetch = [&](int h, uint4 (&v)[Q8_PART][KF]) __attribute__((always_inline)) {
            uint32_t off[Q8_PART][KF];
#pragma unroll
            for (int jj = 0; jj < Q8_PART; ++jj) {
                const int j = h + jj;
#pragma unroll
                for (int k = 0; k < KF; ++k) {
                    const uint32_t word = j < 4 ? w[k].x : j < 8 ? w[k].y : j < 12 ? w[k].z : w[k].w;
                    // selector bytes: 0 = lane_bytes byte 0, 4 + n = byte n of the code word, 1 = lane_bytes byte 1, 0x0c = zero
                    const uint32_t sel = 0x0c000000u | (k == 0 ? 0x000c0000u : 0x00010000u) | ((4u + (j & 3)) << 8);
                    off[jj][k] = __builtin_amdgcn_perm(word, lane_bytes, sel);
                }
            }
#pragma unroll
            for (int jj = 0; jj < Q8_PART; ++jj)
#pragma unroll
                for (int k = 0; k < KF; ++k) {
                    const u32x4 e = *(const __attribute__((address_space(3))) u32x4 *)(uintptr_t)off[jj][k];   // LDS address = table offset
                    v[jj][k] = make_uint4(e.x, e.y, e.z, e.w);
                }
        };
        // the sums of those positions; bit 7 of every byte goes on top of the bits before, moved down by one: what the shift
        // brings there from the byte above is replaced, and the first sum's lower bits are gone after seven more
        auto collect = [&](int h, const uint4 (&v)[Q8_PART][KF]) __attribute__((always_inline)) {
#pragma unroll
            for (int d = 0; d < Q8_B / 4; ++d) {
                uint32_t &acc = h < 8 ? lo[d] : hi[d];
#pragma unroll
                for (int jj = 0; jj < Q8_PART; ++jj) {
                    uint32_t x = p[d];
#pragma unroll
                    for (int k = 0; k < KF; ++k) {
                        const uint4 &t = v[jj][k];
                        x += d == 0 ? t.x : d == 1 ? t.y : d == 2 ? t.z : t.w;
                    }
                    if ((h + jj) % 8 == 0) acc = x;
                    else asm("v_lshrrev_b32 %0, 1, %0\n\tv_bfi_b32 %0, %2, %1, %0" : "+v"(acc) : "v"(x), "v"(top_bits));
                }
            }
        };
        uint4 va[Q8_PART][KF], vb[Q8_PART][KF];
        fetch(0, va);
#pragma unroll
        for (int h = 0; h < 16; h += 2 * Q8_PART) {
            __builtin_amdgcn_sched_barrier(0);
            fetch(h + Q8_PART, vb);
            __builtin_amdgcn_sched_barrier(0);
            collect(h, va);
            __builtin_amdgcn_sched_barrier(0);
            if (h + 2 * Q8_PART < 16) fetch(h + 2 * Q8_PART, va);
            __builtin_amdgcn_sched_barrier(0);
            collect(h + Q8_PART, vb);
        }
        return true;
    };

    // (no condition around a load or store of a step: the waits for a step's codes would then count on none of the stores
    // behind them and wait for those as well)
    for (uint32_t it = 0; it < nsteps; it += 2, g += 2 * step) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u == 1 && it + 1 == nsteps) break;
            load(g + (uint32_t)(u + 1) * step, w[(u + 1) % 2], ci[(u + 1) % 2]);
            const uint32_t gu = g + (uint32_t)u * step;
            uint32_t lo[Q8_B / 4], hi[Q8_B / 4], valid = 0;
            if (gu < end && gu >= begin && misses(w[u], ci[u], lo, hi)) {
                // the padding behind a pair's last item, and positions at or beyond the end
                valid = (1u << (ci[u] >> 16)) - 1u;                  // the label's count is at most 16
                const uint32_t id0 = gu + lane * 16;
                if (id0 + 16 > end || id0 + 16 < id0) valid &= id0 < end ? (1u << (end - id0)) - 1u : 0u;
                valid |= valid << 16;
            } else {
#pragma unroll
                for (int d = 0; d < Q8_B / 4; ++d) lo[d] = hi[d] = 0xFFFFFFFFu;
            }
#pragma unroll
            for (int d = 0; d < Q8_B / 4; ++d) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    // two queries' 16 bits: byte 2 e of lo and hi, byte 2 e + 1 of lo and hi
                    const uint32_t miss = __builtin_amdgcn_perm(hi[d], lo[d], e == 0 ? 0x05010400u : 0x07030602u);
                    const uint32_t hm = ~miss & valid;
                    // neighbouring lanes swap: the even one stores 32 positions of the first query, the odd one of the second
                    const uint32_t other = icq_dpp<0xB1, 0xf, 0u>(hm);               // quad_perm [1, 0, 3, 2]
                    const uint32_t both = __builtin_amdgcn_perm(other, hm, swap_sel);
                    // written once, read once by stage 2: kept out of the caches the code rows are re-read from
                    char *row = reinterpret_cast<char *>(masks + (size_t)(qbase + ((4 * d + 2 * e) & wrap)) * mask_stride + (gu >> 4));
                    __builtin_nontemporal_store(both, reinterpret_cast<uint32_t *>(row + store_at));
                }
            }
        }
    }
}

template <int KF>
int launch_q8(const icq_index *ix, const float *lut, int Q, const float *thr, uint16_t *masks, size_t mask_stride,
              int64_t scan_end, hipStream_t s) {
    const size_t lds = sizeof(uint4) * (size_t)(KF * ICQ_LUT_W * Q8_C + 2 * ICQ_LUT_W * 2 + KF * ICQ_LUT_W) +
                       sizeof(float) * (2 * (KF + 2) + 3) * Q8_B;
    ICQ_HIP_TRY(icq_allow_lds(reinterpret_cast<const void *>(&scan_pairs_q8_kernel<KF>), lds, true));
    const int groups = (Q + Q8_B - 1) / Q8_B;
    const uint32_t step = (uint32_t)Q8_WAVES * 1024u;
    // whole rounds of equally loaded blocks, the fill of a block's tables worth about two steps, as in icq_scan16.hip
    int64_t chunks = icq_scan_pieces(ix->num_cu, groups, (scan_end + step - 1) / step, 2);
    const uint32_t per = (uint32_t)(((scan_end + chunks - 1) / chunks + step - 1) / step * step);
    chunks = (scan_end + per - 1) / per;
    for (int g0 = 0; g0 < groups; g0 += 65535) {
        const int ng = groups - g0 < 65535 ? groups - g0 : 65535;
        const int q0 = g0 * Q8_B, nq = (Q - q0) < ng * Q8_B ? (Q - q0) : ng * Q8_B;
        dim3 grid((unsigned)chunks, (unsigned)ng);
        scan_pairs_q8_kernel<KF><<<grid, Q8_THREADS, lds, s>>>(
            ix->g2_rows, ix->g2_npad, (uint32_t)ix->g2_npos, lut + (int64_t)q0 * ix->K * ICQ_LUT_W, ix->K, ix->m, thr + q0, nq, per,
            ix->g2_info, masks + (size_t)q0 * mask_stride, mask_stride, (uint32_t)scan_end);
    }
    return icq_check_launch();
}

}  // namespace

int icq_launch_scan_masks_q8(const icq_index *ix, const float *lut, int Q, const float *thr, uint16_t *masks,
                             size_t mask_stride, int64_t scan_end, hipStream_t s) {
    if (ix->Kf == 3) return launch_q8<1>(ix, lut, Q, thr, masks, mask_stride, scan_end, s);
    return launch_q8<2>(ix, lut, Q, thr, masks, mask_stride, scan_end, s);
}
