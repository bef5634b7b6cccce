// Internal declarations shared by the HIP translation units of libicq.
// Not installed; the public contract is include/icq.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "icq.h"
#include "icq_lds.h"
#include "icq_pieces.h"

#define ICQ_EXPORT extern "C" __attribute__((visibility("default")))
#define ICQ_LUT_W 256          // table row width (entries j >= m hold +inf)
#define ICQ_WAVE 64            // gfx950 wavefront
#define ICQ_ALIGN 256          // workspace sub-buffer alignment

// Events around the stages of the latest icq_search (icq_index_set_stage_timing).
struct icq_stage_timer {
    hipEvent_t ev[ICQ_TIMED_CALLS][4];
    long long calls;           // searches recorded since the last read (slot = call % ICQ_TIMED_CALLS)
    int batches;               // most sub-batches among them
};

struct icq_index {
    int K, m, d, Kf, Ks;       // Ks = K - Kf slow codebooks
    int d_pad;                 // d rounded up to a multiple of 16 (zero filled)
    int item_stride;           // bytes per item record in `items`
    int device;
    int num_cu;
    int64_t N, Npad;           // Npad: N rounded up to a multiple of 4096
    float *cb;                 // [K*256][d_pad] codewords, rows j >= m are zero
    float *cnorm;              // [K*256] squared codeword norms, +inf for j >= m (in cb's allocation, as the next three)
    uint4 *half_hi, *half_lo;  // the codewords as two halves each, for the encoder (icq_encode.hip); half_lo may be nullptr
    float4 *enc_meta;          // [K] scale of those, largest codeword norm, largest error of the first half
    uint8_t *fast;             // [Kf][Npad] fast sub-codes, zero padded
    uint8_t *items;            // [N][item_stride] all K sub-codes of an item, item-major
    // Grouping by fast-code tuple (Kf <= 2): items with the same fast sub-codes share their
    // crude distance, so batch-mode stage 1 evaluates each tuple once.
    int groups;                // 256^Kf, or 0 when the index is not grouped
    int scan_mode;             // ICQ_SCAN_AUTO / ICQ_SCAN_STREAMED / ICQ_SCAN_GROUPED
    uint32_t *group_start;     // [groups + 1] first grouped position of each tuple
    uint32_t *group_cursor;    // [groups] end of each tuple's items (the build's cursors); read by every bounded search (icq_bound.hip)
    uint32_t *perm;            // [N] grouped position -> item id
    uint8_t *items_grouped;    // [N][item_stride] the item records in grouped order
    // Grouping by the first two fast sub-codes (Kf = 3, 4 and N large enough, icq_group2.hip): the
    // items ordered by that pair -- the pairs themselves in a scattered order, so that any stretch of
    // positions holds unrelated pairs -- every pair's run padded to whole 16 positions.  Stage 1 then
    // streams only the remaining Kf - 2 fast rows and forms the pair's table sum once per 16
    // positions.  Uses group_start [65537], group_cursor [65536] (end of each pair's
    // items, before its padding), perm [g2_npad] (ICQ_PAD_ID in the padding) and
    // items_grouped [g2_npad][item_stride] as the Kf <= 2 grouping does, or g2_halves in its place.
    int g2;                    // 1 when this grouping exists
    int64_t g2_npos;           // positions stage 1 walks: an upper bound of the padded total, whole block steps
    int64_t g2_npad;           // row stride of g2_rows = length of perm / items_grouped (g2_npos + read-ahead spare)
    uint2 *g2_halves;          // [2][g2_npad] first and second halves of records of 16 bytes where stage 2 reads the second half of few, else nullptr
    uint8_t *g2_rows;          // [Kf - 2][g2_npad] the remaining fast sub-codes in grouped order
    uint32_t *g2_info;         // [g2_npad / 16] c0 | c1 << 8 | valid positions << 16 of each 16 positions
    icq_stage_timer *timer;    // nullptr unless stage timing is on
};

// Position of pair (c0, c1) in the grouped order and back: multiplication by an odd constant is a
// bijection on 16 bits that sends neighbouring pairs far apart.
#define ICQ_G2_MUL 0x9E37u
#define ICQ_G2_INV 0x7787u     // ICQ_G2_MUL * ICQ_G2_INV == 1 (mod 65536)
static inline __host__ __device__ uint32_t icq_g2_slot_of_pair(uint32_t pair) { return (pair * ICQ_G2_INV) & 0xFFFFu; }
static inline __host__ __device__ uint32_t icq_g2_pair_of_slot(uint32_t slot) { return (slot * ICQ_G2_MUL) & 0xFFFFu; }
// automatic: when a pair's run averages 64 items or more, so that the padding to 16 weighs little
static inline bool icq_g2_usable(const icq_index *ix) {
    if (!ix->g2 || ix->scan_mode == ICQ_SCAN_STREAMED) return false;
    return ix->scan_mode == ICQ_SCAN_GROUPED || ix->N >= 64ll * 65536;
}
// The same for a search that keeps hit bits and is bounded before stage 2: from fewer items on where many queries share
// the walk, while the padding (half as many positions again at 7.5e5 items and 65536 pairs) does not outweigh two streamed rows fewer and
// what stage 2 gains.  Whole calls, K = 16, Kf = 4, codebooks shrinking by 0.8 / of one size, us, in id order - by pairs: 1 % surviving:
// 5.3e5 items (padded 1.99 times), 500 / 1000 / 2000 queries 115 - 125 / 127, 164 - 194 / 219, 288 - 315 / 349; 7e5 (1.57), 500 / 1000 / 2000:
// 134 - 129 / 140, 200 - 208 / 225, 359 - 345 / 390; 9e5 (1.46), 500: 154 - 134 / 147; 1e6 (1.43), 128 / 250 / 500 / 1000: 73 - 77 / 77, 101 - 98 / 98,
// 162 - 137 / 150, 265 - 227 / 257; 2e6, 32 / 64 / 500: 69 - 64 / 68, 93 - 77 / 83, 269 - 193 / 226; 4.1e6, 32: 115 - 70 / 89.  0.3 %: 1e6, 250 / 500:
// 83 - 93 / 94, 133 - 128 / 136; 2e6, 64 / 128: 70 - 71 / 76, 93 - 83 / 89.  5 %: 1e6, 250: 188 - 121 / 141.  4096 pairs (64 codewords, 1.03 to 1.06):
// 5.3e5, 250 / 1000: 75 - 77 / 76, 162 - 150 / 181; 1e6, 64: 63 - 57 / 58.
static inline bool icq_g2_pays(const icq_index *ix, int Q) {
    if (icq_g2_usable(ix)) return true;
    return ix->g2 && ix->scan_mode == ICQ_SCAN_AUTO && Q >= 32 && 2 * ix->g2_npos <= 3 * ix->N &&
           (double)ix->N * (double)ix->N * (double)ix->N * (double)Q >= 1.8e20;
}
int icq_encode_pack(icq_index *ix, hipStream_t s);             // enc_meta zero on entry
int icq_group2_build(icq_index *ix, hipStream_t s);
int icq_group2_export(const icq_index *ix, uint8_t *codes_out, hipStream_t s);

// What a candidate list holds.
enum icq_list_kind {
    ICQ_LIST_IDS = 0,          // item ids
    ICQ_LIST_POSITIONS = 1,    // grouped positions (ids through perm, records from items_grouped)
    ICQ_LIST_KEYS = 2,         // stage 1 already wrote one 64-bit key (bits of D, id) per survivor
    ICQ_LIST_DONE = 3          // stage 1 kept the nearest-neighbour lists itself and wrote the results
};

// hm = 2 * hm + (P < t): the comparison's carry shifted in with one add (the compiler's own
// form is a select and an or per item).  After n calls the first comparison sits in bit n - 1, the last in bit 0.
// (Tried: the sign of P - t funnel-shifted in -- v_sub_f32 + v_alignbit_b32 issue in 6.3 clocks per item
// against 10.2 for this pair in isolation -- and the table address as shift + v_and_or_b32; both exact,
// neither shortened the scans, which wait on the LDS and on each other's phases rather than on issue slots.)
__device__ __forceinline__ void icq_hit_shift_in(uint32_t &hm, float P, float t) {
    // the two wait states are the ones the compiler itself puts between a vector instruction that
    // writes VCC and one that reads it (it does not look inside an asm statement)
    // (t is wavefront-uniform where this is used and may stay in a scalar register: first source of the compare)
    asm("v_cmp_gt_f32 vcc, %2, %1\n\ts_nop 1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(hm) : "v"(P), "s"(t) : "vcc");
}

// Order-preserving bits of a float: u(a) < u(b) <=> a < b.
__device__ __forceinline__ uint32_t icq_order_bits(float x) {
    // negative: all bits flipped; else the sign bit set -- as an arithmetic shift and one xor-or
    const uint32_t b = __float_as_uint(x);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}

// What the caller knows of the share of items that survive: nothing, that it is some per cent or more, that it is all.
enum icq_share { ICQ_SHARE_UNKNOWN = 0, ICQ_SHARE_MANY = 1, ICQ_SHARE_ALL = 2 };

// Sub-buffers carved out of the caller's workspace for one query batch.
struct icq_ws_layout {
    size_t lut_off, ids_off, count_off, keycount_off, ticket_off, keys_off, total;
    int splits;                // parts a query's work in stage 2 is cut into
    // icq_search with the item-by-item stage 1: hit bits instead of candidate lists (ids_off holds them)
    bool masked;
    bool pairs;                // those bits are over the pair ordering
    bool tickets;              // the selection may take a query's keys in parts
    size_t mask_stride;        // 16-bit words of hit bits per query
    int64_t scan_end;          // scan positions the hit bits cover (whole chunks)
};

static inline size_t icq_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Layout for `Q` queries processed together.  with_lut / with_cands select the
// parts a call needs (icq_scan_fast and icq_refine get their tables and lists
// from the caller).
// small: without the pair ordering where icq_g2_usable does not ask for it.
icq_ws_layout icq_layout(const icq_index *ix, int Q, int64_t cap, int topk, bool with_lut,
                         bool with_cands, bool small = false);
int icq_stage2_splits(const icq_index *ix, int Q, int64_t cap, int topk);
bool icq_selects(const icq_index *ix, int topk);             // stage 2 selects from keys (else the generic kernel)
// icq_search with the item-by-item stage 1 hands the survivors to stage 2 as one hit bit per scan
// position and query instead of lists.
bool icq_masks_usable(const icq_index *ix, int Q, int topk);
int64_t icq_mask_scan_end(const icq_index *ix, bool pairs);  // positions the hit bits cover: whole stage-2 chunks
// icq_search's body; lut_ext (device, [Q][K][256]) replaces the table build when not null.  The table build
// zeroes the call's counters; with lut_ext the caller has done so: out_survivors (not null then) and the first
// 2 * Q words of the workspace, which is at least that long.
int icq_search_impl(const icq_index *ix, const float *queries, const float *lut_ext, int Q, const float *thresholds,
                    int64_t cap, int topk, uint32_t *out_ids, float *out_dist, uint32_t *out_survivors,
                    void *workspace, size_t workspace_bytes, icq_share share, const float *bound_dist, void *stream);
// Stage 1 into hit bits.
int icq_launch_scan_masks(const icq_index *ix, const float *lut, int Q, const float *thr, uint16_t *masks,
                          size_t mask_stride, int64_t scan_end, bool pairs, bool *superset, hipStream_t s);
// The 16-bit pre-filter over the pair ordering (icq_scan16.hip): hit bits of a superset of the survivors.
bool icq_scan_q16_usable(const icq_index *ix, int Q);
int icq_launch_scan_masks_q16(const icq_index *ix, const float *lut, int Q, const float *thr, uint16_t *masks,
                              size_t mask_stride, int64_t scan_end, bool pairs, hipStream_t s);
// The same in 8 bits, sixteen queries at a time (icq_scan8.hip; over the pair ordering).
int icq_launch_scan_masks_q8(const icq_index *ix, const float *lut, int Q, const float *thr, uint16_t *masks,
                             size_t mask_stride, int64_t scan_end, hipStream_t s);
// Stage 2 from hit bits; keys [Q][cap] (+ slice lists in front, see icq_cand_keys); adds the survivors to cand_count.
// superset: the bits mark a superset of the survivors, and an item counts only if its crude distance
// (the first Kf terms of the sum, the additions of Eq. 2) is below thr[q].  bound_dist (may be nullptr): the caller has no
// use for items of query q beyond bound_dist[q][topk - 1], a finite distance.
int icq_launch_refine_masks(const icq_index *ix, const float *lut, int Q, const uint16_t *masks, size_t mask_stride,
                            int64_t scan_end, bool pairs, int64_t cap, int topk, int splits, unsigned long long *keys,
                            uint32_t *key_count, uint32_t *ticket, uint32_t *cand_count, const float *thr, bool superset,
                            const float *bound_dist, uint32_t *out_ids, float *out_dist, hipStream_t s);
// A bound on the topk-th smallest distance into out_dist[q][topk - 1], +inf for none (icq_bound.hip): given[q][topk - 1] (given may
// be nullptr) or what the nearest runs say, tightened where more than about `cap` of the survivors that `masks` marks reach it.
int icq_launch_near_bound(const icq_index *ix, const float *lut, int Q, const float *thr, int topk, const uint16_t *masks,
                          size_t mask_stride, int64_t scan_end, bool pairs, int64_t cap, const float *given, float *out_dist,
                          hipStream_t s);

// p[0..n) = 0, by a kernel (the call can sit inside a captured graph).
void icq_zero_words(uint32_t *p, int n, hipStream_t s);

// Kernel launchers (each checks nothing; the extern "C" entry points validate).
// zero0, zero1, zero2 (may be nullptr): [Q] words each that the launch also sets to zero.
int icq_launch_build_lut(const icq_index *ix, const float *queries, int Q, float *lut, uint32_t *zero0,
                         uint32_t *zero1, uint32_t *zero2, hipStream_t s);
// cand_part == nullptr: the crude distances are not materialised (the fused path
// recomputes the full sum in stage 2 from the item records).
// list_kind == nullptr: the list must hold item ids (public contract).  Otherwise the
// scan picks the cheapest representation for stage 2 and reports it: finished keys in
// cand_keys ([Q][cap], may be nullptr), grouped positions, or plain ids.
// topk / out_ids / out_dist (may be nullptr): where the scan may write the final lists
// itself (ICQ_LIST_DONE) when its grouped form covers stage 2 as well.
// cand_count is zero on entry.
int icq_launch_scan(const icq_index *ix, const float *lut, int Q, const float *thr,
                    uint32_t *cand_ids, float *cand_part, unsigned long long *cand_keys, int *list_kind,
                    uint32_t *cand_count, int64_t cap, int topk, uint32_t *out_ids, float *out_dist,
                    icq_share share, hipStream_t s);
// Grouped stage 1 fused with stage 2: the final lists when icq_group_fused() holds and
// out_ids is given, else one 64-bit key per survivor in cand_keys.
bool icq_group_fused(const icq_index *ix, int Q, int topk);
int icq_launch_group_keys(const icq_index *ix, const float *lut, int Q, const float *thr,
                          unsigned long long *cand_keys, uint32_t *cand_count, int64_t cap, int topk,
                          uint32_t *out_ids, float *out_dist, hipStream_t s);
// Both stages of a small index in one kernel (icq_small.hip): keys of the survivors in cand_keys.
bool icq_small_usable(const icq_index *ix, int Q, int topk, icq_share share);      // (calls that are not grouped by tuple)
int icq_launch_small(const icq_index *ix, const float *lut, int Q, const float *thr, unsigned long long *cand_keys,
                     uint32_t *cand_count, int64_t cap, hipStream_t s);
// Grouped stage 1 (icq_group.hip); as_positions: list grouped positions instead of ids; cand_part may be nullptr.
bool icq_group_usable(const icq_index *ix, int Q);
int icq_group_fused_parts(const icq_index *ix, int Q);
// The topk smallest keys of every query (icq_select.hip; topk <= 512).  count != nullptr: count[q] <= cap keys at
// keys + q * cap, selected in up to `splits` parts (ticket [Q] zero; not read if splits == 1) and used up;
// count == nullptr: cap keys at keys + q * cap, KEY_PAD where there is none, splits = 1.
int icq_select_splits(const icq_index *ix, int Q, int64_t cap, int topk);
int icq_launch_select(unsigned long long *keys, const uint32_t *count, int64_t cap, int Q, int topk, int splits, uint32_t *ticket,
                      uint32_t *out_ids, float *out_dist, hipStream_t s);
// The same from `parts` ascending lists of topk distinct keys per query, KEY_PAD where one is short.
int icq_launch_join(const unsigned long long *lists, int Q, int parts, int topk, uint32_t *out_ids, float *out_dist, hipStream_t s);
int icq_launch_group_scan(const icq_index *ix, const float *lut, int Q, const float *thr,
                          uint32_t *cand_ids, float *cand_part, bool as_positions, uint32_t *cand_count, int64_t cap,
                          hipStream_t s);
int icq_group_build(icq_index *ix, hipStream_t s);
// cand_part == nullptr: D is the full K-term sum; else D = cand_part + slow terms.
// list_kind says what cand_ids holds, see icq_list_kind.
int icq_launch_refine(const icq_index *ix, const float *lut, int Q, const uint32_t *cand_ids,
                      const float *cand_part, int list_kind,
                      const uint32_t *cand_count, int64_t cap, int topk, int splits,
                      unsigned long long *keys, uint32_t *ticket, uint32_t *out_ids, float *out_dist, hipStream_t s);

#define ICQ_HIP_TRY(expr)                      \
    do {                                       \
        hipError_t e__ = (expr);               \
        if (e__ != hipSuccess) return ICQ_ERR_HIP; \
    } while (0)

static inline int icq_check_launch() {
    return hipGetLastError() == hipSuccess ? ICQ_OK : ICQ_ERR_HIP;
}
