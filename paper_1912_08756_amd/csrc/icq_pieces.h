// How stage 1 cuts the scan positions (host side, no device code).
#pragma once
#include <stdint.h>

// Pieces the scan positions (`steps` block steps) are cut into for `groups` groups of queries, one block per CU at a time: the
// number for which whole rounds of blocks take least, a block's tables costing it as much as `fill` steps.  (As many
// pieces as fill the chip, rounded up, can leave a second round nearly empty: 125 groups in 3 pieces each.)
// Of the numbers that take the same rounds only the largest is looked at, no other has shorter pieces: two to four of them.
// (All of them took 1.9 us of a call of one query, 514 numbers.)
static inline int64_t icq_scan_pieces(int num_cu, int64_t groups, int64_t steps, int64_t fill) {
    int64_t best = 1, least = -1;
    int64_t most = 2 * ((num_cu + groups - 1) / groups) + 2;
    if (most > steps) most = steps;
    for (int64_t c = 1; c <= most; ++c) {
        const int64_t rounds = (groups * c + num_cu - 1) / num_cu;
        c = rounds * num_cu / groups;
        if (c > most) c = most;
        const int64_t cost = rounds * ((steps + c - 1) / c + fill);
        if (least < 0 || cost < least) {
            least = cost;
            best = c;
        }
    }
    return best;
}
