// Rules of the launches: the order in which attention work is dealt to the eight XCDs, and the groups of waves of the search.  No device
// code in here: it compiles for the host too.
#pragma once

namespace fp {

constexpr int kXcds = 8, kCus = 256;
constexpr int kOrderDealt = 0, kOrderByHead = 1, kOrderRounds = 2;

// KV head and row rank of an XCD's `turn`-th super-item (KV head, row); false if there is none.  Consecutive workgroup ids land on
// different XCDs, each with its own L2, and a workgroup stays on its XCD; rows are ranked heaviest (most causal blocks) first.
//
// Sparse lists may be several times as long for one KV head as for another, so that an XCD must not depend on which heads it
// serves: in both orders for them an XCD gets an eighth of every head's rows, there and back (in one direction only, XCD 0 got the
// heaviest row of every eight).
//   dealt    the KV head outermost: the XCDs work on neighbouring rows of one head, whose K and V (128 MiB each at 512K tokens)
//            are what the last-level cache holds at a time, not every head's.
//   rounds   rounds of eight rows, one row of every KV head per XCD and round, each XCD starting at another head: the heaviest rows of
//            all heads run first and the launch ends on light ones.
// In full attention all heads have the same work:
//   by head  an XCD has a KV head of its own (8 / hkv XCDs share one; or it has hkv / 8): one head's K and V are what its L2 sees.
// ROUNDS: whether the kernel's launches can have that order.
template <bool ROUNDS>
__host__ __device__ inline bool attn_item(int order, int xcd, int turn, int m_total, int hkv, int &hk, int &rank) {
    if (order == kOrderByHead) {
        if (hkv < kXcds) {
            const int per = kXcds / hkv, sub = xcd / hkv;   // XCDs per KV head, which of them
            hk = xcd % hkv;
            rank = turn * per + (turn & 1 ? per - 1 - sub : sub);
        } else {
            const int heads = hkv / kXcds;                  // KV heads per XCD
            hk = xcd + kXcds * (turn % heads);
            rank = turn / heads;
        }
        return rank < m_total;
    }
    if (ROUNDS && order == kOrderRounds) {
        const int round = turn / hkv, head = turn - round * hkv + xcd * hkv / kXcds;
        hk = head < hkv ? head : head - hkv;
        // turned from head to head, once round over all of them: a last round of fewer rows takes other XCDs for each
        const int place = (xcd + hk * kXcds / hkv) % kXcds;
        rank = kXcds * round + (round & 1 ? kXcds - 1 - place : place);
        return rank < m_total;
    }
    const int s = turn * kXcds + (turn & 1 ? kXcds - 1 - xcd : xcd);
    hk = s / m_total;
    rank = s - hk * m_total;
    return hk < hkv;
}

constexpr long long kKvCached = 128ll << 20;   // bytes of K and V that the last-level cache (256 MB) holds beside Q and O

// Order of a launch; `parts` is the number of workgroups per q-block.  Attention alone, us, repeated on the same inputs; "equal": all KV
// heads keep the same share of their blocks, "one full": one of them keeps all (32/8: query and KV heads; all orders give the same bits).
//
// Beyond kKvCached the orders that have every head's K and V in use at once lose (by head: 128K tokens of 32/4 heads, 256 MiB, whole pass
// 7505 -> 7612).
// Full attention: by head (dealt -> by head: 8K of 32/4 491.9 -> 470.0, packed 0.5K-9K of 32/8 789.2 -> 744.3, 32K 7292 -> 7298).
// Sparse, one workgroup per CU at most: the longest list sets the time, whichever XCD has it, and K and V of one head per XCD serve
// best (dealt -> by head: 4K of 4/2 equal 31.9 -> 31.6, one full 47.2 -> 44.6; 1000 tokens of 32/8 17.9 -> 18.3, rounds 19.3).
// Sparse, up to 64 workgroups per query head, 96 at head dimension 64, where a CU holds three for two: rounds, which let no heavy row
// start late (dealt -> rounds, equal and one full: 2K of 32/4 42.5 -> 38.6 and 44.4 -> 39.0, 4K 94.0 -> 91.3 and 108.9 -> 104.5, 8K
// 236.2 -> 227.6 and 303.0 -> 297.2, of 32/8 241.1 -> 232.4 and 275.0 -> 271.3; block 64 4K of 32/8 82.9 -> 77.1 and 102.0 -> 97.8;
// block 256 3K of 32/4 79.2 -> 74.8 and 82.0 -> 76.8; head dimension 256 7K of 32/8 372.3 -> 371.9 and 411.4 -> 413.0, on lists of real
// density 315 -> 305; 64 9K of 32/8 173.6 -> 163.7 and 200.3 -> 206.6, 12K of 16/2 134.6 -> 121.2 and 285.2 -> 247.4).  Longer rows are
// balanced either way, and one head's K and V at a time serve better (10K of 32/8 one full 356 -> 359, 16K equal 560 -> 578, block 64 6K
// 144 -> 160, block 256 14K 506 -> 543, head dimension 64 16K of 32/4 315 -> 327, of 16/16 one full 256 -> 297).
// By head would be the fastest for heads that keep alike and is up to twice as slow for others (16K of 32/8, dealt -> by head: equal
// 576 -> 560, one full 743 -> 1361; 8K of 32/4 236 -> 219, 303 -> 383).
inline int attn_order(bool sparse, int head_dim, int parts, int m_total, int hkv, int g, long long kv_bytes) {
    if (kv_bytes > kKvCached) return kOrderDealt;
    if (!sparse || (long long)m_total * hkv * g * parts <= kCus)
        return (hkv < kXcds ? kXcds % hkv == 0 : hkv % kXcds == 0) ? kOrderByHead : kOrderDealt;   // where KV heads go evenly with the XCDs
    return m_total * parts <= (head_dim < 128 ? 96 : 64) ? kOrderRounds : kOrderDealt;
}

// Super-items per XCD, with those that do not exist.
inline int attn_turns(int order, int m_total, int hkv) {
    return order == kOrderRounds ? (m_total + kXcds - 1) / kXcds * hkv : (m_total * hkv + kXcds - 1) / kXcds;
}

// Whether each row of a search launch gets a second group of four waves, which takes every other tile of 32 pooled keys: with no more
// workgroups than CUs there is one wave per SIMD otherwise, which waits for most of a step.  A second set of buffers and longer barriers
// cost about 1 us, at head dimension 256 3 us, so that it pays from some length of the longest row on, earlier the less work a
// tile is: time of two groups over that of one, pooling and search of 2 to 8 rows (scores | lists in one pass):
//   head dimension 64    64-95 key blocks 1.02 | 1.02, 96-127 0.99 | 0.98, 256 0.94 | 0.99, 448 0.90 | 0.95
//   128, block 128       64-95 1.09 | 1.06, 128 1.03 | 1.05, 224 0.98 | 1.02, 352 0.95 | 1.00, 448 0.94 | 0.99
//   block 64, 256        64-95 1.08 | 1.08, 192 1.00 | 1.01, 224 0.97 to 0.99 | 0.98 to 0.99, 448 0.92 to 0.97 | 0.94 to 0.98
//   head dimension 256   64-95 1.17 | 1.13, 224 1.04 | 1.04, 352 1.00 | 1.01, 416 0.99 | 1.00, 512 0.93 | 0.93 (12 rows)
// (2000-token chunk behind 64K tokens, 528 key blocks, 256 workgroups: 53.0 -> 48.0 us.)
inline bool search_two_groups(int head_dim, int block, bool lists, int workgroups, int n_max) {
    const int from = head_dim < 128 ? 96 : head_dim > 128 ? 416 : lists && block == 128 ? 352 : 224;
    return workgroups <= kCus && n_max >= from;
}

}  // namespace fp
