// Internal declarations shared by the host entry points and the kernels of
// libseamdecode.  Not installed; the public interface is include/seamdecode.h.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <algorithm>

namespace sd {

constexpr int kPage = 16;           // tokens per page
constexpr int kWaves = 4;           // waves per workgroup of the split pass
constexpr int kTileTokens = 32;     // tokens one wave consumes per iteration (two pages)
constexpr int kMaxGroup = 16;       // query heads per KV head that fit one MFMA tile
constexpr int kMaxHeadBlocks = 4;   // a KV head with more query heads is served as up to 4 blocks of 16

// A KV head with G > 16 query heads is split into HB = ceil(G / 16) "virtual" KV heads that read the
// same K/V tiles: virtual head gv = g * HB + hb owns the query heads g * G + 16 * hb .. (16 of them, the
// last block G - 16 * (HB - 1)).  With G <= 16 there is one block and gv == g.
struct HeadBlock {
    int g;       // KV head (addresses the pools)
    int head0;   // first query head of the block
    int rows;    // query heads in the block (<= 16)
};
__host__ __device__ inline int head_blocks(int G) { return (G + kMaxGroup - 1) / kMaxGroup; }
__host__ __device__ inline HeadBlock head_block(int gv, int G, int HB)
{
    const int g = gv / HB, hb = gv - g * HB;
    const int left = G - hb * kMaxGroup;
    return HeadBlock{g, g * G + hb * kMaxGroup, left < kMaxGroup ? left : kMaxGroup};
}
// Sequences (decode) or query tokens (causal pass) that share one 16-row column block.
__host__ __device__ inline int units_per_block(int G) { return G <= kMaxGroup / 2 ? kMaxGroup / G : 1; }
constexpr int kXcds = 8;            // accelerator dies, each with its own L2; workgroup i runs on die i % 8
// Deal of a grid's items to the dies.  Items i and i + 1 differ in the head (head fastest, `Hv` of
// them) and would run on different dies; lines that the heads of one sequence have in common (the
// scales of a page's heads lie in one line, so do its block-table entries) would then be fetched
// once per die.  Within every run of 8 * Hv items this hands the Hv items of one sequence to one
// die, one after the other; a ragged last run stays as it is.  A bijection of [0, n).
__device__ inline unsigned xcd_deal(unsigned i, unsigned n, unsigned Hv)
{
    const unsigned run = kXcds * Hv;
    const unsigned k = i / run, j = i - k * run;
    if ((k + 1) * run > n) return i;
    return k * run + (j % kXcds) * Hv + j / kXcds;
}
// Deal of the causal pass's items, (sequence, head) pair x block of query tokens, to the dies.  All query
// blocks of a pair read the same K/V, so they get consecutive slots of ONE die (early items = late positions
// = long ranges first): they run side by side, walk the range at about the same pace, and all but the first find
// the tiles in that die's L2.  Pairs go to the dies in turn, so that the heads of one sequence spread over all
// dies and a ragged batch loads them alike; what is left over (pairs mod 8) is cut into classes of
// query blocks, as many as it takes to give every die the same share.  (Measured against runs of consecutive pairs
// per die, where the die with the longest sequence ends last: 8 whole prompts of 1.5 k to 4 k tokens, 32/8
// heads, d = 64: 547 -> 436 us; 12 resumed fp8 sequences of 2.5 k to 8 k: 1788 -> 1500 us; equal lengths: no change.)
struct PrefillItem {
    int pair, block;   // block >= q_blocks: nothing to do
};
__host__ __device__ inline int prefill_classes(int rest)   // of a left-over pair: 8 / gcd(8, rest)
{
    return rest % 4 == 0 ? 2 : rest % 2 == 0 ? 4 : 8;
}
__host__ __device__ inline PrefillItem prefill_item(unsigned i, int q_blocks, int pairs)
{
    const int die = i % kXcds;
    unsigned k = i / kXcds;
    const unsigned whole = (unsigned)(pairs / kXcds) * (unsigned)q_blocks;   // slots of a die that serve whole pairs
    if (k < whole) return PrefillItem{die + kXcds * (int)(k / q_blocks), (int)(k % q_blocks)};
    k -= whole;
    const int rest = pairs % kXcds, classes = prefill_classes(rest), per_class = (q_blocks + classes - 1) / classes;
    const int unit = die + kXcds * (int)(k / per_class);
    return PrefillItem{pairs - rest + unit / classes, (int)(k % per_class) * classes + unit % classes};
}
__host__ __device__ inline unsigned prefill_grid(int q_blocks, int pairs)
{
    const int rest = pairs % kXcds, classes = prefill_classes(rest);
    return (unsigned)(pairs / kXcds * kXcds) * (unsigned)q_blocks + (rest ? (unsigned)(rest * classes) * (unsigned)((q_blocks + classes - 1) / classes) : 0u);
}
// 2^32 / tokens, rounded up: the high half of x times it is x / tokens for x < 2^24 and tokens <= 256 (a workgroup has at least two).
__host__ inline uint32_t reciprocal_of(unsigned tokens) { return (uint32_t)((((uint64_t)1 << 32) + tokens - 1) / tokens); }
// Longest first.  The order in which the query blocks of a batch start when the kernel looks at the lengths: by the class of their
// range (eighths or quarters of the longest, counted in blocks), descending; within a class sequence after sequence, late blocks first, so that
// neighbours still walk the same K/V together.  A block takes as long as its range, and a list that starts long items late ends late.  The
// heads of a block go to the dies in turn, whatever sequence it is from, so no die is left with the longest sequences either.
//
// `s` gives every sequence's query blocks and where its last one ends (in blocks, rounded up): sum(f) = sum of f(end, blocks) over the sequences,
// top() = the largest end, find(f, m) = the sequence in which the running sum of f passes m, and that sum before it.
constexpr int kMaxOrderedBatch = 64;   // sequences whose ends and blocks one wave holds, one to a lane
struct PrefillBlock {
    int b, block;   // block < 0: there is no k-th block
};
template <class Sequences>
__host__ __device__ inline PrefillBlock prefill_pick(const Sequences &s, int k, int classes)
{
    const int top = s.top();
    // blocks of a sequence that end above the lower edge of class c
    const auto above = [top, classes](int c, int end, int blocks) {
        const int n = c == 0 ? blocks : end - (int)((uint64_t)top * (unsigned)c / (unsigned)classes);
        return n < 0 ? 0 : n < blocks ? n : blocks;
    };
    if (s.sum([above](int end, int blocks) { return above(0, end, blocks); }) <= k) return PrefillBlock{0, -1};
    int lo = 0, hi = classes, higher = 0;   // block k lies in a class of [lo, hi); `higher` blocks end above hi's edge
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        const int n = s.sum([above, mid](int end, int blocks) { return above(mid, end, blocks); });
        if (n > k) lo = mid;
        else hi = mid, higher = n;
    }
    const auto at = s.find([above, lo, hi](int end, int blocks) { return above(lo, end, blocks) - above(hi, end, blocks); }, k - higher);
    return PrefillBlock{at.b, at.blocks - 1 - above(hi, at.end, at.blocks) - (k - higher - at.before)};
}
// The block that workgroup i of a call takes whose size the kernel has chosen: longest first (head fastest); but where all workgroups run at once, so that
// their order is of no account, and a head would not keep its die (heads no multiple of 8), pair by pair, as many workgroups to every die: the blocks of all
// but 7 pairs meet on one die, where the others find in its L2 what the first fetches.  (Random calls that this applies to, longest first over pair by pair: 2 heads
// 1.04 with 8 blocks, 1.17 with 4, 4 heads 1.04 and 1.08; 27 sequences of 7.6 - 8.4 k, 51 queries, 8/2 heads, 4 blocks 124 : 78 us.)  The grid has a multiple
// of 8 workgroups, at least as many as there are blocks.
constexpr int kChosenClasses = 8;
struct PrefillSlot {
    int b, head, block;   // block < 0: nothing to do
};
template <class Sequences>
__host__ __device__ inline PrefillSlot prefill_slot(const Sequences &s, unsigned i, int heads)
{
    const int n = s.sum([](int, int blocks) { return blocks; }) * heads;
    if (heads % kXcds == 0 || n > 256) {
        const PrefillBlock at = prefill_pick(s, (int)(i / heads), kChosenClasses);
        return PrefillSlot{at.b, (int)(i % heads), at.block};
    }
    const int per_die = (n + kXcds - 1) / kXcds, k = (int)(i / kXcds), r = (int)(i % kXcds) * per_die + k;
    if (k >= per_die || r >= n) return PrefillSlot{0, 0, -1};
    const auto at = s.find([heads](int, int blocks) { return blocks * heads; }, r);
    return PrefillSlot{at.b, (r - at.before) / at.blocks, at.blocks - 1 - (r - at.before) % at.blocks};
}
// How a call of the causal pass is cut: column blocks of 16 query rows that a workgroup owns (16, 8, 4 or 2), the waves that share the
// range of a block, and whether the workgroups run in two phases (bf16 pools with head_dim 128).
struct PrefillPlan {
    int blocks, split;
    bool phases, direct;   // 16 blocks over bf16 pools with head_dim 128: in two phases, or straight into LDS in one
    bool on_device;        // 8 or 4 blocks, as the kernel finds better for the lengths (prefill_on_device); blocks and split are those of 8
    int order;             // longest first (prefill_pick), in so many classes; 0: dealt by prefill_item
};
// Large blocks share a tile among most rows; small ones give more workgroups, and below 16 (head_dim 128) or 8 (head_dim 64) several
// waves share a block's range.  The line lies where the workgroups of the next larger block no longer fill the chip: about half a
// workgroup per compute unit at head_dim 128, which runs one at a time, and one at head_dim 64, which runs two or three.  Workgroups whose
// rows are mostly empty end early, and long ranges gain more by being shared, so both move the line up.
// The lines over bf16 pools at head_dim 128 are fitted to 1740 random calls (1 to 24 sequences of 200 to 16 k tokens, 8 to 2048 queries, heads as in
// perf/cases.py), each timed with every block size; by these lines alone a call takes 1.8 % more than with the best size on average, 136 take more than 1.1 and 64 more than 1.2 of it.
// From 1536 tokens on whether 8 or 4 blocks suit a call is a matter of how its lengths are spread: there the kernel chooses (prefill_on_device; with the better of the two for every
// call that it may choose for 1.5 %, 110 and 56), and the lines of 8 and 4 hold for the rest: under 96 workgroups of 8 blocks, single sequences, more than 64, loose bounds on the
// queries.  (192 for 8 over 4 blocks from 2048 tokens on: 800 calls drawn for it, .99 of the time with 8 from 176 workgroups on, .94 from 192 to 255.)  Geometric mean of the time with 16 / 8, 8 / 4 and
// 4 / 2 blocks by workgroups of the larger block, half of its rows in use or more:
//   workgroups              24 - 95   96 - 134   135 - 191   192 - 270   271 - 383   384 - 542   543 and more
//   under 512 tokens   16    1.17      1.12        0.82        0.86        0.84        0.79       0.73
//                       8    1.24      1.07        0.80        0.84        0.86        0.75       0.71
//                       4    1.24      1.02        0.75        0.82        0.84        0.76       0.72
//   under 2048         16    1.41      1.35        1.02        0.94        0.83        0.83       0.78
//                       8    1.38      1.32        0.93        0.85        0.89        0.78       0.76
//                       4    1.37      1.10        0.82        0.79        0.88        0.76       0.73
//   6000 and more      16    1.79      1.67        1.33        1.08        1.14        0.95       0.94
//                       8    1.57      1.43        1.13        0.94        0.96        0.86       0.87
//                       4    1.60      1.43        1.06        0.97        1.00        0.90       0.88
// (From 2048 tokens on 192 - 255 workgroups of 16 blocks stay, 257 - 319 are cut: of 185 calls that one line at 288 would move, 10 become slower by more than
// 8 % with it and 2 with these; the average is the same.)
// (Under 512 tokens a single wave used to walk the range alone: two sequences of 131 - 397 tokens, 220 queries, 8/2 heads 18.5 -> 9.5 us.)
// At head_dim 64 over bf16 pools the lines of 8 and 4 blocks are fitted to 900 such calls; the rule costs 1 % over the best size of each call, the lines further
// down, which stay for fp8 pools, 6 % (three of 278 - 457 tokens, 2 - 16 queries, 16/2 heads 12.0 against 6.9 us with 2 blocks).
//   workgroups              under 96   96 - 127   128 - 191   192 - 255   256 - 383   384 - 511   512 - 767   768 - 1023   1024 and more
//   under 512 tokens    8    0.95        0.92       0.81        0.82        0.69        0.67        0.61         0.59       0.51
//                       4    1.46        1.32       1.16        1.18        0.95        0.91        0.96         0.87       0.85
//   under 2048          8    1.42        1.27       1.17        1.18        0.99        0.80        0.79         0.69       0.64
//                       4    1.61        1.52       1.22        1.23        0.98        0.83        0.96         0.85       0.85
//   4096 and more       8    2.12        1.89       1.76        1.72        1.45        1.31        1.13         1.07       0.96
//                       4    1.95        1.68       1.47        1.35        1.09        0.91        0.98         0.90       0.86
// The other lines were fitted to 4200 random calls (1 to 64 sequences of 1 to
// 12000 tokens, 1 to 3000 queries each, 1 to 32 heads per KV head, bounds tight and 4 and 16 times too wide), each timed with every
// block size; there contexts below kPrefillShort tokens are not split.  Geometric mean of the time with 16 / 8, 8 / 4 and 4 / 2 blocks, by workgroups of
// the larger block (tight bounds; as the kernels that park through registers take them):
//   workgroups       64 - 95  96 - 127  128 - 159  160 - 191  192 - 255  256 - 383  512 - 767  1024 and more
//   head_dim 128  16   1.32     1.22       1.10       1.04       0.96       0.91       0.86       0.76
//                  8   1.27     1.18       1.06       0.98       0.96       0.90       0.78       0.74
//                  4   1.20     1.11       0.99       0.87       0.86       0.92       0.80       0.72
//   head_dim 64   16   1.33     1.34       1.31       1.20       1.28       1.15       1.05       1.02; from 4096 on 0.96
//                  8   1.52     1.40       1.31       1.27       1.34       1.12       0.97       0.77
//                  4   1.41     1.33       1.46       0.92       0.98       0.79       0.81       0.54
// Contexts of 2048 tokens and more, whose last workgroup runs longer, move the lines up again.  At head_dim 64 blocks of 16 are
// for bf16 pools (over fp8 pools they take 1.1 to 1.2 of the time of 8 from 256 workgroups on).
// The grid has room for max_q_len queries of every sequence, and workgroups that find none cost their start: 55 sequences of up to 45 queries under a
// bound of 1302, 4/1 heads 14.6 / 20.8 / 27.5 / 37.8 us with 16 / 8 / 4 / 2 blocks (1155, 2255, 4510 and 8965 workgroups).  No smaller blocks than
// a grid of 4096 allows.
// The two phases leave the matrix pipe to the waves in turn, also to those without rows: by the share of the 16 blocks that the average
// sequence's queries fill, time against one phase: up to 0.1 1.27, 0.2 1.22, 0.3 1.14, 0.5 1.04, 0.8 to 1 0.97, above 4 0.95.  So they, and under
// kPrefillShort tokens, which do not pay for their start-up, the direct loads, are for calls that fill three quarters.
constexpr int kPrefillShort = 512;
__host__ inline PrefillPlan prefill_plan(int kv_dtype, int head_dim, int64_t total_q, int max_q_len, int batch, int heads, int units, int max_context_len)
{
    const auto filled = [&](int blocks, int of) { return total_q * of >= (int64_t)blocks * units * batch; };   // a block's share of 1 / of, on average
    const auto workgroups = [&](int blocks) {   // about: a sequence's last one is half full
        const int64_t n = total_q / (blocks * units) + batch / 2;
        return (n > batch ? n : batch) * heads;
    };
    const auto small_grid = [&](int blocks) { return ((int64_t)max_q_len + blocks * units - 1) / (blocks * units) * batch * heads <= 4096; };
    const bool deep = max_context_len >= 2048;
    if (head_dim == 64) {
        if (kv_dtype == 0 && workgroups(16) >= 2048 && filled(16, 2)) return PrefillPlan{16, 1, false};
        if (kv_dtype == 0) {
            const int line[5][2] = {{96, 192}, {320, 160}, {320, 256}, {640, 320}, {1024, 384}};
            const int *at = line[max_context_len < kPrefillShort ? 0 : max_context_len < 1024 ? 1 : !deep ? 2 : max_context_len < 4096 ? 3 : 4];
            if (workgroups(8) >= at[0] || !small_grid(4)) return PrefillPlan{8, 1, false};
            return workgroups(4) >= at[1] || !small_grid(2) ? PrefillPlan{4, 4, false} : PrefillPlan{2, 8, false};
        }
        if (max_context_len < kPrefillShort || workgroups(8) >= (deep ? 512 : 256) || !small_grid(4)) return PrefillPlan{8, 1, false};
        return workgroups(4) >= (max_context_len >= 4096 ? 384 : deep ? 256 : 128) || !small_grid(2) ? PrefillPlan{4, 4, false} : PrefillPlan{2, 8, false};
    }
    if (kv_dtype == 0) {
        const int depth = max_context_len < kPrefillShort ? 0 : max_context_len < 1024 ? 1 : !deep ? 2 : 3;
        const auto enough = [&](int blocks) {
            const int line[4][3] = {{128, 128, 96}, {144, 144, 96}, {144, 144, 128}, {192, 192, 160}};
            return workgroups(blocks) * 4 >= (int64_t)line[depth][blocks == 16 ? 0 : blocks == 8 ? 1 : 2] * (filled(blocks, 2) ? 4 : 5);
        };
        // A few workgroups of 16 blocks past the 256 that run at once wait for a whole round of them.  Counted no higher than max_q_len allows: the estimate of
        // sequences that fill their blocks is up to 1.5 times their count (101 such calls that it alone puts past the 256 take 0.93 of the time uncut).
        const int64_t w = std::min(workgroups(16), ((int64_t)max_q_len + 16 * units - 1) / (16 * units) * batch * heads);
        const bool just_past = depth == 3 && filled(16, 2) && w > 256 && w < 320;
        const bool full = total_q * 4 >= (int64_t)16 * 3 * units * batch;
        if ((enough(16) && !just_past) || !small_grid(8)) return PrefillPlan{16, 1, full && depth > 0, full && depth == 0};
        if (enough(8) || !small_grid(4)) return PrefillPlan{8, 2, false};
        return enough(4) || !small_grid(2) ? PrefillPlan{4, 4, false} : PrefillPlan{2, 8, false};
    }
    if (max_context_len < kPrefillShort) return PrefillPlan{8, 1, false};
    // (for 8 blocks the cost over all calls is flat between 128 and 192)
    const auto enough = [&](int blocks) { return workgroups(blocks) * 4 >= (blocks == 8 || !filled(blocks, 2) ? 192 : 128) * (deep ? 5 : 4); };
    if (enough(16) || !small_grid(8)) return PrefillPlan{16, 1, false};
    if (enough(8) || !small_grid(4)) return PrefillPlan{8, 2, false};
    // (10 sequences of 480 - 947, 43 - 129 queries, 8/2 heads: 4 blocks 19, 2 blocks 23 us)
    return enough(4) || max_context_len < 1024 || !small_grid(2) ? PrefillPlan{4, 4, false} : PrefillPlan{2, 8, false};
}

// Calls of head_dim 64 over bf16 pools that fill the chip with blocks of 16 take 8 all the same where no sequence may reach 1536 tokens: three workgroups of a compute
// unit fill each other's gaps better than two, and it is for long ranges that a tile's operands are better read once for twice the rows.  16 over 8 blocks, 60
// random calls of 2048 workgroups of 16 blocks and more, run until the chip's clock had settled: under 1024 tokens 1.05, under 1536 1.03, under 2048 1.01, from there on .98, none above
// 1.00.  (In bursts of 10 ms, before it has, 1.13, 1.09, 1.07 and 1.05.)  A grid that a loose bound on the queries leaves mostly empty is not doubled.
__host__ inline PrefillPlan prefill_halved(PrefillPlan plan, int kv_dtype, int head_dim, int64_t total_q, int max_q_len, int batch, int heads, int units, int max_context_len)
{
    const int64_t most = ((int64_t)max_q_len + 8 * units - 1) / (8 * units) * batch * heads, expected = (total_q / (8 * units) + batch / 2) * heads;
    if (kv_dtype == 0 && head_dim == 64 && plan.blocks == 16 && max_context_len < 1536 && most <= 2 * expected) plan.blocks = 8;
    return plan;
}

// Classes of a call's order, 0: dealt pair by pair.  A workgroup finds its block in about 0.8 us (the lengths come from memory, then
// a hundred dependent instructions), so a call whose workgroups all run at once, or of a single sequence, is dealt: six sequences of 800 tokens, 40 queries,
// 8/2 heads, d = 64 7.7 : 8.5 us, dealt : longest first.  So are contexts under 512 tokens, whose time goes into reading queries and writing rows as much as into their
// ranges, and which do better with long and short blocks side by side: nine of 274 - 453, 64/8 heads, whole prompts 65 : 76.  Otherwise:
//   10 of 8 k, 168 - 506 queries, 16/2 heads 401 : 221; 12 fp8 of 2.5 k - 8 k, 700 - 2048 queries, 32/8 1255 : 1204; 8 prompts of 1.5 k - 4 k, d = 64 402 : 399.
// Four or eight classes differ by 0.1 % over 2400 calls; with 32 fewer blocks of a sequence run side by side, which costs large calls a tenth.
// What finding the block costs grows with the rounds of workgroups, what the order can gain with the walk of one of them.  3020 random calls (512 tokens to 16 k,
// 2 to 64 sequences, heads as in perf/cases.py, bf16 and fp8), dealt over longest first, by context / 256 against the rounds, and how many lose and gain more than 8 %:
//                     512 - 767          768 - 1023         1024 - 2047         2048 - 4095         4096 and more
//   no more rounds    1.10 (14, 103)     1.09 (11, 71)      1.10 (23, 187)      1.11 (14, 233)      1.11 (23, 355)
//   more               .97 (32, 3)        .99 (7, 7)        1.00 (1, 4)         1.01 (0, 2)
// (without the calls of the next paragraph)
// From 16 rounds on it is 1.00 at any length (16 of 8192 with 2048 each, 32/8 3257 : 3264 us with four classes, 3287 with eight), and at head_dim 64 under 1024 tokens from one round on.
// In turn over the dies, the blocks of a (sequence, KV head) pair meet on one die only if the heads are a multiple of 8; otherwise several fetch the pair's K/V.  Workgroups of 2
// blocks, 32 rows, over bf16 pools are bound by that where many sequences are walked at once: 24 of 5.7 - 6.4 k, 22 - 58 queries, 8/2 heads fetch 583 MB
// instead of 156 and take 108 instead of 72 us.  1260 such calls, 2 and 4 heads, by sequences: under 12 1.14 (d = 64: 1.07), 12 - 19 .97 (1.00), 20 and more .86
// (.84, down to .53).  Over fp8 pools, half the bytes, they gain: 1.24 and 1.23 with 2 and 4 heads (d = 64 1.19, 1.08).
// (Calls left to the kernel are not asked about here: prefill_slot orders them.)
__host__ inline int prefill_order(const PrefillPlan &plan, int kv_dtype, int head_dim, int64_t total_q, int units, int batch, int heads, int q_blocks, int max_context_len)
{
    if (batch == 1 || batch > kMaxOrderedBatch || max_context_len < kPrefillShort) return 0;
    if (kv_dtype == 0 && plan.blocks == 2 && heads % kXcds != 0 && batch >= 12) return 0;
    // workgroups the chip holds at once (a compute unit one to three: registers, or LDS for the tiles)
    const int slots = 256 * (plan.split == 1 && plan.blocks == 8 ? (head_dim == 64 ? 3 : 2) : head_dim == 64 && plan.blocks != 2 ? 2 : 1);
    const int64_t blocks = total_q / (plan.blocks * units);
    // (dealt pair by pair, dies get alike only if every die gets the same heads)
    if ((int64_t)q_blocks * batch * heads <= slots || (heads % kXcds == 0 && (blocks + batch) * heads <= slots)) return 0;
    const int reach = head_dim == 64 && max_context_len < 1024 ? 256 : std::min(max_context_len, 16 * 256);
    if ((blocks + batch / 2) * heads * 256 > (int64_t)slots * reach) return 0;
    return blocks * heads >= 1536 ? 4 : 8;
}

// 8 or 4 blocks, by the lengths themselves.  The host knows bounds and totals: calls of equal lengths want 8 blocks from 192 workgroups on, ragged ones, whose longest
// range sets the end, many more.  From 1536 tokens on, from 96 workgroups of 8 blocks on and while the grid for 4 is not mostly empty, the kernel
// therefore decides.  Every workgroup estimates both times: a range of `longest` tiles or the chip's share of all tiles, whichever is more, and the share of a last
// round that is not full, the less the more lengths differ; or, if that is more, what the memory takes for the tiles, which are 16 KB each: workgroups
// of a pair find half of what the others of their die fetch in its L2; and a start per round.  (Without the memory, sequences whose queries
// fit one workgroup of 8 blocks and need two of 4 were read twice: 24 of 6.8 - 15.6 k, 15 queries, 64/8 heads 290 us, with it 244.)  us per tile and factors are fitted to 2250
// random calls (2 to 64 sequences, 1.5 k to 16 k tokens, heads as in perf/cases.py), each timed with both sizes.  Against the host's rule, times as fast and calls that gain and lose
// more than 8 %, of 1300 with one to three workgroups of 8 blocks a sequence 1.047, 262 and 5 (without the memory 1.033, 245 and 58), of 1500 with 8 - 2048
// queries 1.023, 214 and 14 (1.022, 219 and 28).  (The better size of each call would give 1.057 and 1.034.)
// 5 sequences of 300 - 6000, 17 - 300 queries, 28/4 heads: 220 workgroups of 8 blocks 81 us, 432 of 4 61.
//
// Deciding costs 1 us, so shorter contexts keep the host's rule (300 calls under 1024 tokens .98), and fewer workgroups (.97), of which none is better with 8.
//
// `s` holds the sequences: longest() in tokens, total(f) = sum of f(queries, tokens), count(tokens, halves) = workgroups of 8 (4, halves = 1) blocks that cover them.
template <class Sequences>
__host__ __device__ inline bool prefill_prefers_four(const Sequences &s, int heads, int tokens)
{
    const float longest = (float)((s.longest() + kTileTokens - 1) / kTileTokens);
    const auto time = [&](int halves, float tile) {
        const int own = tokens >> halves;
        const auto tiles = [&](int nq, int L) { return (L + (L > nq ? L - nq : 0) + (nq < own ? nq : own)) / (2 * kTileTokens); };   // a block's, on average: their ends grow evenly
        const int count = s.total([&](int nq, int) { return s.count(nq, halves); }) * heads;
        const int dies = heads % kXcds == 0 || count <= 256 ? 1 : heads % 4 == 0 ? 2 : heads % 2 == 0 ? 4 : 8;   // over which a pair's blocks spread (prefill_slot)
        const float n = (float)count, walked = (float)s.total([&](int nq, int L) { return s.count(nq, halves) * tiles(nq, L); }) * (float)heads;
        const float fetched = (float)s.total([&](int nq, int L) { const int c = s.count(nq, halves); return (c < dies ? c : dies) * tiles(nq, L); }) * (float)heads;
        const float rounds = n / 256, share = walked / 256, average = walked / (n > 1 ? n : 1), level = average / (longest > 1 ? longest : 1);
        const float last = rounds > 1 ? 0.5f * ((float)(int)(rounds + 0.999f) - rounds) * average * level * level : 0;
        const float compute = tile * ((longest > share ? longest : share) + last), memory = 0.0012f * walked + 0.0008f * fetched;
        return (compute > memory ? compute : memory) + 5 * (rounds > 1 ? rounds : 1);
    };
    return 0.75f * time(0, 0.524f) >= time(1, 0.3f);
}
// Whether the choice is left to the kernel.
__host__ inline bool prefill_on_device(const PrefillPlan &plan, int kv_dtype, int head_dim, int64_t total_q, int max_q_len, int batch, int heads, int units, int max_context_len)
{
    if (kv_dtype != 0 || head_dim != 128 || (plan.blocks != 8 && plan.blocks != 4) || batch == 1 || batch > kMaxOrderedBatch || max_context_len < 1536) return false;
    const int64_t most = ((int64_t)max_q_len + 4 * units - 1) / (4 * units) * batch * heads, expected = (total_q / (4 * units) + batch / 2) * heads;
    return most <= 4096 && most <= 2 * expected + 256 && std::max<int64_t>(total_q / (8 * units) + batch / 2, batch) * heads >= 96;
}

// What runs: the rules above, one after the other.
struct PrefillRoute {
    PrefillPlan plan;
    int tokens;     // query tokens of a workgroup, of 8 blocks where the kernel chooses
    int q_blocks;   // workgroups that cover max_q_len, of 4 blocks where it does
};
__host__ inline PrefillRoute prefill_route(int kv_dtype, int head_dim, int64_t total_q, int max_q_len, int batch, int heads, int units, int max_context_len)
{
    PrefillPlan plan = prefill_plan(kv_dtype, head_dim, total_q, max_q_len, batch, heads, units, max_context_len);
    plan = prefill_halved(plan, kv_dtype, head_dim, total_q, max_q_len, batch, heads, units, max_context_len);
    const int64_t most = std::max<int64_t>(total_q, max_context_len);   // the reciprocal is exact below 2^24
    plan.on_device = most < 1 << 23 && prefill_on_device(plan, kv_dtype, head_dim, total_q, max_q_len, batch, heads, units, max_context_len);
    if (plan.on_device) plan.blocks = 8, plan.split = 2, plan.order = kChosenClasses;
    const int tokens = plan.blocks * units, per_slot = plan.on_device ? tokens / 2 : tokens;
    const int q_blocks = (int)(((int64_t)max_q_len + per_slot - 1) / per_slot);
    if (!plan.on_device && most < 1 << 24) plan.order = prefill_order(plan, kv_dtype, head_dim, total_q, units, batch, heads, q_blocks, max_context_len);
    return PrefillRoute{plan, tokens, q_blocks};
}

// Chunk slots of one output row.  Without a shared prefix, chunk c covers tokens
// [c*chunk, (c+1)*chunk).  With a shared prefix of `sh` tokens (a multiple of
// 16) the first ceil(sh/chunk) slots cover the prefix (the last one may be
// short) and the following ones cover [sh + j*chunk, ...), so that the prefix
// is cut at the same places for every member of a group.
__host__ __device__ inline int shared_slots(int sh, int chunk) { return (sh + chunk - 1) / chunk; }

// Order of the sequences' last (or only) chunks in the split pass: longest first within groups of sequences, for two reasons.  The pass ends when
// its last workgroup does, and long ones that start last leave the chip idle: that takes the batch's last sequences, about two rounds of
// workgroups.  And a die that is dealt whole sequences (fp8; bf16 with fewer than 8 KV heads) gets more tokens than its neighbours,
// unless sequences of like length are dealt in turn: that takes all of them, and costs every workgroup about 1 us, so it is for
// lengths of 2048 and more.  us per step, in batch order : last group only : all groups
//   1024 fp8 sequences of 512 - 4096, 64/8 heads 825 : 817 : 793       800 fp8 of 100 - 8000, 32/4 563 : 537 : 527
//   16 x 16 branches of 64 - 4096, 32/8 458 : 434 : 432                1000 bf16 of 100 - 4000, 16/2 364 : 356 : 350
//   1024 fp8 of 64 - 1024, 64/8 221 : 219 : 228                        600 bf16 of 100 - 2000, 32/8 418 : 409 : 409
// Batches whose workgroups all run at once, or under 1024 tokens (300 us of short workgroups gain nothing), keep their order.
// 150 random decode and prefix calls that are ordered: 1.02 times as fast as in batch order, one loses more than 3 %, 49 gain that much.
constexpr int kMaxOrderedItems = 256;   // sequences whose lengths a wave holds, four to a lane
constexpr int kWorthOrdering = 1024;
struct SplitOrder {
    int group, from;   // sequences of a group; the first sequence that belongs to one (`batch`: none)
};
__host__ inline SplitOrder split_order(int batch, int heads, int longest)   // longest: bound on the tokens of a chunk
{
    const bool deep = longest >= 2048;
    const int round = (deep ? 2048 : 1024) / heads;
    const int group = round < 64 ? 64 : round < kMaxOrderedItems ? round : kMaxOrderedItems;
    if ((int64_t)batch * heads <= 512 || longest < kWorthOrdering) return SplitOrder{group, batch};
    return SplitOrder{group, deep || batch < group ? 0 : batch - group};
}
// Whether a launch writes its finished rows through the L2s.  Few rows are better left in them (4 MB each), from where they reach memory after the
// reads: 16 - 200 sequences of 125 - 1000 tokens, 32/8 heads, up to 3.3 MB of rows lose 2 - 5 % written through, 500 (8.2 MB) +1 %, over fp8 0, 500 of
// 62 - 500 -1 %.  Many are displaced by what is read, one line at a time: 800 of 600 - 4096, 28/4 (11.5 MB) 601 : 586 us, 1000 of 125 - 1000, 32/8
// (16.8 MB) 392 : 382, 1024 fp8 of 512 - 4096, 64/8 (33.5 MB) 780 : 751.
__host__ inline bool stores_through(int64_t bytes) { return bytes >= 10 << 20; }
// Whether its workgroups moreover store in the same windows of the clock.  Memory that reads at its full rate turns around for every few lines that are
// written at any time; rows that all arrive in the same 0.64 of every 6.4 us are written together.  (A read-only walk of 4 GB with 32 MB of
// stores: 604 us without them, 687 plain, 666 written through, 640 and 622 in windows every 20 and 50 us.)  A workgroup waits 3 us for the next window on average,
// which costs nothing as long as the other one of its compute unit reads meanwhile and walks last much longer: us per step without : with windows
//   1024 fp8 of 512 - 4096, 64/8 heads 748 : 726    1024 fp8 of 256 - 2048, 64/8 398 : 381    1024 bf16 of 125 - 1000, 64/8 396 : 378
//   1000 bf16 of 125 - 1000, 32/8 372 : 367         800 bf16 of 512 - 4096, 28/4 578 : 577    1000 bf16 of 62 - 500, 32/8 197 : 199
//   1000 fp8 of 50 - 400, 32/8 100 : 139 if every workgroup waits
//   at head_dim 64, whose compute units hold four workgroups: 1024 fp8 of 512 - 4096, 64/8 398 : 383    800 bf16 of 3000 - 6000, 64/4 566 : 561
//   1024 bf16 of 100 - 1600, 48/16 539 : 543   (15 such calls 1.009 times as fast)
// So the longest sequence may have 384 KB of K/V per head (fp8 of up to 1280 gain 0 - 1 %, bf16 of up to 500 lose as much), and only workgroups that walked 128 KB wait.  Periods of 5 to 13 us and windows of
// a tenth to a quarter of them differ by 1 %.
// The tokens from which on a workgroup waits, 0: no windows.
__host__ inline int window_tokens(int64_t bytes, int longest, int token_bytes)
{
    return stores_through(bytes) && (int64_t)longest * token_bytes >= 384 << 10 ? (128 << 10) / token_bytes : 0;
}
// Workgroups of the split pass that the chip holds at once: a compute unit two at head_dim 128 and four at head_dim 64 (registers, LDS).
__host__ __device__ constexpr int split_round(int head_dim) { return 256 * (head_dim == 64 ? 4 : 2); }

// Arguments of the split-K pass (by value, lives in kernel-argument memory).
struct SplitArgs {
    const uint16_t *q;           // [B][Hq][D] bf16
    const void *k_pages;         // [num_pages][Hkv][16][D]
    const void *v_pages;
    const float *k_scales;       // [num_pages][Hkv] (fp8) or null
    const float *v_scales;
    const int32_t *block_table;  // [B][max_blocks]
    const int32_t *context_lens; // [B]
    float *ws_m;                 // [B][Hq][S]   running max, log2 domain
    float *ws_l;                 // [B][Hq][S]   sum of weights
    float *ws_acc;               // [B][Hq][S][D] weighted V sum
    float *out_direct;           // [B][Hq][D] or null: every sequence is one chunk, write the output instead of partials
    // append and attend in one go (single-chunk mode, bf16 pools; all null otherwise), as in RangeArgs
    const uint16_t *k_new, *v_new;
    uint16_t *k_pages_out, *v_pages_out;
    float scale_log2e;           // scale * log2(e)
    // the shared-prefix items fold a non-negative scale into their exponent: |scale| * log2(e), the sign as a
    // bit flip of the queries (0x80008000 when scale < 0), and zeroed queries with scale 1 when scale == 0
    float abs_scale_log2e;
    uint32_t q_flip, q_keep;
    int32_t B, Hq, Hkv, G;
    int32_t HB;                  // head blocks per KV head: ceil(G / 16)
    int32_t max_blocks, S, chunk_tokens, max_context_len;
    // shared-prefix groups (all zero / null when the call has none)
    const int32_t *group_start;  // [num_groups + 1] first sequence of each group
    const int32_t *shared_len;   // [B] tokens whose pages the sequence shares with its whole group
    int32_t num_groups, group_subs;  // group_subs: workgroups (4 x 16/G sequences each) that cover the largest group
    uint32_t group_items;        // grid entries that serve shared prefixes (they come first)
    int32_t max_shared_len;      // host-known bound on shared_len[]; larger values are clamped to it
    int32_t grid_chunks;         // chunk slots the plain part of the grid spans (S, or S-1 without groups)
    SplitOrder order;            // of the sequences' last chunks
    int32_t store_through;       // finished rows are written through the L2 (stores_through)
    int32_t window_tokens;       // and in windows of the clock by workgroups that walked so many tokens, 0: by none
};

// Hand-over inside a workgroup.  The four waves of a workgroup walk neighbouring pieces (ranges 4i ..
// 4i + 3).  When the LAST segment of a wave's piece began before the piece (then it is the piece's only
// segment and continues the last segment of the wave before), and the wave is not the workgroup's first,
// its result does not go to memory: it is handed through LDS to the wave before, which adds it to its own.
// Such a run of waves leaves one partial (in the slot of its first wave) or, when it holds the whole
// sequence, the finished rows.  Whether range r handed over its part of the sequence whose tiles are
// [o0, o1) of a line of T tiles follows from the geometry alone, so the merge pass needs no marker.
__host__ __device__ inline bool handed_over(int r, int o0, int o1, int T, int per)
{
    const int end = (r + 1) * per < T ? (r + 1) * per : T;
    return r % kWaves != 0 && o0 < r * per && o1 >= end;
}
// The ranges that still hold a part of a sequence spread over ranges r_first .. r_last: r_first, every
// workgroup's first range in between, and r_last unless it handed over.
struct LiveParts {
    int r_first, r_last, first_lead, leads, count;
    __host__ __device__ int range(int i) const { return i == 0 ? r_first : i <= leads ? first_lead + kWaves * (i - 1) : r_last; }
};
__host__ __device__ inline LiveParts live_parts(int o0, int o1, int T, int per)
{
    LiveParts p;
    p.r_first = o0 / per, p.r_last = (o1 - 1) / per;
    p.first_lead = (p.r_first / kWaves + 1) * kWaves;
    p.leads = p.r_last > p.first_lead ? (p.r_last - 1 - p.first_lead) / kWaves + 1 : 0;   // multiples of 4 inside (r_first, r_last)
    p.count = 1 + p.leads + (p.r_last > p.r_first && !handed_over(p.r_last, o0, o1, T, per) ? 1 : 0);
    return p;
}

// Arguments of the range pass (batches without shared prefixes).  Per (virtual) KV head the batch is one line of 32-token tiles (sequence after
// sequence); the line is cut into `ranges` equal ranges and each wave walks one of them.
constexpr int kMaxRangeBatch = 4096;  // sequences whose tile offsets fit the workgroup's LDS
struct RangeArgs {
    const uint16_t *q;
    const void *k_pages, *v_pages;
    const float *k_scales, *v_scales;
    const int32_t *block_table, *context_lens;
    float *out;                  // [B][Hq][D]
    // append and attend in one go (bf16 pools; all null otherwise): row b of k_new / v_new [B][Hkv][D] is the
    // newest token of sequence b, at position context_lens[b] - 1; it is attended from these rows and written
    // into the pool
    const uint16_t *k_new, *v_new;
    uint16_t *k_pages_out, *v_pages_out;
    int32_t *tile_off;           // [B + 1] written for the merge pass: tiles of the sequences before b
    int4 *merge_rec;             // [ranges][Hv] written for the merge pass: {b, tile_off[b], tile_off[b+1], T} of the cut
                                 // sequence whose first part the range holds, or b = -1
    float *ws_m, *ws_l;          // [slots][16]   a wave's partial rows: running max (log2 domain), weight sum
    float *ws_acc;               // [slots][rows_stride][D]   weighted V sums; slot = (range * Hv + head) * 2 + which
    uint32_t *sink;              // probe launches only: one word per wave
    float scale_log2e;           // scale * log2(e)
    int32_t B, Hq, Hkv, G, HB, max_blocks, max_context_len;
    int32_t ranges;              // ranges per virtual head: 4 x (grid / (Hkv * HB))
    int32_t min_tiles;           // a range holds at least this many tiles (unless the batch has fewer)
    int32_t rows_stride;         // rows per partial slot: min(G, 16)
};

struct RangeMergeArgs {
    const int32_t *tile_off;
    const int4 *merge_rec;
    const float *ws_m, *ws_l, *ws_acc;
    float *out;
    int32_t B, Hq, Hkv, G, HB, ranges, min_tiles, rows_stride;
    int32_t by_sequence;         // items are (sequence, head block) instead of (range, head block)
    int32_t groups;              // waves that share the parts of an item (see merge_groups)
};
constexpr int kMergeRows = 4;         // query heads of an item that one workgroup of the merge pass combines
constexpr int kMergeParts = 16;       // parts a wave of it fetches per trip to memory
constexpr int kMaxMergeGroups = 8;    // and the most waves that share the parts of an item
constexpr int kMergeLdsBytes = 64 * (16 + 8);   // LDS of one wave when several do: a lane's sums, a row's maximum and weight sum
// Waves that share the parts of an item.  A sequence leaves at most about one part per workgroup of its head (`rblocks`); one that is
// twice as long as the average 2 * rblocks / batch.  (With room for four times the average 8 sequences of 1 k to 9 k were 2 % slower: a
// barrier for nothing.)
__host__ inline int merge_groups(int rblocks, int batch)
{
    const int64_t parts = (int64_t)2 * rblocks / batch < rblocks ? (int64_t)2 * rblocks / batch : rblocks;
    int groups = 1;
    while (groups < kMaxMergeGroups && groups * kMergeParts < parts) groups *= 2;
    return groups;
}
// Slices of kMergeRows heads of an item that one workgroup of the merge pass takes together: 1, 2 or 4.  Slices of their own spread the parts
// of few items over the chip; where the items alone fill it, they only multiply the workgroups that go through the
// pass's chain of dependent reads.  Merge pass, us with a slice per workgroup : all of them in one:
//   4 slices    256 items   64 sequences, 64/2 heads, d = 128 4.6 : 4.3, the same with one of 24 k tokens 17.6 : 21.8
//               512         128 sequences, 64/4 heads, d = 64 4.8 : 4.2, 64 sequences, 128/4 heads, d = 128 6.6 : 4.7
//              1024         128 sequences, 128/8 heads, d = 64 6.6 : 4.4, with one of 5 k tokens 9.5 : 6.2
//              2048         1373 sequences, one of 4 k and the rest of 67 tokens, 64/4 heads, d = 64 11.3 : 6.4
//   2 slices   1200         300 sequences with one of 5 k tokens, 32/4 heads, d = 64 5.5 : 6.0
//              2048         300 sequences with one of 5 k tokens, 64/8 heads, d = 64 6.2 : 5.1
__host__ inline int merge_width(int64_t items, int rows, int groups)
{
    if (groups > 1 || rows <= kMergeRows) return 1;   // several waves per part share their sums through LDS, a slice at a time
    if (rows <= 2 * kMergeRows) return items >= 2048 ? 2 : 1;
    return items >= 512 ? 4 : 1;
}

struct MergeArgs {
    const float *ws_m, *ws_l, *ws_acc;
    const int32_t *context_lens;
    float *out;                  // [B][Hq][D]
    int32_t B, Hq, S, chunk_tokens, max_context_len;
    const int32_t *shared_len;   // [B] or null, as in SplitArgs
    int32_t max_shared_len;
};

// Arguments of the causal multi-query pass.
struct PrefillArgs {
    const uint16_t *q;           // [total_q][Hq][D] bf16
    const int32_t *q_start;      // [B + 1] first query row of each sequence
    const void *k_pages, *v_pages;
    const float *k_scales, *v_scales;
    const int32_t *block_table, *context_lens;
    float *out;                  // [total_q][Hq][D]
    float scale_log2e;           // |scale| * log2(e); the sign of scale travels in q_flip
    uint32_t q_flip;             // 0x80008000 when scale < 0: every query element changes sign as it is loaded
    uint32_t q_keep;             // 0 when scale == 0 (all scores are zero: zero queries, scale 1), else all ones
    int32_t B, Hq, Hkv, G, HB, max_blocks, max_context_len;  // HB: head blocks per KV head, ceil(G / 16)
    int32_t total_q, max_q_len;  // rows of q; host-known bound on the rows of one sequence
    PrefillPlan plan;
    uint32_t reciprocal;         // of the query tokens of a workgroup (PrefillRoute): 2^32 / tokens, rounded up (plan.order)
    int32_t round_up;            // query tokens of a workgroup - 1
    int32_t q_blocks;            // workgroups that cover max_q_len (PrefillRoute)
};

struct AppendArgs {
    const uint4 *k_new, *v_new;  // [T][Hkv][D] bf16 viewed as 16-byte words
    const int32_t *seq_ids, *positions;   // [T], or both null: row j = sequence j's newest token (see context_lens)
    uint4 *k_pages, *v_pages;
    const int32_t *block_table;
    const int32_t *context_lens;          // used only without index arrays
    int32_t T, Hkv, max_blocks, max_context_len;
};

struct AppendFp8Args {
    const uint4 *k_new, *v_new;  // [T][Hkv][d] bf16 viewed as 16-byte words
    const int32_t *range_seq, *range_start, *range_row0;  // [R], [R], [R+1]
    uint8_t *k_pages, *v_pages;
    float *k_scales, *v_scales;
    const int32_t *block_table;
    int32_t R, Hkv, max_blocks, pages_per_range;
    uint32_t num_tiles;          // 2 * R * pages_per_range * Hkv (K and V tiles)
    int32_t single_rows;         // every range has at most one row (the decode step)
};

struct CopyPagesArgs {
    const int32_t *src_pages, *dst_pages;  // [N]
    uint4 *k_pages, *v_pages;              // pools viewed as 16-byte words
    float *k_scales, *v_scales;            // [num_pages][Hkv] or null
    int32_t N, Hkv, num_pages;
    int32_t page_words;                    // 16-byte words of one page over all heads
};

struct ValidateArgs {
    const int32_t *block_table, *context_lens;
    int32_t *report;             // [2]: bad table entries in use, bad lengths
    int32_t B, max_blocks, num_pages, max_context_len;
};

struct ValidateGroupsArgs {
    const int32_t *block_table, *context_lens, *group_start, *shared_len;
    int32_t *report;             // [4]
    int32_t B, max_blocks, max_context_len, num_groups, max_group_size, max_shared_len;
};

// Launchers: enqueue on `stream`, return the hipError_t of the launch.  When
// `start`/`stop` are given they are bound to the kernel's own begin and end
// timestamps (hipExtLaunchKernelGGL), so their elapsed time is the kernel's
// duration without launch latency.
hipError_t launch_split(const SplitArgs &a, int head_dim, int kv_dtype, hipStream_t stream,
                        hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
hipError_t launch_range(const RangeArgs &a, int head_dim, int kv_dtype, unsigned grid, bool probe, hipStream_t stream,
                        hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
hipError_t launch_range_merge(const RangeMergeArgs &a, int head_dim, hipStream_t stream,
                              hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
hipError_t launch_merge(const MergeArgs &a, int head_dim, hipStream_t stream,
                        hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
hipError_t launch_prefill(const PrefillArgs &a, int head_dim, int kv_dtype, hipStream_t stream,
                          hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
hipError_t launch_append(const AppendArgs &a, int head_dim, hipStream_t stream);
hipError_t launch_append_fp8(const AppendFp8Args &a, int head_dim, hipStream_t stream);
hipError_t launch_copy_pages(const CopyPagesArgs &a, hipStream_t stream);
hipError_t launch_validate(const ValidateArgs &a, hipStream_t stream);
hipError_t launch_validate_groups(const ValidateGroupsArgs &a, hipStream_t stream);

}  // namespace sd
