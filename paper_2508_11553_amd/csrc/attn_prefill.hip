// Causal attention of several query tokens per sequence over the paged cache
// (gfx950, wave64, MFMA): the re-computation of a stretch of a trajectory's own
// stored tokens when it resumes after an interruption.
//
// Sequence b brings n_b = q_start[b+1] - q_start[b] query tokens, its LAST n_b
// positions: query i sits at position pos = L - n_b + i and attends the tokens
// 0 .. pos.  A workgroup owns a block of consecutive query tokens of one
// sequence and one KV head; every wave owns some of them as NB column blocks of
// 16 rows (16 / G tokens times the G query heads of the KV head), which share
// every K operand fetched from LDS and every V^T operand.  The K/V tiles are
// the same for all waves: each is loaded from HBM/L2 once per workgroup, parked
// in LDS as the K image and the ready-made V^T operands, and attended by every
// wave with its own columns.  fp8 codes are converted to bf16 as they are
// parked, once per workgroup, and then take the bf16 pools' tile step (12 sequences of 2.5 k to 8 k tokens, 700 to
// 2048 queries, 32/8 heads: 1.50 -> 1.28 ms against converting K in every consuming wave).
//
// bf16 pools, whose rows need no conversion, have kernels of their own further down for large calls and for split ranges; the general kernel
// serves them where sequences bring few queries (head_dim 128).
//
// The causal limit is a per-lane token bound in the score mask; a wave stops
// once a tile starts at or past the last position any of its rows may see.
//
// Large calls: each wave carries its rows through the whole range with the
// online softmax, so there is no split and no merge.  Small calls, whose query blocks
// would leave compute units idle, take smaller blocks and split their range over the waves of
// the workgroup (prefill_plan): kSplit neighbouring waves own the same rows and
// every kSplit-th tile each, and add up their (max, sum, weighted sum) through LDS at
// the end.  Nothing leaves the workgroup, so no workspace is needed.
#include <cfloat>
#include <type_traits>

#include "attn_tile.h"

namespace sd {

// The sequences of a batch as prefill_pick asks for them, one to a lane.
struct WaveSequences {
    int end, blocks;
    SD_DEV WaveSequences(int end_, int blocks_) : end(end_), blocks(blocks_) {}
    SD_DEV WaveSequences(const PrefillArgs &a, int lane) : end(0), blocks(0)
    {
        int qs = 0, next = 0, L = 0;
        if (lane < a.B) qs = a.q_start[lane], next = a.q_start[lane + 1], L = a.context_lens[lane];
        {
            const int nq = min(next - qs, a.max_q_len);
            L = max(0, min(L, a.max_context_len));
            // rounded up; a.reciprocal = 2^32 / tokens of a workgroup, rounded up: exact below 2^24
            if (lane < a.B && qs >= 0 && nq > 0 && (int64_t)qs + nq <= a.total_q) {
                blocks = (int)__umulhi((unsigned)(nq + a.round_up), a.reciprocal);
                end = (int)__umulhi((unsigned)(L + a.round_up), a.reciprocal);
            }
        }
    }
    SD_DEV int top() const { return wave_max(end); }
    template <class F>
    SD_DEV int sum(F f) const { return __builtin_amdgcn_readlane(wave_scan(f(end, blocks)), 63); }
    struct Found {
        int b, before, end, blocks;
    };
    template <class F>
    SD_DEV Found find(F f, int m) const
    {
        const int own = f(end, blocks), incl = wave_scan(own);
        const int b = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl > m) | 1ull << 63);   // m is less than the sum
        return Found{b, __builtin_amdgcn_readlane(incl - own, b), __builtin_amdgcn_readlane(end, b), __builtin_amdgcn_readlane(blocks, b)};
    }
};

// Their queries and tokens, as prefill_prefers_four asks for them, and the sequences cut into the tokens of a workgroup or (halves = 1) half of them.
struct WaveLengths {
    int nq, L;   // 0 queries: nothing to do
    int round_up;
    uint32_t reciprocal;
    SD_DEV WaveLengths(const PrefillArgs &a, int lane) : nq(0), L(0), round_up(a.round_up), reciprocal(a.reciprocal)
    {
        int qs = 0, next = 0, stored = 0;
        if (lane < a.B) qs = a.q_start[lane], next = a.q_start[lane + 1], stored = a.context_lens[lane];
        const int n = min(next - qs, a.max_q_len);
        if (lane < a.B && qs >= 0 && n > 0 && (int64_t)qs + n <= a.total_q) nq = n, L = max(0, min(stored, a.max_context_len));
    }
    SD_DEV int count(int tokens, int halves) const { return (int)__umulhi((unsigned)((tokens << halves) + round_up), reciprocal); }   // as above
    SD_DEV int longest() const { return wave_max(nq > 0 ? L : 0); }
    template <class F>
    SD_DEV int total(F f) const { return __builtin_amdgcn_readlane(wave_scan(nq > 0 ? f(nq, L) : 0), 63); }
    SD_DEV WaveSequences cut(int halves) const { return nq > 0 ? WaveSequences(count(L, halves), count(nq, halves)) : WaveSequences(0, 0); }
};

// Which query rows a wave owns (everything but `n`-dependent values is wave-uniform).
struct PrefillRows {
    HeadBlock hb;
    int b, qs, nq, L;
    int base;           // position of query 0 (may be negative)
    int kv_end;         // tokens the workgroup's last row sees
    int tpb, iw0;       // query tokens per column block; the wave's first query token
    int max_end;        // its last row's limit
    int min_end;        // its first visible row's limit
    int first_end;      // limit of the last row of its first column block; those of the others lie tpb apart
    bool active;        // some row of the wave sees a token

    // The rows of wave group `group` of `groups` with `blocks` column blocks each; false: the workgroup has nothing to do.
    SD_DEV bool find(const PrefillArgs &a, int groups, int group, int blocks)
    {
        const int Hv = a.Hkv * a.HB;
        tpb = units_per_block(a.G);
        int seq, head, jb;
        if (a.plan.order) {   // head fastest
            const PrefillBlock at = prefill_pick(WaveSequences(a, threadIdx.x & 63), (int)(blockIdx.x / Hv), a.plan.order);
            seq = at.b, head = blockIdx.x % Hv, jb = at.block;
        } else {
            const PrefillItem item = prefill_item(blockIdx.x, a.q_blocks, a.B * Hv);
            seq = item.pair / Hv, head = item.pair % Hv, jb = a.q_blocks - 1 - item.block;
        }
        if (jb < 0) return false;
        return take(a, seq, head, jb, groups, group, blocks);
    }
    // The same, in block jb of a sequence and (virtual) head; tpb is known.
    SD_DEV bool take(const PrefillArgs &a, int seq, int head, int jb, int groups, int group, int blocks)
    {
        const int tpw = blocks * tpb;   // query tokens per wave
        b = seq;
        hb = head_block(head, a.G, a.HB);
        qs = a.q_start[b];
        nq = min(a.q_start[b + 1] - qs, a.max_q_len);
        const int i0 = jb * groups * tpw;
        if (i0 >= nq) return false;
        if (qs < 0 || (int64_t)qs + nq > a.total_q) return false;  // rows outside q: nothing is read or written
        L = max(0, min(a.context_lens[b], a.max_context_len));
        base = L - nq;
        kv_end = max(0, base + min(nq, i0 + groups * tpw));
        iw0 = i0 + group * tpw;
        const int iw1 = min(iw0 + tpw, nq);
        active = iw0 < nq && base + iw1 > 0;
        max_end = base + iw1;
        min_end = max(0, base + iw0) + 1;
        first_end = base + iw0 + tpb;
        return true;
    }
    // row of column block c in this lane (n = lane & 15): query token, whether it exists, whether it sees a token
    // (recomputed where needed rather than kept in registers across the loop)
    SD_DEV int locate(const PrefillArgs &a, int c, int n, bool &in_range, bool &row_ok, int64_t &row) const
    {
        const int i = iw0 + c * tpb + n / hb.rows;
        in_range = n / hb.rows < tpb && i < nq;
        row_ok = in_range && base + i >= 0;
        row = ((int64_t)qs + i) * a.Hq + hb.head0 + n % hb.rows;
        return i;
    }
    // Q^T operands, limits and empty sums of the wave's column blocks.  Rows that see nothing ride along with zero queries, masked
    // only past the sequence's end.  The exponent's reference starts finite: a wave may meet only tokens that a row does not see.
    template <class B, int NB, class State>
    SD_DEV void load(const PrefillArgs &a, int lane, u32x4 (&qop)[NB][B::kDim / 32], int (&row_end)[NB], State (&st)[NB]) const
    {
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            bool in_range, row_ok;
            int64_t row;
            const int i = locate(a, c, lane & 15, in_range, row_ok, row);
            row_end[c] = row_ok ? base + i + 1 : L;
#pragma unroll
            for (int s = 0; s < B::kDim / 32; ++s)
                qop[c][s] = row_ok ? (*reinterpret_cast<const u32x4 *>(a.q + row * B::kDim + B::q_offset(s, lane)) & a.q_keep) ^ a.q_flip
                                   : u32x4{0, 0, 0, 0};
            reset(st[c]);
            st[c].m = -FLT_MAX;
        }
    }
};

// The parts of a group's rows, added in order: kSplit waves left maxima and weight sums in ms and ls, and their rows where image(row, 16-byte
// word) finds them; every wave finishes its share.
template <int D, int NB, int kSplit, class Image>
SD_DEV void add_parts(const PrefillArgs &a, const PrefillRows &rows, int group, int part, int lane, const float *ms, const float *ls, Image image)
{
    constexpr int kRowWords = D / 4;
    for (int idx = part * 64 + lane; idx < NB * 16 * kRowWords; idx += kSplit * 64) {
        const int rr = idx / kRowWords, word = idx % kRowWords;
        const int c = rr >> 4, rn = rr & 15;
        bool in_range, row_ok;
        int64_t row;
        rows.locate(a, c, rn, in_range, row_ok, row);
        if (!in_range) continue;
        float M = -FLT_MAX, den = 0.f;
        f32x4 num = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < kSplit; ++s) M = max_of(M, ms[(group * kSplit + s) * NB * 16 + rr]);
#pragma unroll
        for (int s = 0; s < kSplit; ++s) {
            const int at = (group * kSplit + s) * NB * 16 + rr;
            const float w = __builtin_amdgcn_exp2f(ms[at] - M);
            den += w * ls[at];
            num += w * image(at, word);
        }
        *reinterpret_cast<f32x4 *>(a.out + row * D + word * 4) = row_ok ? num / den : f32x4{0, 0, 0, 0};
    }
}

template <class P, int kW, int NB>
struct PrefillLds {
    static constexpr int kImage = P::kDim + 4;   // floats of a row of a wave's result, padded against bank conflicts
    static constexpr int kMerge = kW * NB * 16 * (kImage + 2) * 4;
};

// A round is kTiles tiles of 32 tokens, held in one of two LDS buffers; a wave brings 2 * kTiles / kW pages of
// it, and because the next round's buffer is the one nobody reads, it parks what it loaded and asks for
// the pages after that without waiting for anybody: one barrier per round, none between a write
// and the reads of the same round.
//
// kSplit == kW (all waves own the same rows) needs no sharing: every wave brings whole tiles into a slot of
// its own and attends them, without any barrier until the results are added up.
template <class P, int kW, int kTiles, int kSplit, int NB, int kWavesPerSimd>
__global__ __launch_bounds__(kW * 64, kWavesPerSimd) void prefill_wide_kernel(PrefillArgs a)
{
    constexpr int D = P::kDim;
    constexpr bool kOwn = kSplit == kW;
    constexpr int kGroups = kW / kSplit;                  // waves with rows of their own
    constexpr int kPages = kOwn ? 2 : 2 * kTiles / kW;    // pages a wave brings per round
    constexpr int kSlot = P::kParkedBytes;
    constexpr int kBuf = kTiles * kSlot;
    constexpr int kTilesBytes = kOwn ? kBuf : 2 * kBuf;
    constexpr int kMergeBytes = kSplit > 1 ? PrefillLds<P, kW, NB>::kMerge : 0;
    static_assert(kOwn ? kTiles == kW : kPages * kW == 2 * kTiles && kTiles % kSplit == 0, "whole pages per wave, whole tiles per split");
    __shared__ __attribute__((aligned(16))) char lds[kTilesBytes > kMergeBytes ? kTilesBytes : kMergeBytes];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = wave / kSplit, part = wave % kSplit;
    PrefillRows rows;
    if (!rows.find(a, kGroups, group, NB)) return;
    const int g = rows.hb.g, L = rows.L;
    const int n = lane & 15;
    int row_end[NB];
    u32x4 qop[NB][D / 32];
    typename P::B::ParkedState st[NB];
    rows.load<typename P::B>(a, lane, qop, row_end, st);

    const int32_t *bt = a.block_table + (int64_t)rows.b * a.max_blocks;
    const int64_t page_bytes = (int64_t)P::kTileBytes * a.Hkv;
    const char *kbase = static_cast<const char *>(a.k_pages) + g * P::kTileBytes;
    const char *vbase = static_cast<const char *>(a.v_pages) + g * P::kTileBytes;
    typedef typename P::Page Page;
    auto issue = [&](Page &r, int page) {
        P::template load_one<false>(r, kbase + page * page_bytes, vbase + page * page_bytes, a.k_scales, a.v_scales,
                                    (int64_t)page * a.Hkv + g, lane);
    };
    // the wave's rows over the parked tile `tile`
    auto step = [&](const char *slot, int tile, auto masked) {
        u32x4 ka[D / 32], kb[D / 32];
        P::B::k_fetch(slot, lane, ka, kb);
        P::B::template attend_parked<NB, decltype(masked)::value, P::kScaled>(ka, kb, slot + P::kImageBytes, qop, st, a.scale_log2e,
                                                                             tile * kTileTokens, lane, row_end, true,
                                                                             slot + P::B::kParkedBytes, rows.first_end, rows.tpb);
    };
    const int ntiles = (rows.kv_end + kTileTokens - 1) / kTileTokens;
    const int last_page = (rows.kv_end + kPage - 1) / kPage - 1;

    if constexpr (kOwn) {
        // tiles wave, wave + kW, ...: those below `plain` end at or before the first visible row's limit
        const int count = ntiles > wave ? (ntiles - wave + kW - 1) / kW : 0;
        const int plain = rows.min_end / kTileTokens;
        char *mine = lds + wave * kSlot;
        if (count > 0) {
            Page r[2];
            auto tile_of = [&](int i) { return wave + kW * min(i, count - 1); };
            auto page_of = [&](int i, int h) { return bt[min(2 * tile_of(i) + h, last_page)]; };
            int next[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                issue(r[h], page_of(0, h));
                next[h] = page_of(1, h);
            }
            auto turn = [&](int i, auto masked) {
                const int tile = tile_of(i);
#pragma unroll
                for (int h = 0; h < 2; ++h) P::park_one(r[h], mine, h, lane, tile * kTileTokens + h * kPage, L);
#pragma unroll
                for (int h = 0; h < 2; ++h) {   // past the end the last tile is asked for again; nobody attends it
                    issue(r[h], next[h]);
                    next[h] = page_of(i + 2, h);
                }
                wave_lds_fence();
                step(mine, tile, masked);
                wave_lds_fence();
            };
            const int count_plain = min(count, plain > wave ? (plain - wave + kW - 1) / kW : 0);
            int i = 0;
#pragma unroll 1
            for (; i < count_plain; ++i) turn(i, std::false_type{});
#pragma unroll 1
            for (; i < count; ++i) turn(i, std::true_type{});
        }
    } else {
        // page i of this wave: tile and half of the round it belongs to
        auto tile_of = [&](int i) { return (wave * kPages + i) >> 1; };
        auto half_of = [&](int i) { return (wave * kPages + i) & 1; };
        // page i of round rd -> its half of its tile's slot in `buf`
        auto park = [&](Page &r, char *buf, int rd, int i) {
            const int my_tile = tile_of(i), my_page = half_of(i);
            P::park_one(r, buf + my_tile * kSlot, my_page, lane, (kTiles * rd + my_tile) * kTileTokens + my_page * kPage, L);
        };
        const int rounds = (ntiles + kTiles - 1) / kTiles;
        // page i this wave brings for round rd (pages past the end re-read the last one; nobody attends them)
        auto page_of = [&](int rd, int i) { return bt[min(2 * kTiles * min(rd, rounds - 1) + wave * kPages + i, last_page)]; };
        if (rounds > 0) {
            Page r[kPages];
            int next_page[kPages], after_next[kPages];  // read ahead of their use
#pragma unroll
            for (int i = 0; i < kPages; ++i) {
                issue(r[i], page_of(0, i));
                next_page[i] = page_of(1, i);
                after_next[i] = page_of(2, i);
            }
#pragma unroll
            for (int i = 0; i < kPages; ++i) {
                park(r[i], lds, 0, i);
                if (rounds > 1) issue(r[i], next_page[i]);
            }
            __syncthreads();
            for (int rd = 0; rd < rounds; ++rd) {
                const char *cur = lds + (rd & 1) * kBuf;
                // round rd + 1's page goes to the other buffer (last read in round rd - 1), round rd + 2's is requested
#pragma unroll
                for (int i = 0; i < kPages; ++i) {
                    next_page[i] = after_next[i];
                    after_next[i] = page_of(rd + 3, i);
                    if (rd + 1 < rounds) {
                        park(r[i], lds + ((rd + 1) & 1) * kBuf, rd + 1, i);
                        if (rd + 2 < rounds) issue(r[i], next_page[i]);
                    }
                }
                if (rows.active) {
                    // the round's tiles below the diagonal of every row of the wave, then those on it
                    const int t0 = kTiles * rd * kTileTokens;
                    const int j_end = min(kTiles, (rows.max_end - t0 + kTileTokens - 1) / kTileTokens);
                    const int j_plain = max(0, min(j_end, (rows.min_end - t0) / kTileTokens));
                    int j = part;
#pragma unroll 1
                    for (; j < j_plain; j += kSplit) step(cur + j * kSlot, kTiles * rd + j, std::false_type{});
#pragma unroll 1
                    for (; j < j_end; j += kSplit) step(cur + j * kSlot, kTiles * rd + j, std::true_type{});
                }
                __syncthreads();
            }
        }
    }

    auto weight_sum = [&](int c) { return P::kScaled ? P::B::scaled_weight_sum(st[c]) : P::B::weight_sum(st[c]); };
    if constexpr (kSplit == 1) {
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const float l = weight_sum(c);
            bool in_range, row_ok;
            int64_t row;
            rows.locate(a, c, n, in_range, row_ok, row);
            if (!in_range) continue;
            const float inv = row_ok ? 1.0f / l : 0.0f;  // rows before the sequence's first token get zeros
#pragma unroll
            for (int k = 0; k < D / 16; ++k) st[c].acc[k] = row_ok ? st[c].acc[k] * inv : f32x4{0, 0, 0, 0};
            P::store_acc(st[c], a.out + row * D, lane >> 4);
        }
    } else {
        // The results of the kSplit waves of a group, through LDS: rows [wave][block][16][D], then maxima and weight sums.
        constexpr int kImage = PrefillLds<P, kW, NB>::kImage;
        float *image = reinterpret_cast<float *>(lds);
        float *ms = image + kW * NB * 16 * kImage, *ls = ms + kW * NB * 16;
        __syncthreads();   // the tiles are no longer needed
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            P::store_acc(st[c], image + ((wave * NB + c) * 16 + n) * kImage, lane >> 4);
            if (lane < 16) {
                ms[(wave * NB + c) * 16 + n] = st[c].m;
                ls[(wave * NB + c) * 16 + n] = weight_sum(c);
            }
        }
        __syncthreads();
        add_parts<D, NB, kSplit>(a, rows, group, part, lane, ms, ls, [&](int at, int word) { return *reinterpret_cast<const f32x4 *>(image + at * kImage + word * 4); });
    }
}

// ---------------------------------------------------------------------------
// bf16 pools, large calls and split ranges.  K and V rows go from memory straight into LDS, without passing through registers: a tile's
// slot holds K of its two pages and V of its two pages as rows, and the V^T operands are formed by
// transposing LDS reads.  That leaves the registers and the vector instructions of parking (a fifth of the tile step's) to
// the tile step.  A row's 16-byte pieces are permuted as they are loaded, so that the reads spread over all banks:
// K piece c of row r sits at c ^ r (as in k_store), V's 32-byte units at unit ^ row.
//
// The slots are separate arrays, and the loops are written out over them: reads of one array do not wait for loads
// into another only where the compiler can tell the two apart.
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 *LdsVector;
typedef __attribute__((address_space(3))) s16x4 *LdsTransposed;

// 16 bytes per lane from global memory straight into LDS: lane l's, at byte `offset` of the `bytes` at `src` (wave-uniform), land
// at dst + 16 * l.
SD_DEV void load_to_lds(const char *src, int bytes, int offset, char *dst)
{
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(src), 0, bytes, 0x00027000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)dst, 16, offset, 0, 0, 0);
}
// Waits for all but the newest N loads into LDS of this wave; for its LDS reads and writes.  (s_waitcnt: vmcnt in bits 0-3 and 14-15, expcnt
// in 4-6, lgkmcnt in 8-11.)
template <int N>
SD_DEV void wait_loads()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0f70);
    asm volatile("" ::: "memory");
}
SD_DEV void wait_lds()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
}
// A bare barrier: what must have arrived is waited for by name, loads under way stay under way.
SD_DEV void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// What one wave brings of every slot, and where the operands of a slot lie for a lane.
template <int D>
struct RowSlot {
    static constexpr int kPageBytes = Bf16Path<D>::kTileBytes;   // K or V of one page and head
    static constexpr int kBytes = 4 * kPageBytes;                // K of pages 0 and 1, V of pages 0 and 1
    static constexpr int kRowBytes = D * 2, kPieces = D / 8;
    SD_DEV static int v_unit(int row) { return D == 128 ? row & 7 : row >> 1 & 3; }
    // byte of a K (kind 0) or V (kind 1) page that belongs at byte `at` of its image
    SD_DEV static int source(int kind, int at)
    {
        const int row = at / kRowBytes, piece = at % kRowBytes / 16;
        return row * kRowBytes + (piece ^ (kind ? v_unit(row) << 1 : row % kPieces)) * 16;
    }
    // K row lane & 15, d = 32 s + 8 (lane >> 4) .. +8, of the slot's first page (the second kPageBytes on)
    SD_DEV static int k_at(int s, int lane) { return (lane & 15) * kRowBytes + ((4 * s + (lane >> 4)) ^ (lane % 16 % kPieces)) * 16; }
    // V^T operand k, first page: the transposing read gives this lane column 16 k + (lane & 15) of rows 4 (lane >> 4) .. +3
    SD_DEV static int v_at(int k, int lane)
    {
        const int row = 4 * (lane >> 4) + ((lane >> 2) & 3);
        return 2 * kPageBytes + row * kRowBytes + 8 * (lane & 3) + ((k ^ v_unit(row)) << 5);
    }
    // `at` is one offset from an array: with more address arithmetic the compiler loses track of which array it is
    SD_DEV static void fetch_k(const char *buf, int offset, int lane, u32x4 (&ka)[D / 32], u32x4 (&kb)[D / 32])
    {
#pragma unroll
        for (int s = 0; s < D / 32; ++s) {
            const int at = offset + k_at(s, lane);
            ka[s] = *(LdsVector)(buf + at);
            kb[s] = *(LdsVector)(buf + (at + kPageBytes));
        }
    }
    SD_DEV static u32x4 v_operand(const char *buf, int offset, int k, int lane)
    {
        const int at = offset + v_at(k, lane);
        const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTransposed)(buf + at)));
        const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTransposed)(buf + (at + kPageBytes))));
        return u32x4{x[0], x[1], y[0], y[1]};
    }
    // acc[k][r] = O[row lane & 15][d = 16 k + 4 (lane >> 4) + r]
    template <class State>
    SD_DEV static void store(const State &st, float *dst, int lane, bool row_ok, float l)
    {
        const float inv = 1.0f / l;
#pragma unroll
        for (int k = 0; k < D / 16; ++k)   // rows before the sequence's first token get zeros
            *reinterpret_cast<f32x4 *>(dst + 16 * k + 4 * (lane >> 4)) = row_ok ? st.acc[k] * inv : f32x4{0, 0, 0, 0};
    }
};

// What the kernels below bring of a sequence and KV head: pages of K or V straight into LDS.
template <int D>
struct PageRows {
    typedef RowSlot<D> Slot;
    static constexpr int kLoads = Slot::kPageBytes / 1024;   // of a K or V page
    ConstTable table;
    const char *kbase, *vbase;
    int64_t page_bytes;
    int ntiles, last_page, L, lane;
    SD_DEV PageRows(const PrefillArgs &a, const PrefillRows &rows, int lane_)
        : table((ConstTable)(a.block_table + (int64_t)rows.b * a.max_blocks)), kbase(static_cast<const char *>(a.k_pages) + rows.hb.g * Slot::kPageBytes),
          vbase(static_cast<const char *>(a.v_pages) + rows.hb.g * Slot::kPageBytes), page_bytes((int64_t)Slot::kPageBytes * a.Hkv),
          ntiles((rows.kv_end + kTileTokens - 1) / kTileTokens), last_page((rows.kv_end + kPage - 1) / kPage - 1), L(rows.L), lane(lane_) {}
    // past the end the last page once more; nobody attends it
    SD_DEV int id(int tile, int half) const { return table[min(2 * tile + half, last_page)]; }
    // loads first .. first + loads of K (kind 0) or V of one page, whose image begins at buf + at
    SD_DEV void bring(int kind, int page, char *buf, int at, int first = 0, int loads = kLoads) const
    {
        const char *src = (kind ? vbase : kbase) + page * page_bytes;
#pragma unroll
        for (int j = first; j < first + loads; ++j) load_to_lds(src, Slot::kPageBytes, Slot::source(kind, j * 1024 + lane * 16), buf + (at + j * 1024));
    }
    // V rows of tokens that do not exist may hold anything: zeros
    SD_DEV void clean(char *buf, int at, int tok0) const
    {
        if (tok0 + kPage <= L) return;
#pragma unroll
        for (int j = 0; j < kLoads; ++j)
            if (tok0 + (j * 1024 + lane * 16) / Slot::kRowBytes >= L) *reinterpret_cast<u32x4 *>(buf + (at + j * 1024 + lane * 16)) = u32x4{0, 0, 0, 0};
    }
};

// The rows a wave leaves in LDS for add_parts, the 16-byte words of row r permuted by r.
template <class P, int NB>
struct PartImage {
    static constexpr int kBytes = NB * 16 * P::kDim * 4;
    SD_DEV static f32x4 *word(char *wave_image, int row, int word) { return reinterpret_cast<f32x4 *>(wave_image + row * (P::kDim * 4) + (word ^ (row & 15)) * 16); }
};
// Accumulators as RowSlot's operands leave them -> finished rows; wave w's image is image_of(w), where tiles were.
template <class P, int NB, int kSplit, class ImageOf>
SD_DEV void leave_parts(const PrefillArgs &a, const PrefillRows &rows, typename P::ParkedState (&st)[NB], int wave, int lane, float *ms, float *ls, ImageOf image_of)
{
    constexpr int D = P::kDim;
    __syncthreads();   // the tiles are no longer needed
    char *mine = image_of(wave);
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        const int row = c * 16 + (lane & 15);
#pragma unroll
        for (int k = 0; k < D / 16; ++k) *PartImage<P, NB>::word(mine, row, 4 * k + (lane >> 4)) = st[c].acc[k];
        if (lane < 16) {
            ms[wave * NB * 16 + row] = st[c].m;
            ls[wave * NB * 16 + row] = P::weight_sum(st[c]);
        }
    }
    __syncthreads();
    add_parts<D, NB, kSplit>(a, rows, wave / kSplit, wave % kSplit, lane, ms, ls,
                             [&](int at, int word) { return *PartImage<P, NB>::word(image_of(at / (NB * 16)), at % (NB * 16), word); });
}

// Calls over bf16 pools that do not fill the chip with blocks of 16 (head_dim 128): 8 waves of two column blocks each, kSplit waves own the
// same rows and every kSplit-th tile; a round is kSplit tiles, a tile step per wave.
//
// What bounds it is how a round's parts line up: with one step per wave between barriers nothing covers the time a wave spends on its own loads.
// The kernel that parks through registers took 3300 cycles a round with kSplit = 4: a step of 1150, then 1150 in which 64 KB of K images and V^T operands
// were written to LDS and 400 - 700 in which 96 load instructions (V in 8-byte pieces) went through the address unit.  Loads straight into LDS
// need no writes and 64 instructions; issued in one go at the start of the round they still hold up the wave's step (2900 cycles), so half of them
// follow the K operands and half the V^T operands (2350).
// (Cycles by time stamps, from builds that wrote them out.)
// One sequence of 8192, 512 queries, 32/8 heads (kSplit 4): 98 -> 78 us; five sequences of 300 - 6000, 17 - 300 queries, 28/4
// heads, cut to 4 blocks: 75 -> 60 us; 1740 random calls with kSplit 2: 0.91 of the time.
// kSplit 0: the size of the workgroups is chosen here, from the lengths (prefill_prefers_four).  (A kernel of 4 blocks alone is 0.3 us faster in calls of 15 us.)
template <int kSplit>
__global__ __launch_bounds__(512, 2) void prefill_wide_kernel_direct(PrefillArgs a)
{
    constexpr int D = 128, NB = 2, kW = 8, S = D / 32;
    typedef Bf16Path<D> P;
    typedef RowSlot<D> Slot;
    // Two tiles to an array; where workgroups only ever have 4 blocks, the tiles of both sides (below) share one, which halves the code (small
    // calls, which fetch it as they start, 0.3 us).
    constexpr int kBuf = (kSplit == 4 ? 4 : 2) * Slot::kBytes, kMore = kSplit == 4 ? 16 : kBuf;
    __shared__ __attribute__((aligned(16))) char buf0[kBuf], buf1[kBuf], buf2[kMore], buf3[kMore];
    __shared__ float ms[kW * NB * 16], ls[kW * NB * 16];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // 8 blocks: four groups of two waves; 4 blocks: waves 0, 1, 4, 5 and 2, 3, 6, 7
    const int group_of_eight = wave >> 1, group_of_four = wave >> 1 & 1;
    bool four = kSplit == 4;
    PrefillRows rows;
    if constexpr (kSplit == 0) {
        const int Hv = a.Hkv * a.HB;
        const WaveLengths lengths(a, lane);
        four = prefill_prefers_four(lengths, Hv, a.round_up + 1);
        const PrefillSlot at = prefill_slot(lengths.cut(four), blockIdx.x, Hv);
        if (at.block < 0) return;
        rows.tpb = units_per_block(a.G);
        if (!rows.take(a, at.b, at.head, at.block, four ? 2 : 4, four ? group_of_four : group_of_eight, NB)) return;
    } else {
        if (!rows.find(a, kW / kSplit, four ? group_of_four : group_of_eight, NB)) return;
    }
    int row_end[NB];
    u32x4 qop[NB][S];
    typename P::ParkedState st[NB];
    rows.load<P>(a, lane, qop, row_end, st);

    const PageRows<D> pages(a, rows, lane);
    constexpr int kLoads = PageRows<D>::kLoads;
    const int part = wave & 1;   // the tile of a pair that this wave attends
    // The step over tile first + part, whose rows lie at buf + at; the V^T operands are followed by behind().
    auto step = [&](const char *buf, int at, const u32x4 (&ka)[S], const u32x4 (&kb)[S], int first, auto behind) {
        auto attend = [&](int tile, auto masked) {
            P::template attend_fetched<NB, decltype(masked)::value, false>(
                ka, kb, [&](int k) {
                    const u32x4 v = Slot::v_operand(buf, at, k, lane);
                    if (k == D / 16 - 1) {
                        __builtin_amdgcn_sched_barrier(0);
                        behind();
                    }
                    return v;
                }, qop, st, a.scale_log2e, tile * kTileTokens, lane, row_end, true, nullptr, rows.first_end, rows.tpb);
        };
        // (Loops of one turn or none: of two branches the compiler joins what they have in common ahead of them, the operands' reads above all, and spills.)
        const int t0 = first * kTileTokens;
        const int j_end = rows.active ? min(2, (rows.max_end - t0 + kTileTokens - 1) / kTileTokens) : 0;
        const int j_plain = max(0, min(j_end, (rows.min_end - t0) / kTileTokens));
        int j = part;
#pragma unroll 1
        for (; j < j_plain; j += 2) attend(first + j, std::false_type{});
#pragma unroll 1
        for (; j < j_end; j += 2) attend(first + j, std::true_type{});
        if (part >= j_end) behind();
    };
    auto image_of = [&](int w) {
        constexpr int kPer = kBuf / PartImage<P, NB>::kBytes;
        const int b = w / kPer;
        return (b == 0 ? buf0 : b == 1 ? buf1 : b == 2 ? buf2 : buf3) + w % kPer * PartImage<P, NB>::kBytes;
    };

    // A round is two tiles in one of the four arrays, asked for three rounds ahead; a wave brings half of a tile's K or V.
    auto eight = [&] {
        const int rounds = (pages.ntiles + 1) / 2;
        const int my_tile = wave >> 2, my_page = wave >> 1 & 1, my_kind = wave & 1;
        const int my_at = my_tile * Slot::kBytes + my_page * Slot::kPageBytes;
        auto page_of = [&](int rd) { return pages.id(2 * min(rd, rounds - 1) + my_tile, my_page); };
        auto bring_half = [&](int half, char *buf, int page) {
            pages.bring(my_kind, page, buf, my_at + my_kind * 2 * Slot::kPageBytes, half * kLoads / 2, kLoads / 2);
        };
        auto bring_round = [&](char *buf, int page) { bring_half(0, buf, page); bring_half(1, buf, page); };
        auto clean = [&](char *buf, int rd) {
            if (my_kind) pages.clean(buf, my_at + 2 * Slot::kPageBytes, (2 * rd + my_tile) * kTileTokens + my_page * kPage);
        };
        auto turn = [&](int rd, char *cur, char *next, char *fill, int page) {
            u32x4 ka[S], kb[S];
            Slot::fetch_k(cur, part * Slot::kBytes, lane, ka, kb);
            __builtin_amdgcn_sched_barrier(0);
            bring_half(0, fill, page);
            step(cur, part * Slot::kBytes, ka, kb, 2 * rd, [&] { bring_half(1, fill, page); });
            wait_loads<2 * kLoads>();   // round rd + 1 has arrived
            clean(next, rd + 1);
            wait_lds();
            phase_barrier();
        };
        if (rounds > 0) {
            bring_round(buf0, page_of(0));
            bring_round(buf1, page_of(1));
            bring_round(buf2, page_of(2));
            int page = page_of(3);
            wait_loads<2 * kLoads>();
            clean(buf0, 0);
            wait_lds();
            phase_barrier();
            for (int rd = 0;;) {
                { const int after = page_of(rd + 4); turn(rd, buf0, buf1, buf3, page); page = after; }
                if (++rd == rounds) break;
                { const int after = page_of(rd + 4); turn(rd, buf1, buf2, buf0, page); page = after; }
                if (++rd == rounds) break;
                { const int after = page_of(rd + 4); turn(rd, buf2, buf3, buf1, page); page = after; }
                if (++rd == rounds) break;
                { const int after = page_of(rd + 4); turn(rd, buf3, buf0, buf2, page); page = after; }
                if (++rd == rounds) break;
            }
            wait_loads<0>();   // no load may land in what follows
        }
        leave_parts<P, NB, 2>(a, rows, st, wave, lane, ms, ls, image_of);
    };
    // Waves 0 - 3 take tiles 0, 1, 4, 5, ... through two of the arrays, waves 4 - 7 tiles 2, 3, 6, 7, ... through the others; a wave brings K and V of one
    // page per round, a round ahead.
    auto by_four = [&] {
        const int rounds = (pages.ntiles + 3) / 4;
        const int side = wave >> 2, my_tile = wave >> 1 & 1, my_page = wave & 1;
        const int side_at = kSplit == 4 ? side * 2 * Slot::kBytes : 0, my_at = side_at + my_tile * Slot::kBytes + my_page * Slot::kPageBytes;
        auto page_of = [&](int rd) { return pages.id(4 * min(rd, rounds - 1) + 2 * side + my_tile, my_page); };
        auto bring_half = [&](int half, char *buf, int page) { pages.bring(half, page, buf, my_at + half * 2 * Slot::kPageBytes); };   // K, V
        auto clean = [&](char *buf, int rd) {
            pages.clean(buf, my_at + 2 * Slot::kPageBytes, (4 * rd + 2 * side + my_tile) * kTileTokens + my_page * kPage);
        };
        auto turn = [&](int rd, char *cur, char *next, int page) {
            u32x4 ka[S], kb[S];
            Slot::fetch_k(cur, side_at + part * Slot::kBytes, lane, ka, kb);
            __builtin_amdgcn_sched_barrier(0);
            bring_half(0, next, page);
            step(cur, side_at + part * Slot::kBytes, ka, kb, 4 * rd + 2 * side, [&] { bring_half(1, next, page); });
            wait_loads<0>();   // round rd + 1 has arrived
            clean(next, rd + 1);
            wait_lds();
            phase_barrier();
        };
        auto walk = [&](char *even, char *odd) {
            bring_half(0, even, page_of(0));
            bring_half(1, even, page_of(0));
            int page = page_of(1);
            wait_loads<0>();
            clean(even, 0);
            wait_lds();
            phase_barrier();
            for (int rd = 0;;) {
                { const int after = page_of(rd + 2); turn(rd, even, odd, page); page = after; }
                if (++rd == rounds) break;
                { const int after = page_of(rd + 2); turn(rd, odd, even, page); page = after; }
                if (++rd == rounds) break;
            }
        };
        if (rounds > 0) {
            if (kSplit == 4 || side == 0)
                walk(buf0, buf1);
            else
                walk(buf2, buf3);
        }
        leave_parts<P, NB, 4>(a, rows, st, 4 * group_of_four + 2 * side + part, lane, ms, ls, image_of);
    };
    if constexpr (kSplit == 2)
        eight();
    else if constexpr (kSplit == 4)
        by_four();
    else if (four)
        by_four();
    else
        eight();
}

// All waves own the same rows and every wave loads tiles of its own: nobody waits for anybody.  K of the next tile is asked for as soon as the operands of this
// one are in registers, and V likewise, so one tile's room per wave is enough.  head_dim 128: the compute unit takes 128 KB in 2500 cycles, 0.8 of the 64
// bytes a cycle its L1 delivers.  One sequence of 8192, 64 queries, 32/8 heads 61 -> 40 us against parking through registers; head_dim 64 (two
// workgroups per compute unit): one of 8192, 512 queries 74 -> 51, 64 queries over 16384 64 -> 53; 24 random calls 1.03 times as fast, one 7 % slower.
template <int D, int kW, int NB>
__global__ __launch_bounds__(kW * 64, 2) void prefill_wide_kernel_own(PrefillArgs a)
{
    constexpr int S = D / 32;
    typedef Bf16Path<D> P;
    typedef RowSlot<D> Slot;
    constexpr int kHalf = 2 * Slot::kPageBytes, kImages = kW / 2 * PartImage<P, NB>::kBytes;
    constexpr int kBuf = kW * kHalf > kImages ? kW * kHalf : kImages;
    __shared__ __attribute__((aligned(16))) char kbuf[kBuf], vbuf[kBuf];
    __shared__ float ms[kW * NB * 16], ls[kW * NB * 16];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    PrefillRows rows;
    if (!rows.find(a, 1, 0, NB)) return;
    int row_end[NB];
    u32x4 qop[NB][S];
    typename P::ParkedState st[NB];
    rows.load<P>(a, lane, qop, row_end, st);

    const PageRows<D> pages(a, rows, lane);
    constexpr int kLoads = PageRows<D>::kLoads;
    auto attend = [&](const u32x4 (&ka)[S], const u32x4 (&kb)[S], auto v_of, int tile, auto masked) {
        P::template attend_fetched<NB, decltype(masked)::value, false>(ka, kb, v_of, qop, st, a.scale_log2e, tile * kTileTokens, lane, row_end, true,
                                                                      nullptr, rows.first_end, rows.tpb);
    };
    const int count = pages.ntiles > wave ? (pages.ntiles - wave + kW - 1) / kW : 0;
    if (count > 0) {
        const int at = wave * kHalf;
        auto tile_of = [&](int i) { return wave + kW * min(i, count - 1); };
        auto page_of = [&](int i, int h) { return pages.id(tile_of(i), h); };
        int next[2] = {page_of(1, 0), page_of(1, 1)};
#pragma unroll
        for (int h = 0; h < 2; ++h) pages.bring(0, page_of(0, h), kbuf, at + h * Slot::kPageBytes);
#pragma unroll
        for (int h = 0; h < 2; ++h) pages.bring(1, page_of(0, h), vbuf, at + h * Slot::kPageBytes);
        auto turn = [&](int i, auto masked) {
            const int tile = tile_of(i);
            u32x4 ka[S], kb[S];
            wait_loads<2 * kLoads>();   // K is there
            Slot::fetch_k(kbuf, at, lane, ka, kb);
            wait_lds();
            const int after[2] = {page_of(i + 2, 0), page_of(i + 2, 1)};
#pragma unroll
            for (int h = 0; h < 2; ++h) pages.bring(0, next[h], kbuf, at + h * Slot::kPageBytes);   // past the end the last tile once more; nobody attends it
            attend(ka, kb, [&](int k) {
                if (k == 0) {
                    wait_loads<2 * kLoads>();   // V is there
                    if ((tile + 1) * kTileTokens > rows.L) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) pages.clean(vbuf, at + h * Slot::kPageBytes, tile * kTileTokens + h * kPage);
                        wait_lds();
                    }
                }
                return Slot::v_operand(vbuf, at - 2 * Slot::kPageBytes, k, lane);
            }, tile, masked);
            wait_lds();
#pragma unroll
            for (int h = 0; h < 2; ++h) pages.bring(1, next[h], vbuf, at + h * Slot::kPageBytes);
            next[0] = after[0], next[1] = after[1];
        };
        const int plain = rows.min_end / kTileTokens;
        const int count_plain = min(count, plain > wave ? (plain - wave + kW - 1) / kW : 0);
        int i = 0;
#pragma unroll 1
        for (; i < count_plain; ++i) turn(i, std::false_type{});
#pragma unroll 1
        for (; i < count; ++i) turn(i, std::true_type{});
        wait_loads<0>();
    }
    leave_parts<P, NB, kW>(a, rows, st, wave, lane, ms, ls, [&](int w) { return (w < kW / 2 ? kbuf : vbuf) + w % (kW / 2) * PartImage<P, NB>::kBytes; });
}

// head_dim 64: workgroups of 4 waves; a round is two tiles in one of several arrays.  Softmax and matrix instructions of a wave's step take about as
// long, one after the other, so what counts is other waves to fill the gaps: with two column blocks per wave (142 registers) and three arrays, asked for two
// rounds ahead, a compute unit holds three workgroups.  Against the general kernel with as many blocks and waves: 160 random calls 1.05 times as fast, up to 1.15 (10
// sequences of 87 - 595, 227 - 1365 queries, 16/2 heads 18.0 -> 16.9 us; 14 of 582 - 785, whole prompts, 32/4 62.5 -> 56.3).  Four workgroups' worth of
// waves (16 to a compute unit, 128 registers) are no faster than the general kernel.
// With four blocks per wave, four arrays and three rounds ahead it holds two, and a tile's operands are read once for twice the rows: for the
// largest calls (16 x 8192 / 2048, 32/8 heads 1909 -> 1828 us against the general kernel).
//
// head_dim 128: 8 waves of two column blocks, one workgroup to a compute unit; a wave brings K or V of one page per round.  For contexts of a few tiles, which do not pay
// for the start-up of the two phases below.  Against the general kernel, 179 random calls under 512 tokens whose average sequence fills three quarters of a
// workgroup's blocks or more 1.08 times as fast, under 128 tokens 1.15 (14 sequences of 95 - 115, whole prompts, 32/4 heads 19.5 -> 15.1 us); 31 emptier ones .98,
// as all waves wait for rounds that few of them attend.
template <int D, int kW, int NB>
__global__ __launch_bounds__(kW * 64, D == 64 && NB == 2 ? 3 : 2) void prefill_direct_kernel(PrefillArgs a)
{
    constexpr int kTiles = 2, kAhead = D == 64 && NB == 2 ? 2 : 3;
    typedef Bf16Path<D> P;
    typedef RowSlot<D> Slot;
    constexpr int kLoads = Slot::kPageBytes / 1024;   // of a K or V page
    constexpr int kKinds = 4 * kTiles / kW;   // a wave brings K and V of one page per round, or one of them
    static_assert(kKinds == 1 || kKinds == 2, "whole pages per wave");
    __shared__ __attribute__((aligned(16))) char buf0[kTiles * Slot::kBytes], buf1[kTiles * Slot::kBytes], buf2[kTiles * Slot::kBytes], buf3[kAhead == 3 ? kTiles * Slot::kBytes : 16];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    PrefillRows rows;
    if (!rows.find(a, kW, wave, NB)) return;
    int row_end[NB];
    u32x4 qop[NB][D / 32];
    typename P::ParkedState st[NB];
    rows.load<P>(a, lane, qop, row_end, st);

    const ConstTable bt = (ConstTable)(a.block_table + (int64_t)rows.b * a.max_blocks);
    const int64_t page_bytes = (int64_t)Slot::kPageBytes * a.Hkv;
    const char *kbase = static_cast<const char *>(a.k_pages) + rows.hb.g * Slot::kPageBytes;
    const char *vbase = static_cast<const char *>(a.v_pages) + rows.hb.g * Slot::kPageBytes;
    const int ntiles = (rows.kv_end + kTileTokens - 1) / kTileTokens;
    const int last_page = (rows.kv_end + kPage - 1) / kPage - 1;
    const int rounds = (ntiles + kTiles - 1) / kTiles;
    // past the end the last page once more; nobody attends it
    const int my_page = kKinds == 2 ? wave : wave % (2 * kTiles), my_kind = wave / (2 * kTiles);
    auto page_of = [&](int rd) { return bt[min(2 * kTiles * min(rd, rounds - 1) + my_page, last_page)]; };
    const int my_k = (my_page >> 1) * Slot::kBytes + (my_page & 1) * Slot::kPageBytes, my_v = my_k + 2 * Slot::kPageBytes;
    auto bring = [&](char *buf, int page) {
        if (kKinds == 2 || my_kind == 0)
#pragma unroll
            for (int j = 0; j < kLoads; ++j) load_to_lds(kbase + page * page_bytes, Slot::kPageBytes, Slot::source(0, j * 1024 + lane * 16), buf + (my_k + j * 1024));
        if (kKinds == 2 || my_kind == 1)
#pragma unroll
            for (int j = 0; j < kLoads; ++j) load_to_lds(vbase + page * page_bytes, Slot::kPageBytes, Slot::source(1, j * 1024 + lane * 16), buf + (my_v + j * 1024));
    };
    // V rows of tokens that do not exist may hold anything: zeros
    auto clean = [&](char *buf, int rd) {
        const int tok0 = (2 * kTiles * rd + my_page) * kPage;
        if ((kKinds == 1 && my_kind == 0) || tok0 + kPage <= rows.L) return;
#pragma unroll
        for (int j = 0; j < kLoads; ++j)
            if (tok0 + (j * 1024 + lane * 16) / Slot::kRowBytes >= rows.L) *reinterpret_cast<u32x4 *>(buf + (my_v + j * 1024 + lane * 16)) = u32x4{0, 0, 0, 0};
    };
    auto step = [&](const char *buf, int j, int tile, auto masked) {
        u32x4 ka[D / 32], kb[D / 32];
        Slot::fetch_k(buf, j * Slot::kBytes, lane, ka, kb);
        P::template attend_fetched<NB, decltype(masked)::value, false>(
            ka, kb, [&](int k) { return Slot::v_operand(buf, j * Slot::kBytes, k, lane); }, qop, st, a.scale_log2e, tile * kTileTokens,
            lane, row_end, true, nullptr, rows.first_end, rows.tpb);
    };
    constexpr int kPer = kKinds * kLoads;   // loads a wave issues per round
    auto turn = [&](int rd, char *cur, char *next, char *fill, int page) {
        bring(fill, page);   // round rd + kAhead
        if (rows.active) {
            const int t0 = kTiles * rd * kTileTokens;
            const int j_end = min(kTiles, (rows.max_end - t0 + kTileTokens - 1) / kTileTokens);
            const int j_plain = max(0, min(j_end, (rows.min_end - t0) / kTileTokens));
            int j = 0;
#pragma unroll 1
            for (; j < j_plain; ++j) step(cur, j, kTiles * rd + j, std::false_type{});
#pragma unroll 1
            for (; j < j_end; ++j) step(cur, j, kTiles * rd + j, std::true_type{});
        }
        wait_loads<(kAhead - 1) * kPer>();   // round rd + 1 has arrived
        clean(next, rd + 1);
        wait_lds();
        phase_barrier();
    };
    if (rounds > 0) {
        bring(buf0, page_of(0));
        bring(buf1, page_of(1));
        if constexpr (kAhead == 3) bring(buf2, page_of(2));
        int page = page_of(kAhead);
        wait_loads<(kAhead - 1) * kPer>();
        clean(buf0, 0);
        wait_lds();
        phase_barrier();
        for (int rd = 0;;) {
            { const int after = page_of(rd + kAhead + 1); turn(rd, buf0, buf1, kAhead == 3 ? buf3 : buf2, page); page = after; }
            if (++rd == rounds) break;
            { const int after = page_of(rd + kAhead + 1); turn(rd, buf1, buf2, buf0, page); page = after; }
            if (++rd == rounds) break;
            { const int after = page_of(rd + kAhead + 1); turn(rd, buf2, kAhead == 3 ? buf3 : buf0, buf1, page); page = after; }
            if (++rd == rounds) break;
            if constexpr (kAhead == 3) {
                { const int after = page_of(rd + kAhead + 1); turn(rd, buf3, buf0, buf2, page); page = after; }
                if (++rd == rounds) break;
            }
        }
        wait_loads<0>();   // no load may outlive the workgroup
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        bool in_range, row_ok;
        int64_t row;
        rows.locate(a, c, lane & 15, in_range, row_ok, row);
        const float l = P::weight_sum(st[c]);
        if (in_range) Slot::store(st[c], a.out + row * D, lane, row_ok, l);
    }
}

// head_dim 128: one workgroup of 8 waves per compute unit, two waves per SIMD that take turns at the matrix pipe.  A tile is two
// phases: the matrix phase (scores of tile t + 1, weighted sum of tile t: 34 matrix instructions) and the vector phase (softmax
// of tile t).  Waves 4 to 7 run one phase behind waves 0 to 3, and a barrier ends every phase, so that while
// one wave of a SIMD issues matrix instructions the other does its exponentials.  Tiles are asked for four ahead, into one of
// six slots: a slot is read last (V, by the late waves) two tiles after it was due, and filled again from then on.
//
// What bounds it (16 x 8192 / 2048 queries, 32/8 heads: 3.45 -> 3.22 ms on one machine, 1.2 PFLOP/s): the matrix pipe is busy 55 % of the
// time; without the loads into LDS the kernel takes 0.88 of its time, without any operand reads 0.9, without the exponentials 0.99, with
// matrix instructions and barriers alone 0.70.  Operand reads and loads moved between the two phases, and more of
// them beside the matrix instructions, gave 3.25 - 3.35 ms.
__global__ __launch_bounds__(512, 2) void prefill_pingpong_kernel(PrefillArgs a)
{
    constexpr int D = 128, NB = 2, kW = 8, S = D / 32, K = D / 16;
    typedef Bf16Path<D> P;
    typedef RowSlot<D> Slot;
    constexpr int kLoads = Slot::kBytes / 1024 / kW;   // of a wave per tile
    __shared__ __attribute__((aligned(16))) char buf0[Slot::kBytes], buf1[Slot::kBytes], buf2[Slot::kBytes], buf3[Slot::kBytes], buf4[Slot::kBytes], buf5[Slot::kBytes];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    PrefillRows rows;
    if (!rows.find(a, kW, wave, NB)) return;
    int row_end[NB];
    u32x4 qop[NB][S];
    typename P::ParkedState st[NB];
    rows.load<P>(a, lane, qop, row_end, st);

    const ConstTable bt = (ConstTable)(a.block_table + (int64_t)rows.b * a.max_blocks);
    const int64_t page_bytes = (int64_t)Slot::kPageBytes * a.Hkv;
    const int ntiles = (rows.kv_end + kTileTokens - 1) / kTileTokens;
    const int last_page = (rows.kv_end + kPage - 1) / kPage - 1;
    const int mine = rows.active ? (rows.max_end + kTileTokens - 1) / kTileTokens : 0;   // tiles this wave attends
    const float c = a.scale_log2e;

    // this wave brings bytes [kLoads * 1024 * wave, ..) of every slot, which lie in one page's K or V
    const int my_at = kLoads * 1024 * wave, my_kind = my_at / (2 * Slot::kPageBytes), my_page = my_at / Slot::kPageBytes & 1;
    const int my_off = my_at % Slot::kPageBytes;
    const char *pool = static_cast<const char *>(my_kind ? a.v_pages : a.k_pages) + rows.hb.g * Slot::kPageBytes;
    int from[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) from[j] = Slot::source(my_kind, my_off + j * 1024 + lane * 16);
    // past the end the last page once more; nobody attends it
    auto page_of = [&](int t) { return bt[min(2 * min(t, ntiles - 1) + my_page, last_page)]; };
    auto bring = [&](char *buf, int page) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) load_to_lds(pool + page * page_bytes, Slot::kPageBytes, from[j], buf + (my_at + j * 1024));
    };
    // V rows of tokens that do not exist may hold anything: zeros
    auto clean = [&](char *buf, int t) {
        const int tok0 = t * kTileTokens + my_page * kPage;
        if (my_kind == 0 || tok0 + kPage <= rows.L) return;
#pragma unroll
        for (int j = 0; j < kLoads; ++j)
            if (tok0 + (my_off + j * 1024 + lane * 16) / Slot::kRowBytes >= rows.L) *reinterpret_cast<u32x4 *>(buf + (my_at + j * 1024 + lane * 16)) = u32x4{0, 0, 0, 0};
    };

    u32x4 ka[S], kb[S], va[K], pop[NB];
    f32x4 sa[NB], sb[NB];
    const u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};  // bf16 1.0 pairs: the weight sum
    auto fetch_k = [&](const char *buf) { Slot::fetch_k(buf, 0, lane, ka, kb); };
    auto fetch_v = [&](const char *buf) {
#pragma unroll
        for (int k = 0; k < K; ++k) va[k] = Slot::v_operand(buf, 0, k, lane);
    };
    auto first_products = [&]() {
#pragma unroll
        for (int i = 0; i < NB; ++i) sa[i] = sb[i] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                sa[i] = mfma_bf16_k32(ka[s], qop[i][s], sa[i]);
                sb[i] = mfma_bf16_k32(kb[s], qop[i][s], sb[i]);
            }
    };
    auto second_products = [&]() {
#pragma unroll
        for (int i = 0; i < NB; ++i) st[i].acc[K] = mfma_bf16_k32(ones, pop[i], st[i].acc[K]);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < NB; ++i) st[i].acc[k] = mfma_bf16_k32(va[k], pop[i], st[i].acc[k]);
    };
    // as in Bf16Path::attend_parked: weights against the reference as it stands, which moves only when one of them reaches 2
    auto softmax = [&](int t) {
        float x[NB][8];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[i][e] = sa[i][e];
                x[i][4 + e] = sb[i][e];
            }
        if ((t + 1) * kTileTokens > rows.min_end) {   // wave-uniform
#pragma unroll
            for (int i = 0; i < NB; ++i) mask_scores(x[i], t * kTileTokens, row_end[i], lane >> 4);
        }
        auto weights = [&](int i) {
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i][e], c, -st[i].m));
#pragma unroll
            for (int e = 0; e < 8; e += 2) pop[i][e >> 1] = cvt_pk_bf16(p[e], p[e + 1]);
        };
        unsigned big = 0;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            weights(i);
            big |= pop[i][0] | pop[i][1] | pop[i][2] | pop[i][3];
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64((big & 0x40004000u) != 0) != 0, 0)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const unsigned own = (pop[i][0] | pop[i][1] | pop[i][2] | pop[i][3]) & 0x40004000u;
                if (__builtin_amdgcn_ballot_w64(own != 0) != 0) {
                    advance_max(st[i], max_of(st[i].m, head_max(max8(x[i])) * c + kLead));
                    weights(i);
                }
            }
        }
    };
    auto turn = [&](int t, const char *cur, const char *next, char *arrive, char *fill, int page) {
        // vector phase: tile t + 4 is asked for, the K operands of tile t + 1 arrive beside the softmax
        bring(fill, page);
        fetch_k(next);
        softmax(t);
        wait_loads<2 * kLoads>();   // tile t + 2 has arrived
        clean(arrive, t + 2);
        wait_lds();
        phase_barrier();
        // matrix phase: the V^T operands arrive beside the scores
        fetch_v(cur);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        first_products();
        if (t < mine) second_products();   // wave-uniform: not past the wave's last row, where V may be anything
        __builtin_amdgcn_s_setprio(0);
        phase_barrier();
    };
    if (ntiles > 0) {
        bring(buf0, page_of(0));
        bring(buf1, page_of(1));
        bring(buf2, page_of(2));
        bring(buf3, page_of(3));
        wait_loads<2 * kLoads>();
        clean(buf0, 0);
        clean(buf1, 1);
        wait_lds();
        int page = page_of(4);
        phase_barrier();
        fetch_k(buf0);
        if (wave >= kW / 2) phase_barrier();   // one phase behind from here on
        first_products();
        phase_barrier();
        for (int t = 0;;) {
            { const int after = page_of(t + 5); turn(t, buf0, buf1, buf2, buf4, page); page = after; }
            if (++t == ntiles) break;
            { const int after = page_of(t + 5); turn(t, buf1, buf2, buf3, buf5, page); page = after; }
            if (++t == ntiles) break;
            { const int after = page_of(t + 5); turn(t, buf2, buf3, buf4, buf0, page); page = after; }
            if (++t == ntiles) break;
            { const int after = page_of(t + 5); turn(t, buf3, buf4, buf5, buf1, page); page = after; }
            if (++t == ntiles) break;
            { const int after = page_of(t + 5); turn(t, buf4, buf5, buf0, buf2, page); page = after; }
            if (++t == ntiles) break;
            { const int after = page_of(t + 5); turn(t, buf5, buf0, buf1, buf3, page); page = after; }
            if (++t == ntiles) break;
        }
        if (wave < kW / 2) phase_barrier();   // every wave has met the same number
        wait_loads<0>();                      // no load may outlive the workgroup
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        bool in_range, row_ok;
        int64_t row;
        rows.locate(a, i, lane & 15, in_range, row_ok, row);
        const float l = P::weight_sum(st[i]);
        if (in_range) Slot::store(st[i], a.out + row * D, lane, row_ok, l);
    }
}

hipError_t launch_prefill(const PrefillArgs &a, int head_dim, int kv_dtype, hipStream_t stream, hipEvent_t start,
                          hipEvent_t stop)
{
    const unsigned pairs = (unsigned)a.B * (unsigned)(a.Hkv * a.HB);
    const unsigned slots = pairs * (unsigned)a.q_blocks, grid = a.plan.on_device ? (slots + kXcds - 1) / kXcds * kXcds : a.plan.order ? slots : prefill_grid(a.q_blocks, pairs);
    if (grid == 0) return hipSuccess;
    auto go = [&](auto kernel, int waves) {
        const dim3 g(grid), b(waves * 64);
        if (start || stop)
            hipExtLaunchKernelGGL(kernel, g, b, 0, stream, start, stop, 0, a);
        else
            hipLaunchKernelGGL(kernel, g, b, 0, stream, a);
    };
    // the instances for the plans: waves, tiles of a round, split, column blocks per wave, waves per SIMD
    auto wide = [&](auto path) {   // head_dim 128: one workgroup of 8 waves per compute unit
        typedef decltype(path) P;
        if constexpr (std::is_same<P, Bf16Path<128>>::value) {
            if (a.plan.on_device) return go(prefill_wide_kernel_direct<0>, 8);
            switch (a.plan.blocks) {
            case 16:   // (a context of a few tiles does not pay for the start-up of the two phases: 127 tokens, 32/8 heads 14.7 against 15.9 us)
                return a.plan.phases ? go(prefill_pingpong_kernel, 8) : a.plan.direct ? go(prefill_direct_kernel<128, 8, 2>, 8) : go(prefill_wide_kernel<P, 8, 4, 1, 2, 2>, 8);
            case 8: return go(prefill_wide_kernel_direct<2>, 8);
            case 4: return go(prefill_wide_kernel_direct<4>, 8);
            default: return go(prefill_wide_kernel_own<128, 8, 2>, 8);
            }
        } else {
            switch (a.plan.blocks) {
            case 16: return go(prefill_wide_kernel<P, 8, 4, 1, 2, 2>, 8);
            case 8: return a.plan.split == 1 ? go(prefill_wide_kernel<P, 4, 2, 1, 2, 2>, 4) : go(prefill_wide_kernel<P, 8, 4, 2, 2, 2>, 8);
            case 4: return go(prefill_wide_kernel<P, 8, 4, 4, 2, 2>, 8);
            default: return go(prefill_wide_kernel<P, 8, 8, 8, 2, 2>, 8);
            }
        }
    };
    auto narrow = [&](auto path) {   // head_dim 64: half the operands per tile, so a wave has room for four blocks, or a compute unit for three workgroups
        typedef decltype(path) P;
        if constexpr (std::is_same<P, Bf16Path<64>>::value) {
            switch (a.plan.blocks) {
            case 16: return go(prefill_direct_kernel<64, 4, 4>, 4);
            case 8: return go(prefill_direct_kernel<64, 4, 2>, 4);
            case 4: return go(prefill_wide_kernel_own<64, 4, 4>, 4);
            default: return go(prefill_wide_kernel_own<64, 8, 2>, 8);
            }
        } else {
            switch (a.plan.blocks) {
            case 8: return go(prefill_wide_kernel<P, 4, 2, 1, 2, 3>, 4);
            case 4: return go(prefill_wide_kernel<P, 4, 4, 4, 4, 2>, 4);
            default: return go(prefill_wide_kernel<P, 8, 8, 8, 2, 2>, 8);
            }
        }
    };
    if (kv_dtype == 0 && head_dim == 128)
        wide(Bf16Path<128>{});
    else if (kv_dtype == 0 && head_dim == 64)
        narrow(Bf16Path<64>{});
    else if (kv_dtype == 1 && head_dim == 128)
        wide(Fp8Path{});
    else if (kv_dtype == 1 && head_dim == 64)
        narrow(Fp8Path64{});
    else
        return hipErrorNotSupported;
    return hipGetLastError();
}

}  // namespace sd
