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
// Bound by the matrix pipe and by the latency between dependent stages with two waves per SIMD: 16 x 8192 / 2048 queries,
// 32/8 heads, d = 128, bf16 runs at 1.1 PFLOP/s.
//
// The causal limit is a per-lane token bound in the score mask; a wave stops
// once a tile starts at or past the last position any of its rows may see.
//
// Large calls: each wave carries its rows through the whole range with the
// online softmax, so there is no split and no merge.  Small calls, whose query blocks
// would leave compute units idle, take smaller blocks and split their range over the waves of
// the workgroup (prefill_blocks): kSplit neighbouring waves own the same rows and
// every kSplit-th tile each, and add up their (max, sum, weighted sum) through LDS at
// the end.  Nothing leaves the workgroup, so no workspace is needed.
#include <cfloat>
#include <type_traits>

#include "attn_tile.h"

namespace sd {

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
    const int Hv = a.Hkv * a.HB;
    const PrefillItem item = prefill_item(blockIdx.x, a.q_blocks, a.B * Hv);
    if (item.block >= a.q_blocks) return;
    const int jb = a.q_blocks - 1 - item.block;
    const HeadBlock hb = head_block(item.pair % Hv, a.G, a.HB);
    const int g = hb.g;
    const int b = item.pair / Hv;
    const int tpb = units_per_block(a.G);  // query tokens per column block
    const int tpw = NB * tpb;              // and per wave
    const int group = wave / kSplit, part = wave % kSplit;

    // everything below up to the loop is workgroup-uniform
    const int qs = a.q_start[b];
    const int nq = min(a.q_start[b + 1] - qs, a.max_q_len);
    const int i0 = jb * kGroups * tpw;
    if (i0 >= nq) return;
    if (qs < 0 || (int64_t)qs + nq > a.total_q) return;  // rows outside q: nothing is read or written
    const int L = max(0, min(a.context_lens[b], a.max_context_len));
    const int base = L - nq;                                        // position of query 0 (may be negative)
    const int kv_end = max(0, base + min(nq, i0 + kGroups * tpw));  // tokens the block's last row sees

    // this wave's rows
    const int iw0 = i0 + group * tpw;
    const int iw1 = min(iw0 + tpw, nq);
    const bool active = iw0 < nq && base + iw1 > 0;  // some row of the wave sees a token
    const int wave_max_end = base + iw1;              // its last row's limit
    const int wave_min_end = max(0, base + iw0) + 1;  // its first visible row's limit
    const int n = lane & 15;
    // row of column block c in this lane: query token, whether it exists, whether it sees a token
    // (recomputed where needed rather than kept in registers across the loop)
    auto locate = [&](int c, int n, bool &in_range, bool &row_ok, int64_t &row) {
        const int i = iw0 + c * tpb + n / hb.rows;
        in_range = n / hb.rows < tpb && i < nq;
        row_ok = in_range && base + i >= 0;
        row = ((int64_t)qs + i) * a.Hq + hb.head0 + n % hb.rows;
        return i;
    };
    int row_end[NB];
    u32x4 qop[NB][D / 32];
    typename P::B::ParkedState st[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        bool in_range, row_ok;
        int64_t row;
        const int i = locate(c, n, in_range, row_ok, row);
        // rows that see nothing ride along with zero queries, masked only past the sequence's end
        row_end[c] = row_ok ? base + i + 1 : L;
#pragma unroll
        for (int s = 0; s < D / 32; ++s)
            qop[c][s] = row_ok ? (*reinterpret_cast<const u32x4 *>(a.q + row * D + P::B::q_offset(s, lane)) & a.q_keep) ^ a.q_flip
                               : u32x4{0, 0, 0, 0};
        reset(st[c]);
        st[c].m = -FLT_MAX;   // finite: a split may meet only tokens that a row does not see
    }

    const int32_t *bt = a.block_table + (int64_t)b * a.max_blocks;
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
                                                                             slot + P::B::kParkedBytes);
    };
    const int ntiles = (kv_end + kTileTokens - 1) / kTileTokens;
    const int last_page = (kv_end + kPage - 1) / kPage - 1;

    if constexpr (kOwn) {
        // tiles wave, wave + kW, ...: those below `plain` end at or before the first visible row's limit
        const int count = ntiles > wave ? (ntiles - wave + kW - 1) / kW : 0;
        const int plain = wave_min_end / kTileTokens;
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
                if (active) {
                    // the round's tiles below the diagonal of every row of the wave, then those on it
                    const int t0 = kTiles * rd * kTileTokens;
                    const int j_end = min(kTiles, (wave_max_end - t0 + kTileTokens - 1) / kTileTokens);
                    const int j_plain = max(0, min(j_end, (wave_min_end - t0) / kTileTokens));
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
            locate(c, n, in_range, row_ok, row);
            if (!in_range) continue;
            const float inv = row_ok ? 1.0f / l : 0.0f;  // rows before the sequence's first token get zeros
#pragma unroll
            for (int k = 0; k < D / 16; ++k) st[c].acc[k] = row_ok ? st[c].acc[k] * inv : f32x4{0, 0, 0, 0};
            P::store_acc(st[c], a.out + row * D, lane >> 4);
        }
    } else {
        // The results of the kSplit waves of a group, through LDS: rows [wave][block][16][D], then maxima and
        // weight sums.  Every wave then finishes its share of its group's rows, parts added in order.
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
        constexpr int kRowWords = D / 4;   // 16-byte words of a row
        for (int idx = part * 64 + lane; idx < NB * 16 * kRowWords; idx += kSplit * 64) {
            const int rr = idx / kRowWords, col = idx % kRowWords * 4;
            const int c = rr >> 4, rn = rr & 15;
            bool in_range, row_ok;
            int64_t row;
            locate(c, rn, in_range, row_ok, row);
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
                num += w * *reinterpret_cast<const f32x4 *>(image + at * kImage + col);
            }
            *reinterpret_cast<f32x4 *>(a.out + row * D + col) = row_ok ? num / den : f32x4{0, 0, 0, 0};
        }
    }
}

hipError_t launch_prefill(const PrefillArgs &a, int head_dim, int kv_dtype, hipStream_t stream, hipEvent_t start,
                          hipEvent_t stop)
{
    const unsigned grid = prefill_grid(a.q_blocks, a.B * a.Hkv * a.HB);
    if (grid == 0) return hipSuccess;
    auto go = [&](auto kernel, int waves) {
        const dim3 g(grid), b(waves * 64);
        if (start || stop)
            hipExtLaunchKernelGGL(kernel, g, b, 0, stream, start, stop, 0, a);
        else
            hipLaunchKernelGGL(kernel, g, b, 0, stream, a);
    };
    // the instances for the four block sizes of prefill_blocks: waves, tiles of a round, split, column blocks per wave, waves per SIMD
    auto wide = [&](auto path) {   // head_dim 128: one workgroup of 8 waves per compute unit
        typedef decltype(path) P;
        switch (a.blocks) {
        case 16: return go(prefill_wide_kernel<P, 8, 4, 1, 2, 2>, 8);
        case 8: return go(prefill_wide_kernel<P, 8, 4, 2, 2, 2>, 8);
        case 4: return go(prefill_wide_kernel<P, 8, 4, 4, 2, 2>, 8);
        default: return go(prefill_wide_kernel<P, 8, 8, 8, 2, 2>, 8);
        }
    };
    auto narrow = [&](auto path) {   // head_dim 64: half the operands per tile, so a wave has room for four blocks, or a compute unit for three workgroups
        typedef decltype(path) P;
        switch (a.blocks) {
        case 16: return go(prefill_wide_kernel<P, 4, 4, 1, 4, 2>, 4);
        case 8: return go(prefill_wide_kernel<P, 4, 2, 1, 2, 3>, 4);
        case 4: return go(prefill_wide_kernel<P, 4, 4, 4, 4, 2>, 4);
        default: return go(prefill_wide_kernel<P, 8, 8, 8, 2, 2>, 8);
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
