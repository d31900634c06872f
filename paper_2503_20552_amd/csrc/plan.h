// The order and the cut of a pass of one workgroup per item, made on the device from the lengths.
//
// Longer rows first, in equal partitions of a length that follows from the tokens the pass really has.  The
// hardware hands items out in their order as workgroups end, so what stands last decides how long the last
// compute units work alone: in the batch's own order that is any row's last partition, by descending
// length it is the shortest rows.  And a partition costs its workgroup about 6 us besides its tokens (8 where
// rows meet inside the pass): rows that are no burden to the tail stay whole.
//
// One workgroup per row, which reads all lengths: its place in the list follows from those alone, with no exchange
// between workgroups.  The list has no holes: with places left empty between the items (partitions
// that shrink as the work runs out, their places by a closed form) 256 requests of median length 1500 took
// 402 to 416 us, with this list 380 (in the batch's own order 407).
#pragma once

#include "adr_device.h"

#include <algorithm>

namespace adr {

constexpr uint32_t kNoRow = 0xffffffffu; // in place of an item's row: past the last item
constexpr int kSlots = 768;              // workgroups the chip holds at once, three to a compute unit

// Tiles of a partition, as a share of what a slot has to do if all do the same: kShareMost of it, or, where that
// is more than kPlanTiles, as little as kShareLeast (a pass of few and very long rows must be cut
// somewhere).  us a step with shares of 0.5 / 0.75 / 1 / 1.25 / 1.5 / 2: 128 requests x 8 kv-heads, heavy-tailed
// lengths 77 / 74 / 72 / 69 / 73 / 70, 160 of up to 3000 tokens 174 / 172 / 167 / 164 / 164 / 166, 256 of
// median length 1500 385 / 380 / 380 / 380 / 379 / 384.
constexpr uint32_t kPlanTiles = 256;
constexpr float kShareMost = 1.25f, kShareLeast = 0.125f;

// With fewer rows than places most rows are cut, and long ones must not stand alone at the end: partitions of
// kFewShare and no less than kFewTiles, kFewParts of a row as long as none is longer than kFewLong.  Rows are merged
// by a kernel of their own here: nearly every item would keep its place until it is counted (a step of 37
// requests x 8 kv-heads 49 and 52 us).
// Rows of one length, or nearly (the longest no more than kFewEven times the mean), come in rounds whatever their
// order, and the last round should be a small one: they are cut as without a plan, into no more than kEvenItems.
// us a step, in the batch's order and planned: eight layers of 40 requests of median length 1000, replayed, 413 and
// 389, 128 of median 1500, heads of 64, 111 and 107, 75 of the same, pages of 64, 125 and 122, 80 of heavy-tailed
// lengths 61.5 and 54; 33 of 6000 tokens 142 and, without the exception, 150.
constexpr uint32_t kFewTiles = 16, kFewParts = 5, kEvenItems = 4800;
constexpr float kFewShare = 0.75f, kFewLong = 2.f, kFewEven = 1.1f;

constexpr uint32_t kPlanRowTiles = 1 << 20; // tiles of a row that count (any number of rows' tiles adds up in 32 bits)

// Places in the list that can be taken, kv-heads counted once: one per row and one per whole partition of all tokens.
inline int64_t plan_places(int B, int H, int max_seq_len, bool few)
{
    const int64_t tiles = (int64_t)B * std::min<int64_t>(((int64_t)max_seq_len + kPageSize - 1) / kPageSize, kPlanRowTiles);
    const int64_t least = (int64_t)(kSlots / (kShareLeast * H)), most = (int64_t)(kSlots / (kShareMost * H));
    const int64_t places = few ? (int64_t)(kEvenItems / H + 1) : std::max(most, std::min(least, tiles / kPlanTiles));
    return (B + places + 2 + 7) / 8 * 8;
}

// Over a workgroup of T threads, in every thread: the sum of a, and b by `op` (from 0 on).
template <int T, typename Op>
__device__ __forceinline__ void group_reduce(uint32_t &a, uint32_t &b, Op op)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        a += (uint32_t)__shfl_xor((int)a, off);
        b = op(b, (uint32_t)__shfl_xor((int)b, off));
    }
    if constexpr (T > 64) {
        __shared__ uint32_t parts[T / 64][2];
        __syncthreads(); // (an earlier call's have been read)
        if ((threadIdx.x & 63) == 0) {
            parts[threadIdx.x / 64][0] = a;
            parts[threadIdx.x / 64][1] = b;
        }
        __syncthreads();
        a = b = 0;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) {
            a += parts[w][0];
            b = op(b, parts[w][1]);
        }
    }
}

// How the rows of a pass are cut: in partitions of `most` tiles or less, but no more than `parts` of them as long as
// those have `longest` tiles or less.
struct PlanCut {
    uint32_t most, longest, parts;
    uint32_t grain; // tokens a partition is a multiple of: two tiles for each of four waves, or one
};
__device__ __forceinline__ PlanCut plan_cut(const PlanParams &p, uint32_t all, uint32_t longest_row)
{
    const float slot = (float)all * p.heads_per_slot;
    PlanCut c = {(uint32_t)ceilf(kShareMost * slot), 1u, 0u, (uint32_t)kCutLeast};
    if (p.few) {
        c.most = max((uint32_t)ceilf(kFewShare * slot), kFewTiles);
        c.parts = kFewParts;
        if ((float)longest_row * (float)p.B <= kFewEven * (float)all) {
            c.most = max((uint32_t)p.even_tiles, (uint32_t)ceilf((float)longest_row * (float)p.B * (p.heads_per_slot * kSlots / kEvenItems)));
            c.parts = 0;
            c.grain = kCutLeast / 2;
            return c;
        }
        c.longest = max((uint32_t)ceilf(kFewLong * slot), c.most);
        return c;
    }
    if (c.most > kPlanTiles)
        c.most = max((uint32_t)ceilf(kShareLeast * slot), kPlanTiles);
    c.most = max(c.most, (uint32_t)(kCutLeast / kPageSize));
    return c;
}

// Row of L tokens: its partitions, and the tokens of each.
__device__ __forceinline__ int plan_parts(int L, const PlanCut &c, int max_parts, int &tokens)
{
    const uint32_t tiles = min(((uint32_t)L + kPageSize - 1) / kPageSize, kPlanRowTiles);
    tokens = L;
    if (tiles <= c.most)
        return 1;
    uint32_t n = (tiles + c.most - 1) / c.most;
    if (c.parts)
        n = min(n, max(c.parts, (tiles + c.longest - 1) / c.longest));
    n = min(n, (uint32_t)max_parts);
    tokens = (int)((((uint32_t)L + n - 1) / n + c.grain - 1) / c.grain * c.grain);
    return (L + tokens - 1) / tokens;
}

// Row b's items, {row, its length, tokens per partition, partition | partitions << 16}, and the words its partitions'
// arrivals are counted in, or their number for the merge kernel.
template <int T>
__device__ __forceinline__ void plan_row(const PlanParams &p, int b)
{
    const auto length = [&](int i) { return max(min(p.seq_lens[i], p.max_seq_len), 0); };
    const int mine = length(b);
    uint32_t all = 0, longest = 0;
    for (int i = threadIdx.x; i < p.B; i += T) {
        const uint32_t tiles = min(((uint32_t)length(i) + kPageSize - 1) / kPageSize, kPlanRowTiles);
        all += tiles;
        longest = max(longest, tiles);
    }
    group_reduce<T>(all, longest, [](uint32_t x, uint32_t y) { return max(x, y); });
    const PlanCut cut = plan_cut(p, all, longest);
    uint32_t ahead = 0, behind = 0;
    int tokens;
    for (int i = threadIdx.x; i < p.B; i += T) {
        const int L = length(i);
        const uint32_t n = plan_parts(L, cut, p.max_parts, tokens);
        if (L > mine || (L == mine && i < b))
            ahead += n;
        else if (i != b)
            behind += n;
    }
    group_reduce<T>(ahead, behind, [](uint32_t x, uint32_t y) { return x + y; });
    const int n = plan_parts(mine, cut, p.max_parts, tokens);
    // (The last row's workgroup also marks what is left of the list.)
    const uint32_t end = min(behind ? ahead + n : (uint32_t)p.max_items, (uint32_t)p.max_items);
    for (uint32_t j = threadIdx.x; ahead + j < end; j += T)
        p.items[ahead + j] = u32x4{j < (uint32_t)n ? (uint32_t)b : kNoRow, (uint32_t)mine, (uint32_t)tokens, j | (uint32_t)n << 16};
    if (p.part_counts && threadIdx.x == 0)
        p.part_counts[b] = n;
    if (p.arrivals && n > 1)
        for (int i = threadIdx.x; i < p.heads; i += T)
            p.arrivals[(int64_t)b * p.heads + i] = 0u;
}

} // namespace adr
