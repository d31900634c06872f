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
constexpr uint32_t kPlanRowTiles = 1 << 20; // tiles of a row that count (any number of rows' tiles adds up in 32 bits)

// Places in the list that can be taken, kv-heads counted once: one per row and one per whole partition of all tokens.
inline int64_t plan_places(int B, int H, int max_seq_len)
{
    const int64_t tiles = (int64_t)B * std::min<int64_t>(((int64_t)max_seq_len + kPageSize - 1) / kPageSize, kPlanRowTiles);
    const int64_t least = (int64_t)(kSlots / (kShareLeast * H)), most = (int64_t)(kSlots / (kShareMost * H));
    return (B + std::max(most, std::min(least, tiles / kPlanTiles)) + 2 + 7) / 8 * 8;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
        x += (uint32_t)__shfl_xor((int)x, off);
    return x;
}

// Sums of two values over a workgroup of T threads, in every thread.
template <int T>
__device__ __forceinline__ void group_sums(uint32_t &a, uint32_t &b)
{
    a = wave_sum(a);
    b = wave_sum(b);
    if constexpr (T > 64) {
        __shared__ uint32_t sums[T / 64][2];
        __syncthreads(); // (an earlier call's sums have been read)
        if ((threadIdx.x & 63) == 0) {
            sums[threadIdx.x / 64][0] = a;
            sums[threadIdx.x / 64][1] = b;
        }
        __syncthreads();
        a = b = 0;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) {
            a += sums[w][0];
            b += sums[w][1];
        }
    }
}

// Row of L tokens: partitions of `most` tiles or less, and the tokens of each.
__device__ __forceinline__ int plan_parts(int L, uint32_t most, int max_parts, int &tokens)
{
    const uint32_t tiles = min(((uint32_t)L + kPageSize - 1) / kPageSize, kPlanRowTiles);
    tokens = L;
    if (tiles <= most)
        return 1;
    const uint32_t n = min((tiles + most - 1) / most, (uint32_t)max_parts);
    tokens = (int)((((uint32_t)L + n - 1) / n + kCutLeast - 1) / kCutLeast * kCutLeast);
    return (L + tokens - 1) / tokens;
}

// Row b's items: {row, its length, tokens per partition, partition | partitions << 16}.  Returns the partitions.
template <int T>
__device__ __forceinline__ int plan_row(const PlanParams &p, int b)
{
    const auto length = [&](int i) { return max(min(p.seq_lens[i], p.max_seq_len), 0); };
    const int mine = length(b);
    uint32_t all = 0, none = 0;
    for (int i = threadIdx.x; i < p.B; i += T)
        all += min(((uint32_t)length(i) + kPageSize - 1) / kPageSize, kPlanRowTiles);
    group_sums<T>(all, none);
    uint32_t most = (uint32_t)ceilf((float)all * (kShareMost * p.heads_per_slot));
    if (most > kPlanTiles)
        most = max((uint32_t)ceilf((float)all * (kShareLeast * p.heads_per_slot)), kPlanTiles);
    most = max(most, (uint32_t)(kCutLeast / kPageSize));
    uint32_t ahead = 0, behind = 0;
    int tokens;
    for (int i = threadIdx.x; i < p.B; i += T) {
        const int L = length(i);
        const uint32_t n = plan_parts(L, most, p.max_parts, tokens);
        if (L > mine || (L == mine && i < b))
            ahead += n;
        else if (i != b)
            behind += n;
    }
    group_sums<T>(ahead, behind);
    const int n = plan_parts(mine, most, p.max_parts, tokens);
    // (The last row's workgroup also marks what is left of the list.)
    const uint32_t end = min(behind ? ahead + n : (uint32_t)p.max_items, (uint32_t)p.max_items);
    for (uint32_t j = threadIdx.x; ahead + j < end; j += T)
        p.items[ahead + j] = u32x4{j < (uint32_t)n ? (uint32_t)b : kNoRow, (uint32_t)mine, (uint32_t)tokens, j | (uint32_t)n << 16};
    return n;
}

} // namespace adr
