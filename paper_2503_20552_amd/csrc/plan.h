// The order and the cut of a pass of one workgroup per item, made on the device from the lengths.
//
// Longer items first, each row in equal partitions of a length that follows from the tokens the pass really has.  The
// hardware hands items out in their order as workgroups end, so what stands last decides how long the last
// compute units work alone: in the batch's own order that is any row's last partition, by descending
// length it is the shortest ones.  The length is the items': by the rows', the halves of a row that is just cut stand ahead of
// whole rows that are longer than they are (us a step, by rows and by items: 75 requests of median length 1500 116.4 and
// 114.6, 48 of 4000 180.2 and 177.5, 320 x 1 71.5 and 70.1, heads of 64 102.1 and 101.2, eight layers of 40 378.9 and 380.2,
// others within 0.5 %).  An fp8 cache by rows: 256 requests 187.7 and by items 189.1.  And a partition costs its workgroup about
// 6 us besides its tokens (8 where rows meet inside the pass): rows that are no burden to the tail stay whole.
//
// One workgroup per row, which reads all lengths: its place in the list follows from those alone, with no exchange
// between workgroups.  The list has no holes: with places left empty between the items (partitions
// that shrink as the work runs out, their places by a closed form) 256 requests of median length 1500 took
// 402 to 416 us, with this list 380 (in the batch's own order 407).
#pragma once

#include "adr_device.h"

namespace adr {

static_assert(kPlanTile == kPageSize && kPlanGrain == kCutLeast, "");

constexpr uint32_t kNoRow = 0xffffffffu; // in place of an item's row: past the last item
constexpr uint32_t kInTurn = 1u << 31; // beside it: the kv-heads go in turn (decode_mfma.hip)

// Over a workgroup of T threads, in every thread: the sums of v[0] to v[N - 2], and v[N - 1] by `op` (from 0 on).
template <int T, int N, typename Op>
__device__ __forceinline__ void group_reduce(uint32_t (&v)[N], Op op)
{
    const auto add = [&](uint32_t (&to)[N], int i, uint32_t x) { to[i] = i + 1 < N ? to[i] + x : op(to[i], x); };
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int i = 0; i < N; ++i)
            add(v, i, (uint32_t)__shfl_xor((int)v[i], off));
    if constexpr (T > 64) {
        __shared__ uint32_t parts[T / 64][N];
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int i = 0; i < N; ++i)
                parts[threadIdx.x / 64][i] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v[i] = 0;
#pragma unroll
            for (int w = 0; w < T / 64; ++w)
                add(v, i, parts[w][i]);
        }
    }
}

// Row b's items, {row, its length, tokens per partition, partition | partitions << 16}, and the words its partitions'
// arrivals are counted in, or their number for the merge kernel.
template <int T>
__device__ __forceinline__ void plan_row(const PlanParams &p, int b)
{
    const auto length = [&](int i) { return max(min(p.seq_lens[i], p.max_seq_len), 0); };
    const int mine = length(b);
    uint32_t lengths[3] = {0, 0, 0}; // all tiles, rows with tokens, the longest row's tiles
    for (int i = threadIdx.x; i < p.B; i += T) {
        const uint32_t tiles = plan_tiles(length(i));
        lengths[0] += tiles;
        lengths[1] += tiles > 0;
        lengths[2] = max(lengths[2], tiles);
    }
    group_reduce<T>(lengths, [](uint32_t x, uint32_t y) { return max(x, y); });
    const PlanCut cut = plan_cut(p.rule, lengths[1], lengths[0], lengths[2]);
    const auto parts = [&](int L, int &tokens, int &key) {
        const uint32_t n = plan_parts(L, cut, p.rule.max_parts, tokens);
        key = p.by_items ? tokens : L;
        return n;
    };
    int tokens, key;
    const uint32_t n = parts(mine, tokens, key);
    uint32_t around[2] = {0, 0}; // items ahead of the row's and behind them
    for (int i = threadIdx.x; i < p.B; i += T) {
        int its_tokens, its_key;
        const uint32_t its = parts(length(i), its_tokens, its_key);
        if (its_key > key || (its_key == key && i < b))
            around[0] += its;
        else if (i != b)
            around[1] += its;
    }
    group_reduce<T>(around, [](uint32_t x, uint32_t y) { return x + y; });
    const uint32_t ahead = around[0], behind = around[1];
    if (ahead + n > (uint32_t)p.max_items && threadIdx.x == 0) // (no lengths do that: plan_places)
        record_out_of_bounds(p.bounds, 4, b, ahead + n, p.max_items);
    // (The last row's workgroup also marks what is left of the list.)
    const uint32_t row = b | (lengths[0] >= p.turn_tiles ? kInTurn : 0u);
    const uint32_t end = min(behind ? ahead + n : (uint32_t)p.max_items, (uint32_t)p.max_items);
    for (uint32_t j = threadIdx.x; ahead + j < end; j += T)
        p.items[ahead + j] = u32x4{j < n ? row : kNoRow, (uint32_t)mine, (uint32_t)tokens, j | n << 16};
    if (p.part_counts && threadIdx.x == 0)
        p.part_counts[b] = n;
    if (p.arrivals && n > 1)
        for (int i = threadIdx.x; i < p.heads; i += T)
            p.arrivals[((int64_t)b * p.heads + i) * kArrivalWords] = 0u;
}

} // namespace adr
