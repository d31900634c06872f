// How the rows of a planned pass (plan.h) are cut: plain arithmetic, the same for the host that sizes the list and the
// device that fills it.
#pragma once

#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define ADR_BOTH __host__ __device__ __forceinline__
#else
#define ADR_BOTH inline
#endif

namespace adr {

constexpr int kPlanTile = 16, kPlanGrain = 128; // tokens of a tile; two tiles for each of four waves
constexpr int kSlots = 768; // workgroups the chip holds at once, three to a compute unit

// Tiles of a partition, as a share of what a slot has to do if all do the same: kShareMost of it, or, where that
// is more than kPlanTiles, as little as kShareLeast (a pass of few and very long rows must be cut
// somewhere).  us a step with shares of 0.5 / 0.75 / 1 / 1.25 / 1.5 / 2: 128 requests x 8 kv-heads, heavy-tailed
// lengths 77 / 74 / 72 / 69 / 73 / 70, 160 of up to 3000 tokens 174 / 172 / 167 / 164 / 164 / 166, 256 of
// median length 1500 385 / 380 / 380 / 380 / 379 / 384.
// Passes that the resident kernel served, of many rows: up to kManyTiles (at 256 they fell behind it; us a step, resident, 256
// and 512: 512 requests of 5000 tokens 1636 1670 1611, of median 5000 2187 2174 2145, 256 of 8000 1320 1329 1295, of median
// 4000 982 963 953, of median 1500 400 374 371).  Others not: 24 requests x 32 kv-heads, one of 131072 tokens, 369 and
// 403, 100 x 8 of 9000 616 and 629, fp8 256 of 6000 528 and 531.
constexpr uint32_t kPlanTiles = 256, kManyTiles = 512;
constexpr float kShareMost = 1.25f, kShareLeast = 0.125f;

// With fewer rows than places most rows are cut, and long ones must not stand alone at the end: partitions of
// kFewShare and no less than kFewTiles, kFewParts of a row as long as none is longer than kFewLong.  Rows are merged
// by a kernel of their own here: nearly every item would keep its place until it is counted (a step of 37
// requests x 8 kv-heads 49 and 52 us).
// Rows of one length, or nearly (the longest no more than kFewEven times the mean; empty rows, which fill up a recorded
// batch, are no part of it), come in rounds whatever their order.  They are cut as without a plan, into no more than
// kEvenItems, unless longer partitions fill at least half of a last round that is not the first (us a step, cut as without a
// plan and in longer partitions, rounds of those: 33 of 6000 tokens 142 and 147, 1.4; two layers of 16 in a batch of 64 153 and
// 162, 0.8; 48 in a batch of 64 420 and 412, 1.5; 51 of 4956 182 and 174, 1.6; 80 of 4000 225 and 211, 1.7; 60 of 7121 308 and
// 292, 1.9).  An fp8 cache is behind in longer ones throughout (50 of 7000 134 and 140, 1.6; 55 of 7538 158 and 160, 1.7).
// us a step, in the batch's order and planned: eight layers of 40 requests of median length 1000, replayed, 413 and
// 389, 128 of median 1500, heads of 64, 111 and 107, 75 of the same, pages of 64, 125 and 122, 80 of heavy-tailed
// lengths 61.5 and 54.
constexpr uint32_t kFewTiles = 16, kFewParts = 5, kEvenItems = 4800;
constexpr float kFewShare = 0.75f, kFewLong = 2.f, kFewEven = 1.1f;

// Tiles of a row that count, and rows of a pass: their tiles add up in 32 bits.  (More rows are not planned.)
constexpr uint32_t kPlanRowTiles = 1 << 20;
constexpr int kPlanRows = 2048;
ADR_BOTH uint32_t plan_tiles(int L)
{
    const uint32_t tiles = ((uint32_t)L + kPlanTile - 1) / kPlanTile;
    return tiles < kPlanRowTiles ? tiles : kPlanRowTiles;
}

// What the host knows of a pass.
struct PlanRule {
    int few;              // fewer rows than the chip holds workgroups: cut by kFew...,
    int even_tiles;       //   rows of one length in partitions of that many tiles,
    int fill_rounds;      //   or in longer ones that fill a round (a bf16 cache)
    int max_parts;        // partitions of a row at most
    uint32_t whole;       // kPlanTiles or kManyTiles
    float heads_per_slot; // kv-heads (pairs of them) by the workgroups the chip holds
};

// Places in the list that can be taken, kv-heads counted once: one per row and one per whole partition of all tokens.
ADR_BOTH int64_t plan_places(int B, int H, int max_seq_len, const PlanRule &p)
{
    const int64_t tiles = (int64_t)B * plan_tiles(max_seq_len);
    const int64_t least = (int64_t)(kSlots / (kShareLeast * H)), most = (int64_t)(kSlots / (kShareMost * H));
    const int64_t long_ones = least < tiles / p.whole ? least : tiles / p.whole;
    const int64_t places = p.few ? (int64_t)(kEvenItems / H + 1) : most > long_ones ? most : long_ones;
    return (B + places + 2 + 7) / 8 * 8;
}

ADR_BOTH uint32_t larger(uint32_t a, uint32_t b) { return a > b ? a : b; }
ADR_BOTH uint32_t smaller(uint32_t a, uint32_t b) { return a < b ? a : b; }

// How the rows of a pass are cut: in partitions of `most` tiles or less, but no more than `parts` of them as long as
// those have `longest` tiles or less.
struct PlanCut {
    uint32_t most, longest, parts;
    uint32_t grain; // tokens a partition is a multiple of, a power of two: two tiles for each of four waves, or one
};
// Partitions of a row of that many tiles.
ADR_BOTH uint32_t plan_parts(uint32_t tiles, const PlanCut &c)
{
    const uint32_t n = (tiles + c.most - 1) / c.most;
    return c.parts ? smaller(n, larger(c.parts, (tiles + c.longest - 1) / c.longest)) : n;
}
// `rows` with tokens, which have `all` tiles.
ADR_BOTH PlanCut plan_cut(const PlanRule &p, int rows, uint32_t all, uint32_t longest_row)
{
    const float slot = (float)all * p.heads_per_slot;
    PlanCut c = {(uint32_t)ceilf(kShareMost * slot), 1u, 0u, (uint32_t)kPlanGrain};
    if (p.few) {
        c.most = larger((uint32_t)ceilf(kFewShare * slot), kFewTiles);
        c.longest = larger((uint32_t)ceilf(kFewLong * slot), c.most);
        c.parts = kFewParts;
        if ((float)longest_row * (float)rows <= kFewEven * (float)all) {
            const uint32_t even = larger((uint32_t)p.even_tiles, (uint32_t)ceilf((float)longest_row * (float)rows * (p.heads_per_slot * kSlots / kEvenItems)));
            const uint32_t n = plan_parts(longest_row, c);
            const float rounds = (float)(rows * (int)n) * p.heads_per_slot;
            if (!p.fill_rounds || longest_row <= n * even || rounds < 1.f || rounds - floorf(rounds) < 0.5f) {
                c.most = even;
                c.parts = 0;
                c.grain = kPlanGrain / 2;
            }
        }
        return c;
    }
    if (c.most > p.whole)
        c.most = larger((uint32_t)ceilf(kShareLeast * slot), p.whole);
    c.most = larger(c.most, (uint32_t)(kPlanGrain / kPlanTile));
    return c;
}

// Row of L tokens: its partitions, and the tokens of each.
ADR_BOTH int plan_parts(int L, const PlanCut &c, int max_parts, int &tokens)
{
    const uint32_t tiles = plan_tiles(L);
    tokens = L;
    if (tiles <= c.most)
        return 1;
    const uint32_t n = smaller(plan_parts(tiles, c), (uint32_t)max_parts);
    tokens = (int)((((uint32_t)L + n - 1) / n + c.grain - 1) & ~(c.grain - 1));
    return (int)(((uint32_t)L + tokens - 1) / tokens);
}

} // namespace adr
