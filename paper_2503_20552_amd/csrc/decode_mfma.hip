// Decode attention with the QK^T and PV contractions on the matrix cores
// (bf16 or fp8 cache; d = 128 with any group size G <= 16, and d = 64 with two kv-heads taken together).
//
// One workgroup of 4 waves (8 for some whole rows) per (request, kv-head, partition); wave w streams
// tiles w, w+4, ... .  A tile is 16 tokens = one MFMA tile edge (a cache page is one or
// more of them).  Lane l is (r, j) = (l % 16, l / 16).
//
// What bounds it: HBM while it runs (three workgroups to a compute unit keep 96 to 192 KB in flight),
// and per item a chain of round trips (length, page table, first tile) of about 2 us that the other
// two workgroups cover only in part.  Three workgroups need the kernel in 168 registers, which the
// compiler does not try for by itself (159 + 36 accumulation registers, two workgroups): 410 against
// 424 us at 256 requests x 8 kv-heads in partitions of 512 tokens, 71 against 76 us at 128
// requests of 64 heads.  A resident variant (the same loop, three workgroups per unit taking
// items in a fixed rotation from a list of the partitions that exist) was slower: 424 against 412
// and 209 against 208 us; it saves the empty workgroups and pays the chain in series.
//
// d = 64 (PAIR): the rows of two neighbouring kv-heads of a token lie side by side, 256 bytes like one
// row of d = 128.  An item is both heads; their query heads fill the columns of one tile, the first
// kv-head's in columns 0 .. G-1, contracted with chunks 0 .. 7 of a row, the second's in columns
// G .. 2G-1, contracted with chunks 8 .. 15.  P V is taken over the whole row and each head keeps its
// half.  (113 against 121 us for the vector-ALU kernel at 128 requests, 8 kv-heads, G = 4; small
// passes of groups of one are that kernel's.)
//
// fp8 cache: two tiles a step, K and V both by direct-to-LDS loads into one stage of 8 KB per wave, which
// is copied to registers and refilled at once; K is widened to bf16 after the LDS read and meets the
// query as it is (exact: error against 64 bits 5e-6, the resident kernel's two-term fp8 query
// 1.7e-5), V comes out of the LDS transposed (mfma_fp8.h).  The scales of a wave's pages arrive with
// one gather per sixty-four tiles, not page by page.  Measured against the resident kernel, which
// served fp8 before: 9 against 37 us at one request of 2000 tokens, 35 against 60 at 40 requests,
// 130 against 146 at 128, 53 against 79 with groups of eight; heads of 64 (before: vector ALUs)
// 70 against 127.  Three workgroups to a compute unit: four are slower (142 against 130 us at 128
// requests), and so are a second stage with two (132) and three tiles in flight with three (132).
//
// QK^T  S[token][head] = K[16 x 128] * Q^T[128 x 16] as four
//       v_mfma_f32_16x16x32_bf16.  The A operand wants lane (r, j) to hold 16
//       bytes of token r -- sixteen different rows per quarter wave, a pattern
//       the vector memory path serves one lane at a time.  So the K tile takes
//       the coalesced route: four loads that each fetch four complete 256-byte
//       rows and deposit them directly in LDS (no VGPRs), and the operand is
//       then read from LDS.  Row t is stored with its sixteen 16-byte chunks
//       XOR-permuted by t (slot s holds chunk s ^ t), which makes the operand
//       reads -- sixteen rows, same chunk -- hit sixteen different bank groups.
//       Step kk, lane (r, j) contracts chunk kk*4 + j; Q^T (the B operand,
//       head r, loaded once) uses the same order.  Columns past the last
//       head repeat it and are never stored.  Each wave owns two such tiles (the page being consumed and
//       the page in flight).
//       Result layout: lane (r, j) holds S[token 4j+i][head r], i = 0..3.
// softmax  per lane over its 4 tokens, running max shared across the four
//       lane groups j by two wave shuffles; fp32 throughout, base 2.
// PV    O[head][dcol] += P[16 x 16 tokens] * V[16 tokens x 16 dcols], eight
//       v_mfma_f32_16x16x16_bf16 per page (one per e = 0..7, dcol = 8r + e).
//       The S layout above IS the A-operand layout (row = head r, k = token
//       4j+i), so P never moves between lanes.  P is split into a bf16 head
//       and a rounded bf16 remainder (two MFMAs), so the weights keep 17 significant
//       bits (PAIR: three terms, all 24).  V is loaded in its natural layout -- lane (r, j), load u: the 16
//       bytes of token 4j+u at chunk r, i.e. four complete 256-byte rows per
//       instruction -- and the B operand (k = token 4j+u, n = r) for column
//       set e is assembled from those four registers with byte permutes.
//       Result layout: lane (r, j) holds O[head 4j+i][8r + e].
#include "mfma_fp8.h"
#include "plan.h"

#include <algorithm>
#include <type_traits>

namespace adr {

__device__ __forceinline__ void read_k_operand(u32x4 (&ka)[4], const char *ktile,
                                               const uint32_t (&k_read)[4])
{
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
        ka[kk] = *(const u32x4 *)(ktile + k_read[kk]);
}

// Workgroups are numbered row by row: the kv-heads of a partition together (see the kernel),
// then the row's partitions, `stride` of them; a workgroup takes every stride-th partition of its
// row from its own on and leaves at once when the row has none for it.  The grid is sized from
// the caller's bound on the lengths, not from the lengths, so most workgroups may find nothing.
// Two things were measured on the 70B-shaped workload (1 712 items of 13 312 workgroups, 73 us):
// (1) the hardware hands consecutive workgroups to its compute units in turn, so when the number of
// workgroups per row divides the units evenly, a row's few real workgroups fall on the same units
// row after row: 123 us with 16 partitions per row in the grid, 152 us with 64.  The stride is
// therefore odd.  (2) Workgroups that find nothing still cost 0.2 to 0.4 nanoseconds each, and a bound far
// above the lengths makes many of them: the stride stops at 33, or at what makes 68000 workgroups, though
// not below nine, and rows with more partitions have their workgroups loop.  (us per step, 300 tokens a row under a
// bound of 131072, stride 33 and this: 4096 rows fp8 117 and 92, 3840 rows bf16 119 and 112.  Nine for
// everybody is better still for those, 81, but rows that are long then wait for their workgroups: 40
// requests, one in ten of 20000 tokens, 85 against 70.)
// (Where there are few rows, a long one needs its workgroups: the limit is then 4096 of them in all.)
static int grid_stride(int64_t rows, int max_parts)
{
    const int64_t most = std::max<int64_t>(std::max<int64_t>(std::min<int64_t>(33, 68000 / rows), 9), 4096 / rows);
    const int n = (int)std::min<int64_t>(max_parts, most);
    return n > 1 ? (n | 1) : n;
}

constexpr unsigned kTurnRowTokens = 163840; // from that many on, if all rows were as long, its kv-heads go in turn (see the kernel)
constexpr int kNoMore = 1 << 20; // added to a partition's number: past any row's last

constexpr int kChiplets = 8; // of the GPU; the hardware deals workgroups out to them in turn

constexpr int kWaveBytes = kStages * kTileBytes; // LDS of one wave: its K tiles, then its share of the result

// The tiles of one wave in one partition: first, first + NW, ...  Their table entries arrive with one
// vector load, lane n holding the wave's n-th tile, and reach the scalar unit by a lane read; a
// second register holds the next sixty-four.
template <int NW, bool FP8, bool PAIR>
struct TileIds {
    const int32_t *row; // the row's table
    int first, count, last_entry, shift;
    int now, next;
    // fp8: the scales of the tiles' pages, K and V, of the one kv-head or of both of a pair
    static constexpr int SCALES = FP8 ? (PAIR ? 4 : 2) : 1;
    float scale_now[SCALES], scale_next[SCALES];

    __device__ __forceinline__ int load(int n) const
    {
        // (a lane past the last tile reads the last one's entry; never outside the row's table)
        return row[min((first + min(n, max(count - 1, 0)) * NW) >> shift, last_entry)];
    }
    // Scales of the pages `entry` of tiles n (one to a lane); zero past the last tile.
    __device__ __forceinline__ void load_scales(const DecodeParams &p, int h, int entry, int n, float (&to)[SCALES]) const
    {
        if constexpr (FP8) {
#pragma unroll
            for (int i = 0; i < SCALES; ++i)
                to[i] = 0.f;
            if (n < count) {
                const int64_t at = (int64_t)clamp_page(entry, p.num_pages) * p.Hkv + (PAIR ? 2 * h : h);
#pragma unroll
                for (int i = 0; i < SCALES / 2; ++i) {
                    to[2 * i] = p.k_scale[at + i];
                    to[2 * i + 1] = p.v_scale[at + i];
                }
            }
        }
    }
    __device__ __forceinline__ void start(const DecodeParams &p, int b, int first_tile, int tiles)
    {
        row = p.block_table + (int64_t)b * p.max_pages;
        first = first_tile;
        count = tiles;
        last_entry = p.max_pages - 1;
        shift = p.page_shift;
        now = load(threadIdx.x & 63);
        next = 0;
    }
    // Entry of tile n; called for n = 0, 1, 2, ... in turn, in front of the tile's own loads.
    __device__ __forceinline__ int entry(const DecodeParams &p, int h, int n)
    {
        if ((n & 63) == 0) {
            if (n) {
                asm volatile("" : "+v"(next)); // it is waited for here and not at every lane read below
                now = next;
                if constexpr (FP8) {
                    settle(scale_next);
#pragma unroll
                    for (int i = 0; i < SCALES; ++i)
                        scale_now[i] = scale_next[i];
                }
            }
            if (count > n + 64)
                next = load(n + 64 + (threadIdx.x & 63));
        }
        if (FP8 && (n & 63) == 32 && count > n + 32) {
            asm volatile("" : "+v"(next));
            load_scales(p, h, next, n + 32 + (threadIdx.x & 63), scale_next);
        }
        return __builtin_amdgcn_readlane(now, n & 63);
    }
    // Loads of scales are waited for here.
    static __device__ __forceinline__ void settle(float (&s)[SCALES])
    {
#pragma unroll
        for (int i = 0; i < SCALES; ++i)
            asm volatile("" : "+v"(s[i]));
    }
    // fp8: scale i of tile n (0: K, 1: V; a pair's second kv-head: 2, 3).
    __device__ __forceinline__ float scale(int i, int n) const
    {
        return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scale_now[i]), n & 63));
    }
};

// ---- fp8 cache: two tiles (32 tokens) at a time ------------------------------------------------

// Loads of one tile of K or V for one row of D bytes per token: two, of eight rows each; slot c of row t
// holds the row's 16-byte chunk c ^ (t & 7), so that the transposed reads below hit different banks.
__device__ __forceinline__ void load_tile_fp8(char *tile, __amdgpu_buffer_rsrc_t rsrc, const uint32_t (&lane_off)[2])
{
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(tile + i * 1024), 16,
                                                 lane_off[i], 0, 0, kStreamOnce);
    asm volatile("" ::: "memory");
}

// S = K Q^T of one tile, K widened to bf16 (exact).
template <bool PAIR>
__device__ __forceinline__ f32x4 scores_fp8(const u32x2 (&k8)[4], const u32x4 (&qb)[4], bool upper)
{
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, s_up = s;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        f32x4 &acc = PAIR && kk >= 2 ? s_up : s;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fp8x8_to_bf16x8(k8[kk])),
                                                      __builtin_bit_cast(bf16x8, qb[kk]), acc, 0, 0, 0);
    }
    return PAIR && upper ? s_up : s;
}

// One online-softmax step over two tiles and O += P V.
//   sc   base-2 scores of tokens tok + i of the first tile and tok_b + i of the second (i = 0 .. 3)
//   v8   V bytes, transposed: for column block e, four tokens of the first tile, then of the second
template <bool PAIR>
__device__ __forceinline__ void attend_two_fp8(WaveState &st, float (&sc)[8], u32x2 (&v8)[8], float vs_a, float vs_b,
                                               int tok, int tok_b, int t1, int j)
{
    if (tok_b - 4 * j + kPageSize > t1) { // tokens past the end (the second tile as a whole may lie there)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (tok + i >= t1)
                sc[i] = -INFINITY;
            if (tok_b + i >= t1)
                sc[4 + i] = -INFINITY;
        }
        const uint32_t keep_a = tail_mask_fp8(tok, t1), keep_b = tail_mask_fp8(tok_b, t1);
#pragma unroll
        for (int e = 0; e < 8; ++e) { // their rows may hold anything: keep them out of P V
            v8[e][0] &= keep_a;
            v8[e][1] &= keep_b;
        }
    }
    float bm = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
    bm = max_across_rows(bm);
    if (__any(bm > st.m + kMaxSlack)) {
        const float mn = fmaxf(st.m, bm);
        const float alpha = fast_exp2(st.m - mn);
        st.m = mn;
        st.l *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = __shfl(alpha, 4 * j + i);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                st.o[e][i] *= a;
        }
    }
    constexpr int TERMS = PAIR ? 3 : 2; // (see attend_page)
    u32x4 w[TERMS];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float p0 = fast_exp2(sc[2 * k] - st.m), p1 = fast_exp2(sc[2 * k + 1] - st.m);
        st.l += p0;
        st.l += p1;
        p0 *= k < 2 ? vs_a : vs_b;
        p1 *= k < 2 ? vs_a : vs_b;
        uint32_t terms[TERMS];
        split_weights<TERMS>(p0, p1, terms);
#pragma unroll
        for (int t = 0; t < TERMS; ++t)
            w[t][k] = terms[t];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const u32x4 v = fp8x8_to_bf16x8(v8[e]);
#pragma unroll
        for (int t = 0; t < TERMS; ++t)
            st.o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[t]),
                                                              __builtin_bit_cast(bf16x8, v), st.o[e], 0, 0, 0);
    }
}

// The kernel's argument block, read where it is asked for: what a partition's end needs of the parameters does not
// occupy scalar registers through the loop over its tiles (held from the start they did not fit where rows
// meet: 25 to 60 of them went through vector lanes, 0.5 to 1 us per launch).
typedef const __attribute__((address_space(4))) DecodeParams *LateParams;
__device__ __forceinline__ LateParams late_params_of_append()
{
    LateParams p = (LateParams)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// ---- a step's new tokens --------------------------------------------------------------------------

// A pass that appends the step's new tokens itself (APPEND; up to 64 requests): where a tile belongs to a page that any request
// appends to, the new token takes its slot's place in the wave's copy of the tile, and the wave that attends a row's last tile
// also stores it in the cache.  So every row sees every new token, whichever requests share pages, as if the append had
// come first, and no launch of its own is waited for.  The pages stand in a register, a request to a lane, and are compared with each
// tile's.  (The answer is nearly always no, and the compiler is told so: 24 requests x 4 kv-heads of 64 of an fp8 cache in two partitions of
// 2048 tokens 28.8 us, 27.9 so.  Fetched for each row with the first loads of its items, the new tokens came later: 9.4 and 9.9 us for
// three requests of 300 tokens; asked for ahead of the row's last tile, no sooner; at 256 requests' pages in four registers: the same.)
template <bool FP8, bool PAIR, int NW>
struct NewTokens {
    int page; // of the new token of the lane's request, or -1
    int slot; // in that page

    __device__ __forceinline__ void ask(const DecodeParams &p, int length)
    {
        const int b = threadIdx.x & 63;
        page = -1;
        slot = (length - 1) & ((kPageSize << p.page_shift) - 1);
        if (b < p.B && length > 0 && length <= p.max_seq_len) { // (append_position, append_page)
            const int at = (length - 1) >> (4 + p.page_shift);
            page = p.block_table[(int64_t)b * p.max_pages + at];
            if ((unsigned)page >= (unsigned)p.num_pages) {
                if (blockIdx.x == 0 && threadIdx.x < 64)
                    record_out_of_bounds(p.bounds, 3, b, at, page);
                page = -1;
            }
        }
    }
    // The pages are waited for here (behind the first tile's loads).
    __device__ __forceinline__ void settle() { asm volatile("" : "+v"(page)); }
    // No load beside the tiles' is pending where their loop goes on: the compiler would otherwise wait there, for every
    // tile, for all loads in flight (20 requests in whole rows 26.6 us a step, 35.6 so).  The stores come behind that wait: nothing
    // waits for them (8 fp8 requests of 300 tokens 7.8 us, 7.6 so).
    static __device__ __forceinline__ void wait_for_all_loads()
    {
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0), no other counter
#endif
    }
    // put(request, slot in the page, row `row` is among them) for each slot of that page that a new token goes to.  Where several
    // requests name one slot (rows that fill up a batch may all lie on one page) the last one's token stands for all of them: one
    // after the other, 64 of them took 23 us instead of 7, 16 of an fp8 cache 31 instead of 11.
    template <typename Put>
    __device__ __forceinline__ void each(int of, int row, Put put) const
    {
        for (uint64_t m = __ballot(page == of); m;) {
            const int in_page = __builtin_amdgcn_readlane(slot, __ffsll((unsigned long long)m) - 1);
            const uint64_t same = __ballot(page == of && slot == in_page);
            put(63 - __clzll((long long)same), in_page, (same >> row & 1) != 0);
            m &= ~same;
        }
    }

    // bf16: a tile of the pool, K in LDS and V in registers (load_page).  last: it is row b's last tile.
    __device__ __forceinline__ void put_bf16(LateParams p, int h, int tile, char *ktile, PageRegs &regs, int row, bool last) const
    {
        const int lane = threadIdx.x & 63, r = lane & 15, j = lane >> 4;
        const int H = PAIR ? p->Hkv >> 1 : p->Hkv;
        each(tile >> p->page_shift, row, [&](int b, int in_page, bool own) {
            if (in_page / kPageSize != (tile & ((1 << p->page_shift) - 1)))
                return;
            const int slot = in_page % kPageSize;
            const int64_t src = (int64_t)b * p->new_row_stride + h * D + r * 8;
            const u32x4 k = *(const u32x4 *)(p->k_new + src), v = *(const u32x4 *)(p->v_new + src);
            if (j == 0)
                *(u32x4 *)(ktile + slot * (D * 2) + ((r ^ slot) * 16)) = k;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u == (slot & 3) && j == slot >> 2)
                    regs.v[u] = v;
            wait_for_all_loads();
            if (own && last && j == 0) {
                const int64_t dst = (((int64_t)tile * kPageSize + slot) * H + h) * D + r * 8;
                *(u32x4 *)((uint16_t *)p->k_cache + dst) = k;
                *(u32x4 *)((uint16_t *)p->v_cache + dst) = v;
            }
        });
    }

    // fp8: tile number t of a stage (K, K, V, V), and the scales its scores and weights take.  A token in slot 0 of its
    // page also sets the page's scales, for all tiles of the page.
    __device__ __forceinline__ void put_fp8(LateParams p, int h, int tile, int t, char *stage, float &ks, float &vs, int row, bool last) const
    {
        const int lane = threadIdx.x & 63;
        const int H = PAIR ? p->Hkv >> 1 : p->Hkv;
        const bool upper = PAIR && (lane & 15) >= p->G;
        const int of = tile >> p->page_shift;
        each(of, row, [&](int b, int in_page, bool own) {
            const bool here = in_page / kPageSize == (tile & ((1 << p->page_shift) - 1));
            if (!here && in_page != 0)
                return;
            const int slot = in_page % kPageSize;
            const bool keep = own && last;
            const int64_t src = (int64_t)b * p->new_row_stride + h * D + lane * 2;
            float scale[2];
            uint32_t bytes[2];
            const int64_t scale_at = (int64_t)of * p->Hkv + (PAIR ? 2 * h + lane / 32 : h);
#pragma unroll
            for (int which = 0; which < 2; ++which) {
                const uint32_t two = *(const uint32_t *)((which ? p->v_new : p->k_new) + src);
                const float x0 = bf16_lo(two), x1 = bf16_hi(two);
                if (in_page == 0) {
                    float amax = fmaxf(fabsf(x0), fabsf(x1));
#pragma unroll
                    for (int off = 1; off < (PAIR ? 32 : 64); off <<= 1)
                        amax = fmaxf(amax, __shfl_xor(amax, off));
                    scale[which] = new_page_scale(amax);
                    const float s0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scale[which]), 0));
                    const float s1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scale[which]), 32));
                    (which ? vs : ks) = upper ? s1 : s0;
                } else {
                    scale[which] = ((const float *)(which ? p->v_scale : p->k_scale))[scale_at];
                }
                if (here) {
                    const float inv = 1.0f / scale[which];
                    bytes[which] = f32_to_e4m3(x0 * inv) | (f32_to_e4m3(x1 * inv) << 8);
                    *(uint16_t *)(stage + (2 * which + t) * kFp8TileBytes + slot * D + (((lane >> 3) ^ (slot & 7)) * 16) + (lane & 7) * 2) = (uint16_t)bytes[which];
                }
            }
            wait_for_all_loads();
            if (keep)
#pragma unroll
                for (int which = 0; which < 2; ++which) {
                    if (in_page == 0 && lane % (PAIR ? 32 : 64) == 0)
                        ((float *)(which ? p->v_scale : p->k_scale))[scale_at] = scale[which];
                    *(uint16_t *)((uint8_t *)(which ? p->v_cache : p->k_cache) + (((int64_t)tile * kPageSize + slot) * H + h) * D + lane * 2) = (uint16_t)bytes[which];
                }
        });
    }
};

// Where a workgroup's item comes from and where the partitions of a split row meet.  Variants of their own, because
// what one of them needs costs the others scalar registers: with all in one kernel a step of one
// request took 10.6 us instead of 10.1.
enum class Items {
    by_row,      // numbered by row and stride; the partitions are merged by a kernel of its own
    by_row_meet, // numbered the same; the wave that brings a row's last partition merges it
    planned_meet, // listed (plan.h), merged the same
    planned      // listed, merged by the kernel of its own
};

template <Items ITEMS>
__device__ __forceinline__ LateParams late_params()
{
    LateParams p = (LateParams)__builtin_amdgcn_kernarg_segment_ptr();
    if (ITEMS == Items::by_row_meet || ITEMS == Items::planned_meet)
        asm volatile("" : "+s"(p));
    return p;
}

// ---- merging a split row inside the pass -----------------------------------------------------------

// Partial results that another workgroup reads in the same launch: written through to, and read from, the
// memory all chiplets see (sc1, device scope), so that neither side has to write back or invalidate
// an L2.
constexpr int kDeviceScope = 16;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t partial_rsrc(const float *base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ void store_shared(f32x4 x, __amdgpu_buffer_rsrc_t rsrc, int offset)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rsrc, offset, 0, kDeviceScope);
}
__device__ __forceinline__ f32x4 load_shared(__amdgpu_buffer_rsrc_t rsrc, int offset)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, offset, 0, kDeviceScope));
}

// One wave's end of a partition of a split row.  In every partition's workgroup wave w holds the same elements of
// the row's result (four per thread and round), so the waves of a row meet one by one, without a
// barrier: a wave waits until its own partial results are in memory and counts itself in; true for the one that
// finds all others there.  Nobody waits for anybody.
// The counts lie in the call's workspace (not in `out`, which may be any memory a kernel can store to).  A planned pass has
// words of their own for them in `arrivals`.  Other passes may fill every place of the workspace: there a count takes
// the lse of the wave's first head in one place of its row (meet_place), and that partition's lse goes to the wave's
// word in the control area (meet_word), which whoever merges the row, or attends it whole, leaves zero.  Where there are
// more waves than words the counts themselves are bytes of the control area, neighbours in different lines: its four lines
// then take all arrivals of the pass one by one, 10 ns each (one request of 2000 tokens, 256 arrivals: 10.5 us, 9.9 with the
// counts in places of their own), so for rows of few partitions only.
template <int HD>
__device__ __forceinline__ int meet_index(LateParams p, int b, int h)
{
    const int H = HD == D ? p->Hkv : p->Hkv >> 1;
    return (b * H + h) * result_waves(p->G) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}
template <int HD>
__device__ __forceinline__ float *meet_word(LateParams p, int b, int h)
{
    return (float *)p->control + 1 + meet_index<HD>(p, b, h);
}
template <int HD, bool PLANNED>
__device__ __forceinline__ bool arrive(LateParams p, int b, int h, int first_head, int n_parts)
{
    const int head = first_head + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64 / (HD / 4);
    const bool bytes = !PLANNED && p->meet_bytes;
    const int i = bytes ? meet_index<HD>(p, b, h) : 0, shift = i / kMeetWords * 8;
    uint32_t *const count = PLANNED ? p->arrivals + ((int64_t)b * p->Hq + head) * kArrivalWords
                            : bytes ? p->control + 1 + i * 32 % kMeetWords
                                    : (uint32_t *)(p->part_lse + ((int64_t)b * p->max_parts + meet_place(head, p->meet_mask)) * p->Hq + head);
    asm volatile("s_waitcnt vmcnt(0)" ::"s"(count) : "memory"); // (the address is there by then)
    uint32_t before = 0;
    if ((threadIdx.x & 63) == 0)
        before = __hip_atomic_fetch_add(count, 1u << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before = __builtin_amdgcn_readfirstlane(before);
    asm volatile("" ::: "memory");
    const bool last = (bytes ? before >> shift & 0xffu : before) + 1 == (uint32_t)n_parts;
    if (bytes && last && (threadIdx.x & 63) == 0)
        __hip_atomic_fetch_sub(count, (uint32_t)n_parts << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}
// Where partition `part` of head `head` leaves its lse; `first`: it is the wave's first head.
template <int HD>
__device__ __forceinline__ float *lse_word(LateParams p, int b, int h, int part, int head, bool first)
{
    return first && !p->meet_bytes && part == meet_place(head, p->meet_mask)
               ? meet_word<HD>(p, b, h)
               : p->part_lse + ((int64_t)b * p->max_parts + part) * p->Hq + head;
}

// The wave's share of a row, merged from its partitions in a fixed order, whichever wave it is: in S slices of every
// S-th partition, CH of a slice loaded together, as lse_merge_kernel does it with S and CH (the same
// bits).
template <int HD, bool PLANNED, int NW, int S, int CH>
__device__ __forceinline__ void merge_share(LateParams p, int b, int h, int first_head, int heads, int n_parts)
{
    constexpr int QUADS = HD / 4;
    const int counted = first_head + (int)(threadIdx.x >> 6) * 64 / QUADS; // the wave's first head, whose lse stands elsewhere
    const bool moves = !PLANNED && !p->meet_bytes;
    float *const moved = meet_word<HD>(p, b, h);
    const int moved_from = !moves ? -1 : meet_place(counted, p->meet_mask); //   in that place (lse_word)
    for (int idx = threadIdx.x; idx < heads * QUADS; idx += NW * 64) {
        const int head = first_head + idx / QUADS;
        const int c4 = (idx % QUADS) * 4;
        float top[S], total[S];
        f32x4 acc[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            top[s] = -INFINITY;
            total[s] = 0.f;
            acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int i0 = s; i0 < n_parts; i0 += S * CH) {
                const int64_t row = ((int64_t)b * p->max_parts + i0) * p->Hq;
                const __amdgpu_buffer_rsrc_t o_rsrc = partial_rsrc(p->part_o + row * HD), lse_rsrc = partial_rsrc(p->part_lse + row);
                float ls[CH];
                f32x4 xs[CH];
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    ls[u] = -INFINITY;
                    xs[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (i0 + u * S < n_parts) {
                        const int at = u * S * p->Hq + head;
                        if (PLANNED)
                            ls[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(lse_rsrc, at * 4, 0, kDeviceScope));
                        else
                            ls[u] = __hip_atomic_load(head == counted && i0 + u * S == moved_from ? moved : p->part_lse + row + at,
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        xs[u] = load_shared(o_rsrc, (at * HD + c4) * 4);
                    }
                }
                float cm = -INFINITY;
#pragma unroll
                for (int u = 0; u < CH; ++u)
                    cm = fmaxf(cm, ls[u]);
                const float nt = fmaxf(top[s], cm);
                if (nt > -INFINITY) {
                    const float rs = fast_exp2((top[s] - nt) * kLog2e); // 0 when nothing was seen before
                    acc[s] *= rs;
                    total[s] *= rs;
#pragma unroll
                    for (int u = 0; u < CH; ++u) {
                        const float w = fast_exp2((ls[u] - nt) * kLog2e);
                        if (w > 0.f) {
                            acc[s] += w * xs[u];
                            total[s] += w;
                        }
                    }
                    top[s] = nt;
                }
            }
        }
        if constexpr (S > 1) {
            float all = top[0];
#pragma unroll
            for (int s = 1; s < S; ++s)
                all = fmaxf(all, top[s]);
            if (all > -INFINITY) {
                const float w0 = fast_exp2((top[0] - all) * kLog2e);
                acc[0] *= w0;
                total[0] *= w0;
#pragma unroll
                for (int s = 1; s < S; ++s) {
                    const float w = fast_exp2((top[s] - all) * kLog2e);
                    if (w > 0.f) {
                        acc[0] += w * acc[s];
                        total[0] += w * total[s];
                    }
                }
                top[0] = all;
            }
        }
        const f32x4 o = acc[0] * (total[0] > 0.f ? 1.f / total[0] : 0.f);
        const int64_t row = (int64_t)b * p->Hq + head;
        if (p->out_f32) {
            *(f32x4 *)((float *)p->out + row * HD + c4) = o;
        } else {
            u32x2 packed;
            packed[0] = f32_to_bf16(o[0]) | (f32_to_bf16(o[1]) << 16);
            packed[1] = f32_to_bf16(o[2]) | (f32_to_bf16(o[3]) << 16);
            *(u32x2 *)((uint16_t *)p->out + row * HD + c4) = packed;
        }
        if (p->lse && c4 == 0)
            p->lse[row] = total[0] > 0.f ? top[0] + fast_log2(total[0]) * kLn2 : -INFINITY;
    }
    if (moves && (threadIdx.x & 63) == 0) // (for later launches: not written through, which would be waited for, 0.2 us)
        *moved = 0.f;
}

template <bool FP8, bool PAIR, int NW, Items ITEMS, bool APPEND>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW == 4 ? 3 : 2, NW == 4 ? 3 : 8)))
void decode_mfma_kernel(const DecodeParams p)
{
    constexpr bool kMeet = ITEMS == Items::by_row_meet || ITEMS == Items::planned_meet;
    constexpr int HD = PAIR ? D / 2 : D;           // elements of one head
    const int G = p.G;
    const int H = PAIR ? p.Hkv >> 1 : p.Hkv;       // rows of D elements per token
    const int R = PAIR ? 2 * G : G;                // query heads that use one of them

    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    float *ml = (float *)(lds_raw + NW * kWaveBytes); // [NW][16][2]: running max, denominator of each head

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15;
    const int j = lane >> 4;
    const bool upper = PAIR && r >= G;

    const int stride = ITEMS >= Items::planned_meet ? kNoMore : p.grid_stride;
    int length = 0; // of the lane's request (asked for before anything else is waited for)
    if constexpr (APPEND)
        length = p.seq_lens[min(lane, p.B - 1)];
    // Which (row of the cache h, partition, request) this workgroup starts with.  Consecutive workgroups go
    // to the eight chiplets in turn, those of a chiplet to its four shader engines.  bf16: kv-heads fastest, so that a
    // page's heads are read side by side by different chiplets.  fp8: the kv-heads of a partition one after the other
    // on one chiplet -- with eight kv-heads the other order gives a chiplet the same 128 bytes of every 1024, and it
    // costs 250 against 221 us at 255 requests, 130 against 116 at 128, 141 against 129 at 60 requests of 32 kv-heads.
    unsigned unit, h;
    if constexpr (FP8) {
        const unsigned in_chiplet = blockIdx.x / kChiplets;
        h = in_chiplet % H;
        unit = in_chiplet / H * kChiplets + blockIdx.x % kChiplets;
    } else {
        h = blockIdx.x % H;
        unit = blockIdx.x / H;
    }
    typedef const __attribute__((address_space(4))) int32_t *const_ptr;
    int b, L, pt, first_part, n_parts;
    bool in_turn;
    if constexpr (ITEMS >= Items::planned_meet) {
        const u32x4 item = ((const __attribute__((address_space(4))) u32x4 *)p.items)[unit];
        if (item[0] == kNoRow)
            return;
        b = item[0] & ~kInTurn;
        in_turn = item[0] & kInTurn;
        L = item[1];
        pt = item[2];
        first_part = item[3] & 0xffffu;
        n_parts = item[3] >> 16;
    } else {
        first_part = unit % stride;
        b = unit / stride;
        if (FP8 && b >= p.B)
            return;

        L = max(min(((const_ptr)p.seq_lens)[b], p.max_seq_len), 0);
        // No partition is shorter than `least`: without dividing, most workgroups that have none leave here
        // (64 K of them: 77 us with the divisions, 65 without).
        const unsigned least = p.cut > 0 ? p.cut : p.partition_tokens;
        if (first_part > 0 && first_part * least >= (unsigned)L)
            return;
        pt = row_partition(L, p.partition_tokens, p.max_parts, p.cut, p.cut_share);
        n_parts = parts_of(L, pt);
        if (first_part >= n_parts)
            return;
        const unsigned rows = (unsigned)p.B * H;
        in_turn = FP8 || (H >= 4 && rows * n_parts > 256 && (uint64_t)rows * L > kTurnRowTokens);
    }
    // Which head comes first changes from partition to partition: the heads are not read at one rate (pieces at
    // bytes 384 to 511 of every 1024 take a fifth longer in bf16, a third in fp8, whichever chiplet reads them), and a
    // chiplet or an engine that always had the same ones would end late or, since workgroups are handed out in turn,
    // hold up the others (fp8: half of the places empty from the middle of the pass on).  So head h stands where h + u + u/4 + u/16 + u/64
    // would, u the unit's number (fp8: within its chiplet): every fourth, 16th and 64th unit moves it on once more, which is what meets the
    // engines in turn.  us a step with the heads in place and in turn, 256 requests x 8
    // kv-heads of median length 1500 374 and 357, fp8 199 and 190, 64 x 32 of 1000 234 and 224, heavy-tailed lengths 68.6 and 66.3.
    // (In turn by the partition's number alone: no gain, a head of every fourth still meets the same engine.)
    // Not in a short pass: it is on the chip all at once, nothing waits behind a slow head, and heads in place are ahead.  A
    // planned pass goes by the tokens it has (the list says so; adr_api.hip, plan_pass).  Of a bf16 cache without a plan each row goes
    // by its own length: in place with one item to a compute unit or fewer (in turn and in place, one request of 8000 tokens x 8
    // kv-heads 13.7 and 12.1, 3 of 300 9.4 and 8.8, 20 of 300 14.3 and 12.4; whole rows 8 x 1000 tokens 14.2 and 13.1, 32 x 2000 45.0
    // and 41.9, heads of 64 8 x 1000 14.8 and 12.0), and below kTurnRowTokens in a pass of rows as long (whole rows, 512 of up to 224 tokens
    // 10.2 and 10.0, 384 of up to 400 11.7 and 11.2, 296 of up to 400 11.0 and 10.8; 640 of 300 19.6 and 20.0, 800 of 224 20.0
    // and 20.6, 1600 of 120 21.6 and 22.1, 1120 of up to 600 33.6 and 36.2).
    // Nor of a bf16 cache with fewer than four heads, which share the slow
    // bytes evenly or not at all (400 requests x 2 149 and 145, 1000 x 2 356 and 348; 200 x 4 147 and 149, 500 x 4 353 and 362).
    if (in_turn) {
        const unsigned turn = FP8 ? unit / kChiplets : unit;
        h = (h + turn + turn / 4 + turn / 16 + turn / 64) % H;
    }
    TileIds<NW, FP8, PAIR> ids;
    auto start = [&](int part) { // this wave's tiles of a partition
        const int t0 = part * pt, t1 = pt > 0 ? min(L, t0 + pt) : L;
        const int tiles = (t1 - t0 + kPageSize - 1) / kPageSize - wave;
        ids.start(p, b, t0 / kPageSize + wave, tiles > 0 ? (tiles + NW - 1) / NW : 0);
    };
    start(first_part);
    NewTokens<FP8, PAIR, NW> fresh;
    if constexpr (APPEND)
        fresh.ask(p, length);

    // B operand of QK^T: head r's query, chunk order matching the K loads.  (Columns past the last head
    // repeat it, and a column of a pair holds its query in the other kv-head's chunks too: nobody reads
    // what comes of those.  Loads without a condition leave the tiles' loads to go out behind them.)
    u32x4 qb[4];
    {
        const uint16_t *q = p.q + (int64_t)b * p.q_row_stride + (int64_t)(h * R + min(r, R - 1)) * HD;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            qb[kk] = *(const u32x4 *)(q + (PAIR ? (kk * 4 + j) & 7 : kk * 4 + j) * 8);
    }

    // Byte offsets of this lane, bf16:
    //  K load i (to LDS): row t = 4i + j, slot r of that row, which holds chunk r ^ t.
    //  K operand read, step kk: row r, chunk kk*4 + j, which sits in slot (kk*4 + j) ^ r.
    //  V load u (to registers): row 4j + u, chunk r.
    // fp8 (load_tile_fp8):
    //  K and V load i (to LDS): row t = 8i + lane / 8, slot lane % 8.
    //  K operand read, step kk: row r, 8-byte piece kk*4 + j.
    //  V read, transposed: lane c + 2k of its sixteen names token 4j + (k & 3) of the first (k < 4) or
    //  the second tile, half c of chunk e.
    const uint32_t tok_bytes = (uint32_t)H * D * (FP8 ? 1 : 2);
    const uint32_t head_bytes = (uint32_t)h * D * (FP8 ? 1 : 2);
    uint32_t k_lane[4], k_read[4], fp8_lane[2], v_tr[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = 4 * i + j;
        k_lane[i] = head_bytes + t * tok_bytes + ((r ^ t) * 16);
        const int chunk = i * 4 + j;
        k_read[i] = FP8 ? r * D + (((chunk >> 1) ^ (r & 7)) * 16) + (chunk & 1) * 8 : r * (D * 2) + ((chunk ^ r) * 16);
    }
    const uint32_t v_lane = head_bytes + 4 * j * tok_bytes + r * 16;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        fp8_lane[i] = head_bytes + (8 * i + (lane >> 3)) * tok_bytes + (((lane & 7) ^ (lane >> 3)) * 16);
    {
        const int row = 4 * j + ((r >> 1) & 3), tile = 2 + (r >> 3); // the stage's tiles: K, K, V, V
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v_tr[e] = lds_address(lds_raw) + wave * kWaveBytes + tile * kFp8TileBytes + row * D +
                      ((e ^ (row & 7)) << 4) + 8 * (r & 1);
    }
    const uint32_t page_bytes = kPageSize * tok_bytes;
    const char *kc = (const char *)p.k_cache;
    const char *vc = (const char *)p.v_cache;
    char *mine = lds_raw + wave * kWaveBytes;

    for (int part = first_part;;) {
        const int t0 = part * pt;
        const int t1 = pt > 0 ? min(L, t0 + pt) : L;
        const int count = ids.count;

        WaveState st;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            st.o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
        st.m = kNegBig;
        st.l = 0.f;

        // Two page buffers used alternately (K tile in LDS + V rows in registers),
        // so that the loads of tile n+1 are in flight while tile n is consumed.  A
        // wave always issues the next load group, even past its last tile (then with a
        // descriptor of zero bytes: the loads return zeros and fetch nothing), which
        // keeps the number of loads in flight fixed: "all but the newest eight" is
        // always the tile to consume.
        if constexpr (!FP8) if (count > 0) {
            PageRegs A, B;
            u32x4 ka[4];
            int tile_a = 0, tile_b = 0; // where the two lie in the pool
            auto issue = [&](int n, PageRegs &regs, char *tile, int &page) {
                uint32_t range = 0;
                page = 0;
                if (n < count) {
                    const int t = ids.first + n * NW;
                    page = pool_tile_checked(ids.entry(p, h, n), t, p.num_pages, p.page_shift, p.bounds, b);
                    range = page_bytes;
                }
                load_page(regs, tile, page_rsrc(kc, page, page_bytes, range), page_rsrc(vc, page, page_bytes, range),
                          k_lane, v_lane, tok_bytes);
            };
            int tok = t0 + wave * kPageSize + 4 * j;
            const auto touch = [&](int n, int tile, char *ktile, PageRegs &regs) {
                if (APPEND && __builtin_expect(__any(fresh.page == tile >> p.page_shift), 0))
                    fresh.put_bf16(late_params_of_append(), h, tile, ktile, regs, b, ids.first + n * NW == (L - 1) / kPageSize);
            };
            issue(0, A, mine, tile_a);
            if constexpr (APPEND)
                fresh.settle();
            for (int n = 0;;) {
                issue(n + 1, B, mine + kTileBytes, tile_b);
                wait_older_page();
                touch(n, tile_a, mine, A);
                read_k_operand(ka, mine, k_read);
                attend_page<PAIR>(st, A, ka, qb, p.scale_log2e, 1.f, tok, t1, j, upper);
                tok += NW * kPageSize;
                if (++n >= count)
                    break;
                issue(n + 1, A, mine, tile_a);
                wait_older_page();
                touch(n, tile_b, mine + kTileBytes, B);
                read_k_operand(ka, mine + kTileBytes, k_read);
                attend_page<PAIR>(st, B, ka, qb, p.scale_log2e, 1.f, tok, t1, j, upper);
                tok += NW * kPageSize;
                if (++n >= count)
                    break;
            }
        }

        // fp8: one stage of two tiles of K and of V.  It is copied to registers as soon as it is whole and the
        // next two tiles are on their way while these are attended (twelve waves to a compute unit
        // keep up to 96 KB in flight).
        if constexpr (FP8) if (count > 0) {
            int tiles[2]; // where the two lie in the pool
            auto issue = [&](int n) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    uint32_t range = 0;
                    int &page = tiles[t];
                    page = 0;
                    if (n + t < count) {
                        page = pool_tile_checked(ids.entry(p, h, n + t), ids.first + (n + t) * NW, p.num_pages,
                                                 p.page_shift, p.bounds, b);
                        range = page_bytes;
                    }
                    load_tile_fp8(mine + t * kFp8TileBytes, page_rsrc(kc, page, page_bytes, range), fp8_lane);
                    load_tile_fp8(mine + (2 + t) * kFp8TileBytes, page_rsrc(vc, page, page_bytes, range), fp8_lane);
                }
            };
            ids.load_scales(p, h, ids.now, lane, ids.scale_now);
            issue(0);
            ids.settle(ids.scale_now);
            if constexpr (APPEND)
                fresh.settle();
            int tok = t0 + wave * kPageSize + 4 * j;
            for (int n = 0; n < count; n += 2) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                // The scales of these two tiles (zero for a tile that is none), before the ids move on.
                // (n is even, so tile n + 1 belongs to the same sixty-four lanes.)
                float ks[2], vs[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    ks[t] = PAIR && upper ? ids.scale(ids.SCALES - 2, n + t) : ids.scale(0, n + t);
                    vs[t] = PAIR && upper ? ids.scale(ids.SCALES - 1, n + t) : ids.scale(1, n + t);
                }
                if constexpr (APPEND)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        if (n + t < count && __builtin_expect(__any(fresh.page == tiles[t] >> p.page_shift), 0))
                            fresh.put_fp8(late_params_of_append(), h, tiles[t], t, mine, ks[t], vs[t], b, ids.first + (n + t) * NW == (L - 1) / kPageSize);
                u32x2 ka[4], kb[4], v8[8];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    ka[kk] = *(const u32x2 *)(mine + k_read[kk]);
                    kb[kk] = *(const u32x2 *)(mine + kFp8TileBytes + k_read[kk]);
                }
                lds_read_tr8_x8_wait(v_tr, v8);
                settle_k(ka, kb);
                ks[0] *= p.scale_log2e;
                ks[1] *= p.scale_log2e;
                issue(n + 2);
                const f32x4 sa = scores_fp8<PAIR>(ka, qb, upper), sb = scores_fp8<PAIR>(kb, qb, upper);
                float sc[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sc[i] = sa[i] * ks[0];
                    sc[4 + i] = sb[i] * ks[1];
                }
                attend_two_fp8<PAIR>(st, sc, v8, vs[0], vs[1], tok, tok + NW * kPageSize, t1, j);
                tok += 2 * NW * kPageSize;
            }
        }

        const LateParams late = late_params<ITEMS>();
        // The wave's share of the result takes the place of its own K tiles (no load is on its way to
        // them any more, and no other wave reads them).  [R][D] floats, R <= 16.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const float l = sum_across_rows(st.l); // denominators: the four lane groups hold shares
        if (j == 0 && r < R) {
            ml[(wave * 16 + r) * 2] = st.m;
            ml[(wave * 16 + r) * 2 + 1] = l;
        }
        float *so = (float *)mine;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int g = 4 * j + i;
            if (g < R) {
                if constexpr (FP8) { // st.o[e] holds column 16e + r (a bf16 cache: 8r + e)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        so[g * D + 16 * e + r] = st.o[e][i];
                } else {
                    *(f32x4 *)(so + g * D + 8 * r) = f32x4{st.o[0][i], st.o[1][i], st.o[2][i], st.o[3][i]};
                    *(f32x4 *)(so + g * D + 8 * r + 4) = f32x4{st.o[4][i], st.o[5][i], st.o[6][i], st.o[7][i]};
                }
            }
        }
        __syncthreads();

        // Four output elements per thread and round.  (PAIR: of a row's D columns the lower half belongs
        // to the first kv-head's queries, the upper half to the second's.)
        constexpr int QUADS = HD / 4;
        for (int idx = threadIdx.x; idx < R * QUADS; idx += NW * 64) {
            const int g = idx / QUADS;
            const int c4 = (idx % QUADS) * 4;
            const int col = PAIR && g >= G ? HD + c4 : c4;
            float M = kNegBig;
            float wm[NW], wl[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                wm[w] = ml[(w * 16 + g) * 2];
                wl[w] = ml[(w * 16 + g) * 2 + 1];
                M = fmaxf(M, wm[w]);
            }
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
            float den = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float f = fast_exp2(wm[w] - M);
                acc += f * *(const f32x4 *)((const float *)(lds_raw + w * kWaveBytes) + g * D + col);
                den += f * wl[w];
            }
            const f32x4 o = acc * (den > 0.f ? 1.f / den : 0.f);
            const float lse = den > 0.f ? (M + fast_log2(den)) * kLn2 : -INFINITY;
            const int head = h * R + g;
            if (n_parts == 1) {
                const int64_t row = (int64_t)b * late->Hq + head;
                if (late->out_f32) {
                    *(f32x4 *)((float *)late->out + row * HD + c4) = o;
                } else {
                    u32x2 packed;
                    packed[0] = f32_to_bf16(o[0]) | (f32_to_bf16(o[1]) << 16);
                    packed[1] = f32_to_bf16(o[2]) | (f32_to_bf16(o[3]) << 16);
                    *(u32x2 *)((uint16_t *)late->out + row * HD + c4) = packed;
                }
                if (late->lse && c4 == 0)
                    late->lse[row] = lse;
                if (ITEMS == Items::by_row_meet && !late->meet_bytes && lane == 0)
                    *meet_word<HD>(late, b, h) = 0.f;
            } else if (kMeet) {
                const int64_t row = ((int64_t)b * late->max_parts + part) * late->Hq;
                store_shared(o, partial_rsrc(late->part_o + row * HD), (head * HD + c4) * 4);
                if (c4 == 0)
                    __hip_atomic_store(ITEMS == Items::planned_meet ? late->part_lse + row + head
                                                                    : lse_word<HD>(late, b, h, part, head, lane == 0 && idx == (int)threadIdx.x),
                                       lse, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const int64_t row = ((int64_t)b * late->max_parts + part) * late->Hq + head;
                *(f32x4 *)(late->part_o + row * HD + c4) = o;
                if (c4 == 0)
                    late->part_lse[row] = lse;
            }
        }
        if (kMeet && n_parts > 1 && wave * 64 < R * QUADS && arrive<HD, ITEMS == Items::planned_meet>(late, b, h, h * R, n_parts)) {
            if (ITEMS == Items::planned_meet)
                merge_share<HD, true, NW, 1, 8>(late, b, h, h * R, R, n_parts);
            else if (late->meet == 1) // (up to twelve partitions then: merge_slices)
                merge_share<HD, false, NW, 1, 12>(late, b, h, h * R, R, n_parts);
            else
                merge_share<HD, false, NW, 2, 8>(late, b, h, h * R, R, n_parts);
        }
        if (ITEMS != Items::by_row) // (one partition to a workgroup; what the loop holds is free in what stands above)
            break;
        part += stride;
        if (part >= n_parts)
            break;
        start(part);
        __syncthreads(); // the next partition's K tiles go where the per-wave results lie
    }
    if (blockIdx.x == 0) {
        const LateParams late = late_params<ITEMS>();
        const int in_use = ITEMS == Items::by_row_meet ? late->B * H * result_waves(late->G) : 0;
        clear_control(late->control, late->clear_words, in_use);
    }
}

bool decode_mfma_supports(int d, int G, int Hkv);

hipError_t launch_decode_mfma(const DecodeParams &params, int d, bool fp8, hipStream_t stream)
{
    DecodeParams p = params;
    if (!decode_mfma_supports(d, p.G, p.Hkv))
        return hipErrorInvalidValue;
    const bool pair = d == D / 2;
    const int64_t rows = (int64_t)p.B * (pair ? p.Hkv / 2 : p.Hkv);
    p.grid_stride = grid_stride(rows, p.max_parts);
    if (p.meet && !p.items && p.grid_stride < p.max_parts)
        return hipErrorInvalidValue; // a workgroup of a pass that merges inside takes one partition
    int64_t units = p.items ? p.max_items : (int64_t)p.B * p.grid_stride;
    if (fp8)
        units = (units + kChiplets - 1) / kChiplets * kChiplets; // (the surplus finds no request)
    const int64_t blocks = units * (rows / p.B);
    if (blocks > 0x7fffffffLL)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    // Three workgroups to a compute unit everywhere.  Planned passes of a bf16 cache held to two (by the LDS they ask for) are
    // 0.3 to 1 % faster where rows are long (us a step, three and two: 256 requests x 8 kv-heads of median length 1500 370 and 367,
    // 64 x 32 233.6 and 231.9, heads of 64 101.0 and 99.8, 48 of median 4000 201.8 and 197.7; 37 requests 46.4 and 46.8), but an
    // item of a short row is all latency, and a third fewer of them at once show: 512 requests of 1 token 23.7 and
    // 30.9, 256 of 20 15.6 and 18.8, 64 of 100 12.2 and 14.5, 32 of 700 23.0 and 24.9.  The bound does not tell which.
    auto go = [&](auto kernel, int waves) {
        kernel<<<grid, waves * 64, (size_t)waves * (kWaveBytes + 16 * 2 * sizeof(float)), stream>>>(p);
    };
    // Eight waves to an item where whole rows are items and may be long: a row is then at the mercy of
    // the few waves that share it (us, 4 and 8 waves: 64 requests x 32 kv-heads of up to 4096 tokens 277
    // and 238, 128 x 8 of up to 8192 260 and 240, heads of 64 202 and 152, fp8 171 and 157; with rows of up
    // to 1600 tokens four are ahead: 30 and 33, fp8 45 and 61).  And where there are fewer rows than compute units, however short:
    // a unit has one row then, and nothing else to run (one request x 8 kv-heads of up to 300 tokens 5.7 and 5.4, 600 6.7 and 5.9,
    // 2000 12.3 and 10.4, 4000 20.3 and 15.8; 16 x 8 of up to 1000 12.8 and 12.4, 2000 24.6 and 24.1, fp8 12.5 and 11.4, 20.2 and 18.5;
    // heads of 64 in pairs, 16 x 4 22.4 and 19.6, 32 x 4 24.7 and 24.4; with 256 rows bf16 is the same with either, with 512 of up to 600
    // tokens 17.9 and 20.3, fp8 12.6 and 17.1; bf16 rows of one length are 1 to 4 % behind with eight where they make 50000 to 250000 tokens in all, 96 x
    // 1000 16.3 and 16.9, mixed ones 5 to 20 % ahead).  Not where all rows are of 128 tokens or fewer, which leaves a wave one tile at most
    // and twice the results to combine (ten steps replayed: one request x 8 of 40 tokens 46.1 and 47.4, of 126 50.8 and 51.9, fp8 57.6 and
    // 64.5; five of 150 tokens 30.8 and 29.4, fp8 35.2 and 32.2).  And fp8 rows of 128 bytes leave some units to spare: 31 x 8 of 2000 tokens
    // 26.6 and 28.9, of 4000 49.0 and 53.8, of median 1000 38.5 and 36.8; 24 x 8 are level or ahead.
    const bool wide = p.partition_tokens == 0 && (p.max_seq_len >= 4096 || (rows < (fp8 && !pair ? 224 : 256) && p.max_seq_len > 8 * kPageSize));
    auto pick = [&](auto fp8_, auto pair_) {
        constexpr bool F = fp8_.value, P = pair_.value;
        if (wide)
            p.k_new ? go(decode_mfma_kernel<F, P, 8, Items::by_row, true>, 8) : go(decode_mfma_kernel<F, P, 8, Items::by_row, false>, 8);
        else if (p.items)
            p.meet ? go(decode_mfma_kernel<F, P, 4, Items::planned_meet, false>, 4) : go(decode_mfma_kernel<F, P, 4, Items::planned, false>, 4);
        else if (p.meet)
            go(decode_mfma_kernel<F, P, 4, Items::by_row_meet, false>, 4);
        else
            p.k_new ? go(decode_mfma_kernel<F, P, 4, Items::by_row, true>, 4) : go(decode_mfma_kernel<F, P, 4, Items::by_row, false>, 4);
    };
    if (fp8)
        pair ? pick(std::true_type(), std::true_type()) : pick(std::true_type(), std::false_type());
    else
        pair ? pick(std::false_type(), std::true_type()) : pick(std::false_type(), std::false_type());
    return hipGetLastError();
}

// d = 128 with groups of up to sixteen heads; d = 64 where two kv-heads, side by side in a token's row, make
// a row of 128 elements (groups of 1, 2, 4 and 8 heads, as the vector-ALU kernel serves them there).
bool decode_mfma_supports(int d, int G, int Hkv)
{
    return (d == D && G >= 1 && G <= 16) || (d == D / 2 && Hkv % 2 == 0 && (G == 1 || G == 2 || G == 4 || G == 8));
}

} // namespace adr
