// Decode attention with the QK^T and PV contractions on the matrix cores
// (bf16 cache; d = 128 with any group size G <= 16, and d = 64 with two kv-heads taken together).
//
// One workgroup of 4 waves per (request, kv-head, partition); wave w streams
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
// half.  (113 against 121 us for the vector-ALU kernel at 128 requests, 8 kv-heads, G = 4.)
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
//       head r, loaded once) uses the same order.  Heads r >= G are zero
//       columns.  Each wave owns two such tiles (the page being consumed and
//       the page in flight).
//       Result layout: lane (r, j) holds S[token 4j+i][head r], i = 0..3.
// softmax  per lane over its 4 tokens, running max shared across the four
//       lane groups j by two wave shuffles; fp32 throughout, base 2.
// PV    O[head][dcol] += P[16 x 16 tokens] * V[16 tokens x 16 dcols], eight
//       v_mfma_f32_16x16x16_bf16 per page (one per e = 0..7, dcol = 8r + e).
//       The S layout above IS the A-operand layout (row = head r, k = token
//       4j+i), so P never moves between lanes.  P is split into a bf16 head
//       and a bf16 remainder, both rounded (two MFMAs), so the weights keep 17 significant
//       bits (PAIR: three terms, all 24).  V is loaded in its natural layout -- lane (r, j), load u: the 16
//       bytes of token 4j+u at chunk r, i.e. four complete 256-byte rows per
//       instruction -- and the B operand (k = token 4j+u, n = r) for column
//       set e is assembled from those four registers with byte permutes.
//       Result layout: lane (r, j) holds O[head 4j+i][8r + e].
#include "mfma_page.h"

#include <algorithm>

namespace adr {

__device__ __forceinline__ void read_k_operand(u32x4 (&ka)[4], const char *ktile,
                                               const uint32_t (&k_read)[4])
{
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
        ka[kk] = *(const u32x4 *)(ktile + k_read[kk]);
}

// Workgroups are numbered row by row: kv-head fastest (the heads of a page are read together),
// then the row's partitions, `stride` of them; a workgroup takes every stride-th partition of its
// row from its own on and leaves at once when the row has none for it.  The grid is sized from
// the caller's bound on the lengths, not from the lengths, so most workgroups may find nothing.
// Two things were measured on the 70B-shaped workload (1 712 items of 13 312 workgroups, 73 us):
// (1) the hardware hands consecutive workgroups to its compute units in turn, so when the number of
// workgroups per row divides the units evenly, a row's few real workgroups fall on the same units
// row after row: 123 us with 16 partitions per row in the grid, 152 us with 64.  The stride is
// therefore odd.  (2) Workgroups that find nothing still cost about a nanosecond each, and a loose
// bound makes tens of thousands of them: the stride stops at kGridStrideMax, and rows with more
// partitions (rare where this kernel is chosen) have their workgroups loop.
constexpr int kGridStrideMax = 33;
__host__ __device__ inline int grid_stride(int max_parts)
{
    const int n = max_parts < kGridStrideMax ? max_parts : kGridStrideMax;
    return n > 1 ? (n | 1) : n;
}


constexpr int kWaveBytes = kStages * kTileBytes; // LDS of one wave: its K tiles, then its share of the result

// The tiles of one wave in one partition: first, first + NW, ...  Their table entries arrive with one
// vector load, lane n holding the wave's n-th tile, and reach the scalar unit by a lane read; a
// second register holds the next sixty-four.
template <int NW>
struct TileIds {
    const int32_t *row; // the row's table
    int first, last_entry, shift;
    int now, next;

    __device__ __forceinline__ int load(int n) const
    {
        return row[min((first + n * NW) >> shift, last_entry)]; // (clamped: inside the row's table)
    }
    __device__ __forceinline__ void start(const DecodeParams &p, int b, int first_tile)
    {
        row = p.block_table + (int64_t)b * p.max_pages;
        first = first_tile;
        last_entry = p.max_pages - 1;
        shift = p.page_shift;
        now = load(threadIdx.x & 63);
        next = 0;
    }
    // Entry of tile n; called for n = 0, 1, 2, ... in turn, in front of the tile's own loads.
    __device__ __forceinline__ int entry(int n, int count)
    {
        if ((n & 63) == 0) {
            if (n) {
                asm volatile("" : "+v"(next)); // it is waited for here and not at every lane read below
                now = next;
            }
            if (count > n + 64)
                next = load(n + 64 + (threadIdx.x & 63));
        }
        return __builtin_amdgcn_readlane(now, n & 63);
    }
};

template <bool PAIR, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(3)))
void decode_mfma_kernel(const DecodeParams p)
{
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

    const int stride = grid_stride(p.max_parts);
    const int h = blockIdx.x % H;
    const int first_part = (blockIdx.x / H) % stride;
    const int b = blockIdx.x / (H * stride);

    const int L = max(min(((const __attribute__((address_space(4))) int32_t *)p.seq_lens)[b], p.max_seq_len), 0);
    const int pt = row_partition(L, p.partition_tokens, p.max_parts, p.min_part);
    const int n_parts = parts_of(L, pt);
    if (first_part >= n_parts)
        return;
    TileIds<NW> ids;
    ids.start(p, b, first_part * (pt / kPageSize) + wave);

    // B operand of QK^T: head r's query, chunk order matching the K loads
    u32x4 qb[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        qb[kk] = u32x4{0u, 0u, 0u, 0u};
        const int chunk = kk * 4 + j;
        if (r < R && (!PAIR || (kk >= 2) == upper))
            qb[kk] = *(const u32x4 *)(p.q + (int64_t)b * p.q_row_stride + (int64_t)(h * R + r) * HD +
                                      (PAIR ? chunk & 7 : chunk) * 8);
    }

    // Byte offsets of this lane.
    //  K load i (to LDS): row t = 4i + j, slot r of that row, which holds chunk r ^ t.
    //  K operand read, step kk: row r, chunk kk*4 + j, which sits in slot (kk*4 + j) ^ r.
    //  V load u (to registers): row 4j + u, chunk r.
    const uint32_t tok_bytes = (uint32_t)H * D * 2;
    uint32_t k_lane[4], k_read[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = 4 * i + j;
        k_lane[i] = (uint32_t)h * D * 2 + t * tok_bytes + ((r ^ t) * 16);
        k_read[i] = r * (D * 2) + (((i * 4 + j) ^ r) * 16);
    }
    const uint32_t v_lane = (uint32_t)h * D * 2 + 4 * j * tok_bytes + r * 16;
    const uint32_t page_bytes = kPageSize * tok_bytes;
    const char *kc = (const char *)p.k_cache;
    const char *vc = (const char *)p.v_cache;
    char *mine = lds_raw + wave * kWaveBytes;

    for (int part = first_part;;) {
        const int t0 = part * pt;
        const int t1 = pt > 0 ? min(L, t0 + pt) : L;
        const int tiles = (t1 - t0 + kPageSize - 1) / kPageSize - wave;
        const int count = tiles > 0 ? (tiles + NW - 1) / NW : 0; // this wave's tiles

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
        if (count > 0) {
            PageRegs A, B;
            u32x4 ka[4];
            auto issue = [&](int n, PageRegs &regs, char *tile) {
                uint32_t range = 0;
                int page = 0;
                if (n < count) {
                    const int t = ids.first + n * NW;
                    page = pool_tile_checked(ids.entry(n, count), t, p.num_pages, p.page_shift, p.bounds, b);
                    range = page_bytes;
                }
                load_page(regs, tile, page_rsrc(kc, page, page_bytes, range), page_rsrc(vc, page, page_bytes, range),
                          k_lane, v_lane, tok_bytes);
            };
            int tok = t0 + wave * kPageSize + 4 * j;
            issue(0, A, mine);
            for (int n = 0;;) {
                issue(n + 1, B, mine + kTileBytes);
                wait_older_page();
                read_k_operand(ka, mine, k_read);
                attend_page<PAIR>(st, A, ka, qb, p.scale_log2e, 1.f, tok, t1, j, upper);
                tok += NW * kPageSize;
                if (++n >= count)
                    break;
                issue(n + 1, A, mine);
                wait_older_page();
                read_k_operand(ka, mine + kTileBytes, k_read);
                attend_page<PAIR>(st, B, ka, qb, p.scale_log2e, 1.f, tok, t1, j, upper);
                tok += NW * kPageSize;
                if (++n >= count)
                    break;
            }
        }

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
                *(f32x4 *)(so + g * D + 8 * r) = f32x4{st.o[0][i], st.o[1][i], st.o[2][i], st.o[3][i]};
                *(f32x4 *)(so + g * D + 8 * r + 4) = f32x4{st.o[4][i], st.o[5][i], st.o[6][i], st.o[7][i]};
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
                const int64_t row = (int64_t)b * p.Hq + head;
                if (p.out_f32) {
                    *(f32x4 *)((float *)p.out + row * HD + c4) = o;
                } else {
                    u32x2 packed;
                    packed[0] = f32_to_bf16(o[0]) | (f32_to_bf16(o[1]) << 16);
                    packed[1] = f32_to_bf16(o[2]) | (f32_to_bf16(o[3]) << 16);
                    *(u32x2 *)((uint16_t *)p.out + row * HD + c4) = packed;
                }
                if (p.lse && c4 == 0)
                    p.lse[row] = lse;
            } else {
                const int64_t row = ((int64_t)b * p.max_parts + part) * p.Hq + head;
                *(f32x4 *)(p.part_o + row * HD + c4) = o;
                if (c4 == 0)
                    p.part_lse[row] = lse;
            }
        }
        part += stride;
        if (part >= n_parts)
            break;
        ids.start(p, b, part * (pt / kPageSize) + wave);
        __syncthreads(); // the next partition's K tiles go where the per-wave results lie
    }
}

bool decode_mfma_supports(int d, int G, int Hkv);

hipError_t launch_decode_mfma(const DecodeParams &p, int d, hipStream_t stream)
{
    if (!decode_mfma_supports(d, p.G, p.Hkv))
        return hipErrorInvalidValue;
    const bool pair = d == D / 2;
    const dim3 grid((unsigned)((int64_t)p.B * (pair ? p.Hkv / 2 : p.Hkv) * grid_stride(p.max_parts)));
    constexpr int NW = kWaves;
    const size_t lds = (size_t)NW * (kWaveBytes + 16 * 2 * sizeof(float));
    if (pair)
        decode_mfma_kernel<true, NW><<<grid, NW * 64, lds, stream>>>(p);
    else
        decode_mfma_kernel<false, NW><<<grid, NW * 64, lds, stream>>>(p);
    return hipGetLastError();
}

// d = 128 with groups of up to sixteen heads; d = 64 where two kv-heads, side by side in a token's row, make
// a row of 128 elements (groups of 1, 2, 4 and 8 heads, as the vector-ALU kernel serves them there).
bool decode_mfma_supports(int d, int G, int Hkv)
{
    return (d == D && G >= 1 && G <= 16) || (d == D / 2 && Hkv % 2 == 0 && (G == 1 || G == 2 || G == 4 || G == 8));
}

} // namespace adr
