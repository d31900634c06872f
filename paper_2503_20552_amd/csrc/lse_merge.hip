// Log-sum-exp merge of per-partition attention results.
//
// A slice of d/4 threads reads one partition's row of one head: each thread owns four
// consecutive output elements (16-byte loads of the fp32 partials).  A (request, head) row has S
// slices, slice s taking partitions s, s + S, ... in rounds of CH with all their loads issued before
// any is used and carrying a running maximum of the lse values; the slices of a row meet in LDS.
// The order is fixed, so the result is the same from run to run.  Loads past a row's last
// partition are left out.  When the attention pass left a non-zero expired-waits word in the call's
// status block, every row gets NaN instead.
//
// What bounds it: latency.  A launch, the length, then one round trip per round; the partials
// themselves are a few MB out of the caches.  Hence the slices: with one slice per row a request of
// 30000 tokens in partitions of 256 took eight rounds on four workgroups.
#include "adr_device.h"

#include <algorithm>

namespace adr {

template <int D, int S, int CH>
__global__ __launch_bounds__(256) void lse_merge_kernel(const MergeParams p)
{
    constexpr int TPR = D / 4;         // threads per slice
    constexpr int RPB = 256 / TPR / S; // rows per block
    typedef const __attribute__((address_space(4))) int32_t *const_ptr;
    const int slice = threadIdx.x / TPR;
    const int64_t row = (int64_t)blockIdx.x * RPB + slice / S;
    const int s = slice % S;
    const int col = (threadIdx.x % TPR) * 4;
    const bool mine = row < (int64_t)p.B * p.heads;
    const int b = mine ? (int)(row / p.heads) : 0, h = mine ? (int)(row % p.heads) : 0;

    // The length and the status are fetched side by side.
    int first, count;
    const uint32_t expired = p.status ? ((const_ptr)p.status)[kStatusExpiredWaits] : 0u;
    if (p.part_offsets) {
        first = p.part_offsets[b];
        count = p.part_offsets[b + 1] - first;
    } else {
        const int L = max(min(p.seq_lens[b], p.max_seq_len), 0);
        count = p.part_counts ? p.part_counts[b]
                              : parts_of(L, row_partition(L, p.partition_tokens, p.max_parts, p.cut, p.cut_share));
        first = b * p.max_parts;
    }
    // The pass that wrote the partials reported a broken hand-shake between its waves: no row of
    // the call may pass as a result (rows with one partition included).
    const bool broken = expired != 0u;
    // Otherwise a row with one partition already holds what the attention kernel wrote.
    const bool skip = !mine || (!broken && !p.part_offsets && count <= 1);
    if (S == 1 ? skip : __syncthreads_and(skip))
        return;
    if (skip || broken)
        count = 0;

    float top = -INFINITY, total = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int i0 = s; i0 < count; i0 += S * CH) {
        float ls[CH];
        f32x4 xs[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            ls[u] = -INFINITY;
            xs[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (i0 + u * S < count) {
                const int64_t pr = (int64_t)(first + i0 + u * S) * p.heads + h;
                ls[u] = p.part_lse[pr];
                xs[u] = *(const f32x4 *)(p.part_o + pr * D + col);
            }
        }
        float cm = -INFINITY;
#pragma unroll
        for (int u = 0; u < CH; ++u)
            cm = fmaxf(cm, ls[u]);
        const float nt = fmaxf(top, cm);
        if (nt > -INFINITY) {
            const float rs = fast_exp2((top - nt) * kLog2e); // 0 when nothing was seen before
            acc *= rs;
            total *= rs;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const float w = fast_exp2((ls[u] - nt) * kLog2e);
                if (w > 0.f) { // an empty partition's payload is never used
                    acc += w * xs[u];
                    total += w;
                }
            }
            top = nt;
        }
    }
    if (S > 1) {
        __shared__ float meet[256 / TPR][2];
        __shared__ f32x4 meet_acc[256];
        meet_acc[threadIdx.x] = acc;
        if (col == 0) {
            meet[slice][0] = top;
            meet[slice][1] = total;
        }
        __syncthreads();
        if (s != 0)
            return;
        float all = top;
#pragma unroll
        for (int k = 1; k < S; ++k)
            all = fmaxf(all, meet[slice + k][0]);
        if (all > -INFINITY) {
            const float w0 = fast_exp2((top - all) * kLog2e);
            acc *= w0;
            total *= w0;
#pragma unroll
            for (int k = 1; k < S; ++k) {
                const float w = fast_exp2((meet[slice + k][0] - all) * kLog2e);
                if (w > 0.f) {
                    acc += w * meet_acc[threadIdx.x + k * TPR];
                    total += w * meet[slice + k][1];
                }
            }
            top = all;
        }
    }
    if (skip)
        return;
    const float inv = total > 0.f ? 1.f / total : 0.f;
    const float nan = __builtin_nanf("");
    f32x4 o = acc * inv;
    if (broken)
        o = f32x4{nan, nan, nan, nan};
    const int64_t off = row * D + col;
    if (p.out_f32) {
        *(f32x4 *)((float *)p.out + off) = o;
    } else {
        u32x2 w;
        w[0] = f32_to_bf16(o[0]) | (f32_to_bf16(o[1]) << 16);
        w[1] = f32_to_bf16(o[2]) | (f32_to_bf16(o[3]) << 16);
        *(u32x2 *)((uint16_t *)p.out + off) = w;
    }
    if (p.lse_out && col == 0)
        p.lse_out[row] = broken ? nan : total > 0.f ? top + fast_log2(total) * kLn2 : -INFINITY;
}

template <int D>
static void launch_merge(const MergeParams &p, int slices, hipStream_t stream)
{
    const int64_t rows = (int64_t)p.B * p.heads;
    auto go = [&](auto kernel, int S) {
        const int per_block = 256 / (D / 4) / S;
        kernel<<<dim3((unsigned)((rows + per_block - 1) / per_block)), 256, 0, stream>>>(p);
    };
    if (slices >= 8)
        go(lse_merge_kernel<D, 8, 8>, 8);
    else if (slices >= 4)
        go(lse_merge_kernel<D, 4, 8>, 4);
    else if (slices >= 2)
        go(lse_merge_kernel<D, 2, 8>, 2);
    else
        go(lse_merge_kernel<D, 1, 16>, 1);
}

// Slices per row: one per six partitions a row may have, as long as the blocks this makes (most of
// them may find a row of few partitions and leave) stay within 256 rows per partition, of which no more
// than 48 count (a bound far above the lengths allows any number: 8192 rows of one partition, 128
// allowed, 2.3 us more with four slices than with one).  us, one slice
// and the rule's: 32 rows of 118 partitions 12.3 and 4.8, 512 rows 14.6 and 6.0, 1280 rows of up to
// 33 4.8 and 4.1, 4096 rows 6.5 and 6.1; 8192 rows of up to 9 or 33 have one (4.6, 10.6; with
// four 8.5, 11.2).  adr_lse_merge, which knows no bound, has one.
int merge_slices(int64_t rows, int max_parts)
{
    int slices = 1;
    while (slices < 8 && slices * 2 * 6 <= max_parts && rows * slices * 2 <= (int64_t)256 * std::min(max_parts, 48))
        slices *= 2;
    return slices;
}

hipError_t launch_lse_merge(const MergeParams &p, hipStream_t stream)
{
    if ((int64_t)p.B * p.heads == 0)
        return hipSuccess;
    const int slices = merge_slices((int64_t)p.B * p.heads, p.max_parts);
    if (p.d == 128)
        launch_merge<128>(p, slices, stream);
    else if (p.d == 64)
        launch_merge<64>(p, slices, stream);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

} // namespace adr
