// Host side of the C ABI: argument checks and kernel dispatch.  The attention, append, merge and
// copy entry points only enqueue kernels: they never allocate, synchronise or copy.  (The status
// readers at the end synchronise; that is what they are for.)
#include "../../include/adr.h"
#include "adr_device.h"
#include "plan.h"

#include <algorithm>
#include <atomic>
#include <limits.h>

namespace adr {
hipError_t launch_kv_append(const AppendParams &p, bool fp8, hipStream_t stream);
hipError_t launch_plan(const PlanParams &p, hipStream_t stream);
hipError_t launch_decode_valu(const DecodeParams &p, int d, bool fp8, hipStream_t stream);
hipError_t launch_decode_mfma(const DecodeParams &p, int d, bool fp8, hipStream_t stream);
hipError_t launch_decode_stream(const DecodeParams &p, int d, bool fp8, hipStream_t stream);
hipError_t read_stream_faults(unsigned long long *count);
bool decode_stream_supports(int d, int G, int B);
bool decode_valu_supports(int d, int G);
bool decode_mfma_supports(int d, int G, int Hkv);
int merge_slices(int64_t rows, int max_parts);
hipError_t launch_lse_merge(const MergeParams &p, hipStream_t stream);
hipError_t launch_stream_read(const void *src, size_t bytes, void *sink, hipStream_t stream);
hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t stream);
} // namespace adr

namespace {

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

int check_cache(const adr_kv_cache *c)
{
    if (!c || !c->k || !c->v)
        return ADR_ERR_NULL;
    if (c->num_pages <= 0 || c->Hkv <= 0)
        return ADR_ERR_SHAPE;
    if ((c->page_size != 16 && c->page_size != 32 && c->page_size != 64) || (c->d != 64 && c->d != 128))
        return ADR_ERR_UNSUPPORTED;
    if (c->dtype != ADR_BF16 && c->dtype != ADR_FP8_E4M3)
        return ADR_ERR_UNSUPPORTED;
    if (c->dtype == ADR_FP8_E4M3 && (!c->k_scale || !c->v_scale))
        return ADR_ERR_NULL;
    if (!aligned16(c->k) || !aligned16(c->v))
        return ADR_ERR_SHAPE;
    return ADR_OK;
}

int64_t max_parts_for(int max_seq_len, int partition_tokens)
{
    if (partition_tokens <= 0)
        return 1;
    const int64_t n = ((int64_t)max_seq_len + partition_tokens - 1) / partition_tokens;
    return n < 1 ? 1 : n;
}

size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

// Layout of a split pass's workspace: partial outputs, their lse values, then the control area
// (one status block and one block per launch of the resident kernel: 512 rows each).
struct WorkspacePlan {
    size_t part_o_bytes = 0, part_lse_bytes = 0, control_bytes = 0;
    size_t total() const { return part_o_bytes + part_lse_bytes + control_bytes; }
    int control_words() const { return (int)(control_bytes / 4); }
};

WorkspacePlan plan_workspace(int B, int Hq, int d, int max_seq_len, int partition_tokens)
{
    WorkspacePlan w;
    if (partition_tokens < 0 || B <= 0 || Hq <= 0 || d <= 0 || max_seq_len <= 0)
        return w;
    if (partition_tokens > 0) {
        const size_t rows = (size_t)B * (size_t)max_parts_for(max_seq_len, partition_tokens) * Hq;
        w.part_o_bytes = round256(rows * d * sizeof(float));
        w.part_lse_bytes = round256(rows * sizeof(float));
    }
    w.control_bytes = (size_t)adr::kControlBlockBytes * (1 + (B + 511) / 512);
    return w;
}

// Clears a call's control area when no append kernel of the same call does it on its way.
__global__ void control_clear_kernel(uint32_t *words, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        words[i] = 0u;
}

// Do `a` and `b` share a byte?
bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes)
{
    return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

// ---- per-device addresses of this file's static device data -------------------------------
// adr_decode_attention_static keeps its workspace in `scratch`, a static device array, because
// its callers cannot allocate.  In host code the name of a static device variable is only a
// handle: the address a kernel (or a copy) may use comes from hipGetSymbolAddress, once per
// device with that device current (every device holds its own copy of the array at its own
// address).  Everything below uses those addresses, never the names.
static __device__ __align__(256) unsigned char scratch[ADR_STATIC_SCRATCH_BYTES];
#ifdef ADR_DEBUG_BOUNDS
static __device__ adr::BoundsRecord g_bounds;
#endif

struct DeviceData {
    unsigned char *scratch = nullptr;
    adr::BoundsRecord *bounds = nullptr;
};
DeviceData g_device_data[64];
std::atomic<int> g_device_ready[64];

int device_data(const DeviceData **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return ADR_ERR_LAUNCH;
    if (!g_device_ready[dev].load(std::memory_order_acquire)) {
        DeviceData dd;
        if (hipGetSymbolAddress((void **)&dd.scratch, HIP_SYMBOL(scratch)) != hipSuccess || !dd.scratch)
            return ADR_ERR_LAUNCH;
#ifdef ADR_DEBUG_BOUNDS
        if (hipGetSymbolAddress((void **)&dd.bounds, HIP_SYMBOL(g_bounds)) != hipSuccess || !dd.bounds)
            return ADR_ERR_LAUNCH;
#endif
        g_device_data[dev] = dd; // two threads racing here write the same values
        g_device_ready[dev].store(1, std::memory_order_release);
    }
    *out = &g_device_data[dev];
    return ADR_OK;
}

// Where a debug build records out-of-range table entries and positions (nullptr in a release build).
int bounds_record(adr::BoundsRecord **out)
{
    *out = nullptr;
#ifdef ADR_DEBUG_BOUNDS
    const DeviceData *dd = nullptr;
    const int rc = device_data(&dd);
    if (rc != ADR_OK)
        return rc;
    *out = dd->bounds;
#endif
    return ADR_OK;
}

} // namespace

extern "C" {

int adr_version(void) { return 200; }

int adr_stream_create_cu_mask(void **stream, const uint32_t *cu_mask, int n_words)
{
    if (!stream || !cu_mask)
        return ADR_ERR_NULL;
    if (n_words <= 0)
        return ADR_ERR_SHAPE;
    uint32_t any = 0;
    for (int i = 0; i < n_words; ++i)
        any |= cu_mask[i];
    if (!any)
        return ADR_ERR_SHAPE;
    hipStream_t s = nullptr;
    if (hipExtStreamCreateWithCUMask(&s, (uint32_t)n_words, cu_mask) != hipSuccess)
        return ADR_ERR_LAUNCH;
    *stream = (void *)s;
    return ADR_OK;
}

int adr_stream_destroy(void *stream)
{
    if (!stream)
        return ADR_ERR_NULL;
    return hipStreamDestroy((hipStream_t)stream) == hipSuccess ? ADR_OK : ADR_ERR_LAUNCH;
}

int adr_stream_fault_count(uint64_t *count)
{
    if (!count)
        return ADR_ERR_NULL;
    unsigned long long n = 0;
    if (adr::read_stream_faults(&n) != hipSuccess)
        return ADR_ERR_LAUNCH;
    *count = (uint64_t)n;
    return ADR_OK;
}

const char *adr_status_string(int status)
{
    switch (status) {
    case ADR_OK: return "ok";
    case ADR_ERR_NULL: return "a required pointer is NULL";
    case ADR_ERR_SHAPE: return "a size is non-positive, inconsistent or misaligned";
    case ADR_ERR_UNSUPPORTED: return "shape or dtype outside the supported set";
    case ADR_ERR_WORKSPACE: return "workspace missing or too small for the split pass";
    case ADR_ERR_LAUNCH: return "the HIP runtime refused a kernel launch";
    default: return "unknown status";
    }
}

int adr_kv_append(const adr_kv_cache *cache, const void *k_new, const void *v_new,
                  int64_t new_row_stride, const int32_t *block_table, int max_pages_per_req,
                  const int32_t *positions, int B, void *stream)
{
    const int rc = check_cache(cache);
    if (rc != ADR_OK)
        return rc;
    if (!k_new || !v_new || !block_table || !positions)
        return ADR_ERR_NULL;
    if (B < 0 || max_pages_per_req <= 0 || new_row_stride < (int64_t)cache->Hkv * cache->d)
        return ADR_ERR_SHAPE;
    if (!aligned16(k_new) || !aligned16(v_new) || (new_row_stride % 8) != 0)
        return ADR_ERR_SHAPE;
    adr::AppendParams p;
    p.k_cache = cache->k;
    p.v_cache = cache->v;
    p.k_scale = cache->k_scale;
    p.v_scale = cache->v_scale;
    p.k_new = (const uint16_t *)k_new;
    p.v_new = (const uint16_t *)v_new;
    p.new_row_stride = new_row_stride;
    p.block_table = block_table;
    p.positions = positions;
    p.seq_lens = nullptr;
    p.max_seq_len = 0;
    p.page_size = cache->page_size;
    p.max_pages = max_pages_per_req;
    p.num_pages = cache->num_pages;
    p.Hkv = cache->Hkv;
    p.d = cache->d;
    p.B = B;
    p.clear_words = nullptr;
    p.n_clear_words = 0;
    p.meet.part_lse = nullptr;
    p.plan.items = nullptr;
    if (bounds_record(&p.bounds) != ADR_OK)
        return ADR_ERR_LAUNCH;
    const hipError_t e =
        adr::launch_kv_append(p, cache->dtype == ADR_FP8_E4M3, (hipStream_t)stream);
    return e == hipSuccess ? ADR_OK : ADR_ERR_LAUNCH;
}

size_t adr_decode_workspace_bytes(int B, int Hq, int d, int max_seq_len, int partition_tokens)
{
    return plan_workspace(B, Hq, d, max_seq_len, partition_tokens).total();
}

namespace {
// The step's new token, when the call appends before it attends (adr_decode_step).
struct NewToken {
    const void *k, *v;
    int64_t row_stride;
};

// Which kernel serves a pass (negative: the status to return).
enum { KERNEL_VALU = ADR_KERNEL_VALU, KERNEL_STREAM = ADR_KERNEL_MFMA, KERNEL_GRID = ADR_KERNEL_MFMA_GRID };

int choose_kernel(const adr_kv_cache *cache, int B, int Hq, int max_seq_len, int partition_tokens, unsigned flags)
{
    const int G = Hq / cache->Hkv;
    const int d = cache->d;
    const unsigned want = flags & 0xFu;
    const bool fp8 = cache->dtype == ADR_FP8_E4M3;
    if (want == ADR_KERNEL_VALU)
        return adr::decode_valu_supports(d, G) ? KERNEL_VALU : -ADR_ERR_UNSUPPORTED;
    if (want == ADR_KERNEL_MFMA_GRID)
        return !fp8 && d == 128 && adr::decode_mfma_supports(d, G, cache->Hkv) ? KERNEL_GRID : -ADR_ERR_UNSUPPORTED;
    if (want == ADR_KERNEL_MFMA) {
        if (adr::decode_stream_supports(d, G, B))
            return KERNEL_STREAM;
        return !fp8 && d == 128 && adr::decode_mfma_supports(d, G, cache->Hkv) ? KERNEL_GRID : -ADR_ERR_UNSUPPORTED;
    }
    if (want != ADR_KERNEL_AUTO)
        return -ADR_ERR_UNSUPPORTED;
    // Measured on MI355X (us per launch, partitions as pass_cut below makes them).  With few
    // (request, kv-head) pairs the hardware's own hand-out of one workgroup per item, three to a
    // compute unit, beats the resident workgroups' set-up, hand-over and tail:
    //     pairs                        8     64    320   1024 (G = 4)  1024 (G = 8)
    //     one workgroup per item       6     18     44    197            72
    //     resident workgroups         30     35     54    206            79
    // From 2048 on the two meet (397 and 398 with G = 4) and the resident kernel pulls ahead as rows
    // grow (1610 against 1650 with 4096 pairs of mean length 5000; adr_decode_step, which plans its passes, serves up
    // to 2048 requests by item all the same, plan_pass: 1652 and 1628), except in groups of one
    // head, where items of a partition each stay ahead up to 4096 pairs (236 against 248 at 2048), and
    // for rows of up to 2048 tokens, which are then items as they are (2048 rows of 1500 tokens 241
    // against 268, of median 200 74 against 82).
    const bool splits = partition_tokens > 0 && max_seq_len > partition_tokens;
    const int64_t pairs = (int64_t)B * cache->Hkv;
    // fp8: one workgroup per item throughout (us per step, one workgroup per item and resident ones: 256
    // requests x 8 kv-heads of median length 1500 226 and 240, of median 1000 154 and 168, of 3000 tokens
    // 288 and 300, of 300 49 and 71; groups of two 211 and 232, of eight 244 and 326; whole rows 256
    // and 405; 512 requests of median 1500 the same, 442).  One shape is the other way round, 512 requests in
    // groups of four of which one in ten has 32000 to 65000 tokens (1.01 and 0.98 ms); heavy-tailed lengths
    // under the same bound are not (162 and 177), and the arguments do not tell the two apart.
    bool resident = !fp8 && splits && pairs >= (G == 1 ? 4096 : 2048) && max_seq_len > 2048;
    // The test aid is about the resident kernel's waits: where it is asked for, that kernel serves.
    if (flags & ADR_DEBUG_EXPIRE_WAITS)
        resident = fp8 || (splits && (G <= 4 || pairs >= 2048 || max_parts_for(max_seq_len, partition_tokens) > 32));
    if (resident && adr::decode_stream_supports(d, G, B))
        return KERNEL_STREAM;
    // d = 64, two kv-heads a row: ahead of the vector ALUs in groups of two heads or more (us, 2040 against 2048
    // pairs of median length 1500, fp8: groups of eight 128 and 446; bf16 of eight 214 and 436, of four 206
    // and 239; four requests of 300 tokens in groups of four 9 and 12; small fp8 passes in groups of two 5 %
    // behind, large ones 20 % ahead) and in large passes of groups of one (fp8
    // 113 and 207, bf16 195 and 223).  Small passes of groups of one are the vector ALUs': with few
    // items a workgroup's own chain of steps is all there is, and theirs is shorter.  us, by item and on the vector ALUs, eight
    // waves each, whole rows of 8 kv-heads, append and attention: one request of 512 tokens 8.8 and 7.5, of 1000 11.8 and 8.6, of 2000 18.7 and 16.5,
    // four of 512 9.1 and 7.9, of 1000 12.6 and 12.2, 16 of 512 10.3 and 9.8, 64 of 256 9.2 and 10.5; fp8 one of 1000 13.4 and 9.7,
    // four of 2000 20.0 and 17.4, 32 of 512 11.7 and 11.0, 64 of 256 11.2 and 11.5.  The two meet in bf16 near 64000 tokens over all
    // heads, in fp8 near 130000, with 64 requests sooner; the line was drawn below that, when both were slower, and holds for both entry
    // points.  A step is another matter:
    // the item kernel appends inside, and is ahead in bf16 up to 512 tokens (one of 60 4.4 and 6.8, of 200 6.2 and 6.8, of 512 7.7
    // and 7.9, of 1000 10.8 and 10.1, four of 512 7.5 and 8.0) and in all partitions of 256 (8 of 512 9.2 and 10.5), in fp8 up to
    // 200 (6.7 and 6.8, of 512 9.5 and 8.5).  (Neither is the less exact: pairs carry their weights in three bf16 terms, 24 bits.)
    const bool few = d == 64 && G == 1 && pairs * max_seq_len <= 32768 && max_seq_len < 4096;
    if (!few && adr::decode_mfma_supports(d, G, cache->Hkv))
        return KERNEL_GRID;
    if (adr::decode_valu_supports(d, G))
        return KERNEL_VALU;
    return -ADR_ERR_UNSUPPORTED;
}

// The partitions a pass works with, where the caller leaves both the kernel and the merge to the call:
// what lies in the workspace in between is then the library's own affair (it never takes more places
// than the caller's partitions would).
struct PassCut {
    int tokens;    // per partition, when cut is 0
    int max_parts; // partitions of a row at most
    int cut;       // > 0: see row_partition
    uint32_t share;
};

PassCut pass_cut(const adr_kv_cache *cache, int kernel, int B, int max_seq_len, int partition_tokens, unsigned flags)
{
    PassCut cut = {partition_tokens, (int)max_parts_for(max_seq_len, partition_tokens), 0, 0};
    if (partition_tokens <= 0 || kernel == KERNEL_VALU ||
        (flags & (0xFu | ADR_PARTIALS_ONLY | ADR_SINGLE_PARTITION_ITEMS)))
        return cut;
    // Rows of the cache one workgroup walks at a time (two kv-heads of 64 elements are taken together).
    const int64_t rows = (int64_t)B * (kernel == KERNEL_GRID && cache->d == 64 ? cache->Hkv / 2 : cache->Hkv);
    if (kernel == KERNEL_STREAM) {
        // With enough rows for its workgroups: an item's fixed cost is paid half as often with 1024
        // tokens as with 512, and there are half the partial results to merge (398 against 411 us at
        // 2048 pairs, fp8 237 against 254).
        if (rows >= 2048 && partition_tokens < 1024) {
            cut.tokens = partition_tokens * ((1024 + partition_tokens - 1) / partition_tokens);
            cut.max_parts = (int)max_parts_for(max_seq_len, cut.tokens);
        }
        return cut;
    }
    // One workgroup per item.  Short rows are not cut at all, which spares the merge (1 row of 300 tokens
    // 5.9 us against 7.4 in partitions of 128; 1600 rows of 100, bound 800, 32 against 35; 2048 rows of
    // 1500 241 against 277 in partitions of 512; fp8, whose items are half as heavy, 1200 rows of 1500
    // 92 against 102).
    const bool fp8 = cache->dtype == ADR_FP8_E4M3;
    if (max_seq_len <= (rows >= (fp8 ? 1024 : 2048) ? 2048 : rows >= 1024 ? 1024 : 512)) {
        cut.max_parts = 1;
        return cut;
    }
    // Otherwise into what makes about 1200 items of the pass (rows taken to be a quarter as long as the
    // bound on the average), 128 to 1024 tokens each: fewer leave compute units idle, more pay an item's
    // fixed cost (its chain of length, page table and first page, its combine, its place in the merge)
    // for nothing.  us with the merge, partitions of 128 / 256 / 512 / 1024 tokens:
    //     rows                   8              64               256              1024
    //     1000 tokens     8 /  9 / 11 / 11   14 / 14 / 14 / 18   30 / 30 / 32 / 31   111 / 100 /  97 / 100
    //     3000 tokens     9 / 10 / 12 / 18   25 / 25 / 27 / 33   83 / 75 / 74 / 79   327 / 297 / 280 / 266
    //     30000 tokens   31 / 28 / 26 / 25  208 /185 /171 /166
    // (an fp8 cache likewise).  The same length for every row: cut in proportion to their own lengths
    // instead, rows of mixed lengths end in long items (85 against 78 us at 1024 rows of heavy-tailed
    // lengths, 48 against 43 at 296).
    const auto share = [&](int64_t items) { // of a row's length, in units of 2^-32: `items` of the pass if all were as long
        return (uint32_t)std::min<int64_t>((rows << 32) / items, 0xffffffffLL);
    };
    cut.cut = adr::share_of_row(std::min(max_seq_len, adr::kCutLongRow), share(4800));
    // What the bound says beyond 8192 tokens is not taken for the rows' length (a serving system passes its
    // context limit): longer rows are cut by their own, to 3600 items if all were like them and 96 of a row
    // at most while that leaves partitions of 1024 tokens.  us per step, bound 131072 (1048576), partitions that grow with the
    // bound and these: one request of 2000 tokens 19.5 (22.7) and 10.7, of 20000 25.7 (115) and 23; 16 of 2000
    // 50 (56) and 30; 40 of median 1000 66 (93) and 50.
    cut.share = std::max(share(3600), (uint32_t)(((uint64_t)1 << 32) / 96));
    cut.max_parts = (int)std::min<int64_t>(max_parts_for(max_seq_len, cut.cut), cut.max_parts);
    return cut;
}

// Is a split pass planned on the device (plan.h), and served by one workgroup per item then?  Where there are
// at least as many rows as the chip holds workgroups: us a step, without a plan and with one, 256 requests x 8
// kv-heads of median length 1500 400 (the resident kernel) and 372, fp8 218 and 198, of 3000 tokens 528 and 509, 128 of
// 3000 285 and 260, of heavy-tailed lengths 77 and 68, one of 131072 tokens among 95 of 500 169 and 126; 768 x 1, one of
// 1000000 among rows of 64, 366 and 150 (a wave goes through its 559 partitions, eight at a time).
// With a third as many rows (plan_cut.h: kFew...; figures there) where an append kernel plans on its way and eight
// partitions are allowed.  There the mean is ahead and single shapes are not: of 256 to 304 rows 0.92 to 1.05 of the time
// without a plan, 0.995 in the mean of 64 shapes (of 320 and more 0.87 to 1.02); with four to seven partitions
// allowed 0.95 to 1.04, 0.996 over 32 shapes of 288 to 640 rows.
// No more than kPlanRows requests (plan_cut.h): 2048 x 1 of median length 700 take 292 without a plan and 194, 2049 307.
// Without an append kernel to plan on its way a kernel of its own does, and passes for the resident kernel stay
// with it (adr_decode_kernel_choice).  That kernel's 4 us are for nothing where the rows would stay whole in a short pass, and
// where they are of one length; so rows that stay whole without a plan are planned from a bound of kWholeBound tokens
// for each place on (us adr_kv_append and adr_decode_attention without and with a plan, rows of one length / up to it: 800 rows of
// 400 34.2 37.4 / -, 1024 of 900 81.7 85.1 / 48.0 49.1, 2048 of 300 56.8 57.0 / 33.6 33.9; 2048 of 1000 172 176 / 98 92, of 1600
// 279 278 / 153 141, of 2000 345 349 / 190 175, fp8 1280 of 1500 93.6 96.3 / 58.0 54.8).
constexpr int64_t kWholeBound = 2000;
// Tokens of a planned pass, over all kv-heads, from which the heads go in turn (decode_mfma.hip: a shorter pass is on the chip all at
// once).  us a step, in turn and in place: 32 requests x 8 kv-heads of 300 tokens 13.4 and 12.7, 48 of 100 11.8 and 11.3, 128 of 20 10.7
// and 10.3, 8 of 1000 x 4 among 56 of one token 14.6 and 13.8; 64 x 8 of 300 18.9 and 19.1, 256 of 100 24.9 and 25.2, 32 of 700
// 23.1 and 24.1; fp8 48 of 300 14.0 and 14.6, 32 of 300 12.0 and 11.8, 512 of 1 27.3 and 26.9.
constexpr uint32_t kTurnTokens[2] = {131072, 65536}; // bf16, fp8
bool plan_pass(adr::PlanParams &p, const adr_kv_cache *cache, int kernel, int B, int Hq, int max_seq_len,
               int partition_tokens, unsigned flags, bool step)
{
    p.items = nullptr;
    const int H = cache->d == 64 ? cache->Hkv / 2 : cache->Hkv;
    const int64_t max_parts = max_parts_for(max_seq_len, partition_tokens);
    if (kernel == KERNEL_VALU || (kernel == KERNEL_STREAM && (!step || (flags >> 16))) ||
        (flags & (0xFu | ADR_PARTIALS_ONLY | ADR_SINGLE_PARTITION_ITEMS | ADR_DEBUG_EXPIRE_WAITS)) ||
        B > adr::kPlanRows || (int64_t)B * H < (step && max_parts >= 8 ? adr::kSlots / 3 : adr::kSlots) || max_parts < 4 || !adr::decode_mfma_supports(cache->d, Hq / cache->Hkv, cache->Hkv))
        return false;
    p.part_counts = nullptr;
    p.arrivals = nullptr;
    p.heads = Hq;
    p.rule.few = (int64_t)B * H < adr::kSlots;
    p.rule.even_tiles = pass_cut(cache, KERNEL_GRID, B, max_seq_len, partition_tokens, flags).cut / adr::kPageSize;
    const bool whole_rows = p.rule.even_tiles == 0;
    if (whole_rows && (p.rule.few || (!step && (int64_t)B * H * max_seq_len < kWholeBound * adr::kSlots)))
        return false;
    p.rule.fill_rounds = cache->dtype == ADR_BF16;
    p.rule.max_parts = (int)std::min<int64_t>(max_parts - 1, 4096);
    p.rule.whole = kernel == KERNEL_STREAM ? adr::kManyTiles : adr::kPlanTiles;
    p.rule.heads_per_slot = (float)H / adr::kSlots;
    p.by_items = cache->dtype == ADR_BF16;
    p.turn_tiles = cache->dtype == ADR_BF16 && H < 4 ? ~0u : kTurnTokens[cache->dtype != ADR_BF16] / (adr::kPageSize * H);
    p.B = B;
    p.max_seq_len = max_seq_len;
    p.max_items = (int)adr::plan_places(B, H, max_seq_len, p.rule);
    // (behind the list: the merge kernel's partition counts, or the arrivals)
    const size_t behind = p.rule.few ? (size_t)B * sizeof(int32_t) : (size_t)B * Hq * adr::kArrivalWords * sizeof(uint32_t);
    return (size_t)p.max_items * sizeof(adr::u32x4) + behind <= (size_t)B * Hq * cache->d * sizeof(float);
}

constexpr unsigned kFlagBits = 0xFu | ADR_PARTIALS_ONLY | ADR_SINGLE_PARTITION_ITEMS | ADR_WORKSPACE_READY |
                               ADR_DEBUG_EXPIRE_WAITS | (0xFFFu << 16);

int decode_attention(void *out, adr_dtype out_dtype, float *lse, const void *q, int64_t q_row_stride,
                     const adr_kv_cache *cache, const int32_t *block_table, int max_pages_per_req,
                     const int32_t *seq_lens, int B, int Hq, float scale, int max_seq_len,
                     int partition_tokens, void *workspace, size_t workspace_bytes, unsigned flags,
                     void *stream, const NewToken *nt, bool static_scratch = false)
{
    const int rc = check_cache(cache);
    if (rc != ADR_OK)
        return rc;
    if (!out || !q || !block_table || !seq_lens)
        return ADR_ERR_NULL;
    if (nt) {
        if (!nt->k || !nt->v)
            return ADR_ERR_NULL;
        if (nt->row_stride < (int64_t)cache->Hkv * cache->d || (nt->row_stride % 8) != 0 ||
            !aligned16(nt->k) || !aligned16(nt->v))
            return ADR_ERR_SHAPE;
    }
    if (B < 0 || Hq <= 0 || max_pages_per_req <= 0 || max_seq_len < 0)
        return ADR_ERR_SHAPE;
    if (Hq % cache->Hkv != 0 || q_row_stride < (int64_t)Hq * cache->d || (q_row_stride % 8) != 0)
        return ADR_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(out))
        return ADR_ERR_SHAPE;
    if ((int64_t)max_seq_len > (int64_t)max_pages_per_req * cache->page_size)
        return ADR_ERR_SHAPE; // the table cannot describe that many tokens
    if (out_dtype != ADR_BF16 && out_dtype != ADR_F32)
        return ADR_ERR_UNSUPPORTED;
    if (partition_tokens < 0 || partition_tokens % cache->page_size != 0)
        return ADR_ERR_SHAPE;
    if (flags & ~kFlagBits)
        return ADR_ERR_UNSUPPORTED;
    const int G = Hq / cache->Hkv;
    const int d = cache->d;
    const bool fp8 = cache->dtype == ADR_FP8_E4M3;
    int kernel = choose_kernel(cache, B, Hq, max_seq_len, partition_tokens, flags);
    if (kernel < 0)
        return -kernel;
    const int64_t max_parts = max_parts_for(max_seq_len, partition_tokens);
    if ((int64_t)B * cache->Hkv * (max_parts + 1) > 0x7fffffffLL) // (+1: the grids take an odd number per row)
        return ADR_ERR_SHAPE;
    bool split = partition_tokens > 0 && max_parts > 1;
    const WorkspacePlan plan = plan_workspace(B, Hq, d, max_seq_len, partition_tokens);
    if (static_scratch) { // the library's own array stands in for the caller's workspace
        if (plan.total() > (size_t)ADR_STATIC_SCRATCH_BYTES)
            return ADR_ERR_WORKSPACE;
        if (flags & ADR_WORKSPACE_READY)
            return ADR_ERR_UNSUPPORTED; // calls of other sizes keep their control areas elsewhere in the array
        if (B == 0)
            return ADR_OK;
        const DeviceData *dd = nullptr;
        const int drc = device_data(&dd);
        if (drc != ADR_OK)
            return drc;
        workspace = dd->scratch;
        workspace_bytes = ADR_STATIC_SCRATCH_BYTES;
    }
    const bool workspace_fits =
        workspace && ((uintptr_t)workspace & 255u) == 0 && plan.total() > 0 && workspace_bytes >= plan.total();
    if (split && !workspace_fits)
        return ADR_ERR_WORKSPACE;
    if (B == 0)
        return ADR_OK;
    // One workgroup per item: the wave that brings a row's last partition may merge it (decode_mfma.hip), while the
    // queries of other rows are still to be read.  `out` may stand in q's place (an executor may well attend in
    // place: a head's result then replaces its own query, which nobody reads any more), but not across it.
    const size_t out_bytes = (size_t)B * Hq * d * (out_dtype == ADR_F32 ? 4 : 2);
    const bool in_place = out == q && out_dtype == ADR_BF16 && q_row_stride == (int64_t)Hq * d;
    bool meets = split && !(flags & ADR_PARTIALS_ONLY) &&
                 (in_place || !overlap(out, out_bytes, q, ((size_t)(B - 1) * q_row_stride + (size_t)Hq * d) * 2));
    PassCut cut;
    bool meet_bytes = false, appends = false;
    adr::PlanParams list;
    list.items = nullptr;
    if (meets && plan_pass(list, cache, kernel, B, Hq, max_seq_len, partition_tokens, flags, nt != nullptr)) {
        kernel = KERNEL_GRID;
        cut = {partition_tokens, list.rule.max_parts, 0, 0};
        list.items = (adr::u32x4 *)((char *)workspace + (size_t)B * list.rule.max_parts * Hq * d * sizeof(float));
        list.seq_lens = seq_lens;
        meets = !list.rule.few;
        if (meets)
            list.arrivals = (uint32_t *)(list.items + list.max_items);
        else
            list.part_counts = (int32_t *)(list.items + list.max_items);
    } else {
        cut = pass_cut(cache, kernel, B, max_seq_len, split ? partition_tokens : 0, flags);
        split = split && cut.max_parts > 1;
        const int64_t pairs = (int64_t)B * (d == 64 ? cache->Hkv / 2 : cache->Hkv), waves = pairs * adr::result_waves(G);
        // Small steps append inside the attention pass (NewTokens in decode_mfma.hip), unless that would read new tokens where
        // results or partial results have been written.  us a step, with an append kernel and inside: one request x 8 kv-heads of 2000 tokens
        // 10.0 and 8.8, three of 300 10.5 and 8.8, eight of 300 under a bound of 512 8.2 and 6.9, 24 of median length 1000 32.1
        // and 30.2, 28 of up to 6000 64.9 and 62.8, fp8 three of 2000 13.5 and 11.6.  One thing is slower, and the arguments do not tell it
        // from the others: up to three requests that all have 128 tokens or fewer, under bounds that would let them be split; they merged inside the
        // pass before, and nothing was to merge (replayed 5.8 and 6.2 us, called one by one 6.9 and 7.3; from 130 tokens on 8.3 and 7.5).
        // Up to 64 requests: their pages stand in one register; and to as many rows as the chip holds workgroups, beyond which 1.7 us
        // count for little.  Comparing pages costs a wave of an fp8 cache some 0.02 us a tile, and `longest` is what its partition may
        // have: whole rows (eight waves) of 4000 tokens 32.4 and 30.5, of 6000 in heads of 64 41.8 and 42.5, of 30000 179 and 191; up
        // to four partitions, which an append kernel's pass may merge inside: heads of 64 in partitions of 512 tokens 13.8 and 13.5, of
        // 1536 22.4 and 22.7, of 8192 76 and 78, heads of 128 of 1536 20.6 and 20.3, of 2560 26.3 and 26.6; more of them: four rows of 16000
        // tokens in partitions of up to 4096 27.9 and 26.6.  (bf16, twice the bytes a tile: whole rows of 6000 42.4 and 41.7, of 30000 256 and 255.)
        const int longest = !split ? max_seq_len : cut.cut ? (max_seq_len + cut.max_parts - 1) / cut.max_parts : cut.tokens;
        const int too_long = !fp8 ? INT_MAX : !split ? 4096 : cut.max_parts > 4 ? 8192 : d == 64 ? 1024 : 2048;
        if (nt && kernel == KERNEL_GRID && B <= 64 && pairs < adr::kSlots && longest < too_long) {
            const size_t new_bytes = ((size_t)(B - 1) * nt->row_stride + (size_t)cache->Hkv * d) * 2, lse_bytes = lse ? (size_t)B * Hq * sizeof(float) : 0;
            const auto apart = [&](const void *written, size_t bytes) {
                return !overlap(written, bytes, nt->k, new_bytes) && !overlap(written, bytes, nt->v, new_bytes);
            };
            appends = apart(out, out_bytes) && apart(lse, lse_bytes) && apart(workspace, workspace_fits ? plan.total() : 0);
        }
        // Without a plan, where an append kernel clears the words on its way: steps beyond 64 requests, those of an fp8 cache in long
        // partitions, and those whose new tokens share memory with what is written.  A pass that appends itself has nobody to clear the words.
        // Where each item has a compute unit to itself and rows have no more than 16 partitions, which a wave goes through by itself, and up to
        // 768 items where rows have few partitions: what the bound makes room for is mostly empty there.  Elsewhere an item of a split row
        // keeps its place until its results are in memory and counted, 3 us with the memory busy, and others wait for that place.
        // us a step, merged by a kernel of its own and inside (lengths uniform up to the bound): words, 65 requests x 1 kv-head
        // of up to 600 tokens 11.5 and 10.6, 127 x 1 of 1024 16.3 and 15.7, fp8 13.4 and 11.8, 16.0 and 14.9, two long partitions of 4 x 2 in heads
        // of 64 23.5 and 22.3; bytes, 100 x 2 of up to 600 13.8 and 13.0, of 1024 18.4 and 17.9, fp8 16.6 and 15.3; level or behind by 2 %
        // only at their edge (190 x 1 of 2048 25.5 and 26.1, groups of eight 14.0 and 14.1).
        // Without the limits (measured when small steps came here as well): three requests x 8 of 8000 tokens 23.7 and 24.2, 37 of median
        // 1000 51.2 and 54.5, fp8 256 of 1500 220 and 234; three rows of 24 partitions 33.5 and 36.9.
        meets = meets && split && nt && kernel == KERNEL_GRID && !appends;
        if (meets && !(cut.max_parts <= 16 && pairs * cut.max_parts <= adr::kSlots / 3 && waves <= adr::kMeetWords)) {
            meets = cut.max_parts <= 4 && (int64_t)B * cache->Hkv * cut.max_parts <= adr::kSlots && waves <= adr::kMeetBytes;
            meet_bytes = waves > adr::kMeetWords;
        }
    }

    adr::DecodeParams p;
    p.q = (const uint16_t *)q;
    p.q_row_stride = q_row_stride;
    p.k_cache = cache->k;
    p.v_cache = cache->v;
    p.k_scale = cache->k_scale;
    p.v_scale = cache->v_scale;
    p.block_table = block_table;
    p.seq_lens = seq_lens;
    p.out = out;
    p.lse = lse;
    p.part_o = nullptr;
    p.part_lse = nullptr;
    if (split) {
        p.part_o = (float *)workspace;
        p.part_lse = (float *)((char *)workspace + plan.part_o_bytes);
    }
    // A workspace that is large enough also carries the call's control area (an unsplit pass
    // may come with one too); a call without one falls back on the library's static pool.
    p.control = workspace_fits ? (uint32_t *)((char *)workspace + plan.part_o_bytes + plan.part_lse_bytes) : nullptr;
    p.max_pages = max_pages_per_req;
    p.page_shift = cache->page_size == 16 ? 0 : cache->page_size == 32 ? 1 : 2;
    p.B = B;
    p.Hq = Hq;
    p.Hkv = cache->Hkv;
    p.G = G;
    p.num_pages = cache->num_pages;
    p.partition_tokens = split ? cut.tokens : 0;
    p.max_parts = split ? cut.max_parts : 1;
    p.max_seq_len = max_seq_len;
    p.cut = split ? cut.cut : 0;
    p.cut_share = cut.share;
    p.out_f32 = out_dtype == ADR_F32;
    p.scale_log2e = scale * adr::kLog2e;
    p.coalesce = !(flags & ADR_SINGLE_PARTITION_ITEMS);
    p.spin_limit = (flags & ADR_DEBUG_EXPIRE_WAITS) ? 0 : adr::kSpinLimit;
    p.grid_cus = (int)((flags >> 16) & 0xFFFu);
    if (bounds_record(&p.bounds) != ADR_OK)
        return ADR_ERR_LAUNCH;
    list.bounds = p.bounds;

    // The control area must be all zero when the resident kernel starts, when a merge reads the status
    // block, and behind every call that was not told it is (adr.h: a later call may then vouch for it, or
    // the status be read).  A kernel that never touches it clears it on its way; ahead of the resident
    // one, and of counts in bytes, the append kernel does, or else a small kernel.
    const bool counts = meets && !list.items;
    meet_bytes = meet_bytes && counts;
    const bool clear_control = p.control && !(flags & ADR_WORKSPACE_READY);
    const bool clear_ahead = clear_control && (kernel == KERNEL_STREAM || meet_bytes);
    p.clear_words = clear_control && !clear_ahead ? plan.control_words() : 0;

    p.meet = !meets ? 0 : list.items ? 1 : adr::merge_slices((int64_t)B * Hq, cut.max_parts);
    p.items = list.items;
    p.meet_mask = p.max_parts >= 16 ? 15 : p.max_parts >= 8 ? 7 : p.max_parts >= 4 ? 3 : p.max_parts >= 2 ? 1 : 0;
    p.meet_bytes = meet_bytes;
    p.arrivals = list.items ? list.arrivals : nullptr;
    p.max_items = list.items ? list.max_items : 0;

    // The new token goes in first: the append kernel, with the token index taken from seq_lens.
    p.k_new = p.v_new = nullptr;
    if (appends) {
        p.k_new = (const uint16_t *)nt->k;
        p.v_new = (const uint16_t *)nt->v;
        p.new_row_stride = nt->row_stride;
        nt = nullptr;
    }
    if (nt) {
        adr::AppendParams ap;
        ap.k_cache = cache->k;
        ap.v_cache = cache->v;
        ap.k_scale = cache->k_scale;
        ap.v_scale = cache->v_scale;
        ap.k_new = (const uint16_t *)nt->k;
        ap.v_new = (const uint16_t *)nt->v;
        ap.new_row_stride = nt->row_stride;
        ap.block_table = block_table;
        ap.positions = nullptr;
        ap.seq_lens = seq_lens;
        ap.max_seq_len = max_seq_len;
        ap.page_size = cache->page_size;
        ap.max_pages = max_pages_per_req;
        ap.num_pages = cache->num_pages;
        ap.Hkv = cache->Hkv;
        ap.d = d;
        ap.B = B;
        ap.clear_words = clear_ahead ? p.control : nullptr; // on its way, for the kernels behind it
        ap.n_clear_words = clear_ahead ? plan.control_words() : 0;
        ap.meet = {counts && !meet_bytes ? p.part_lse : nullptr, p.max_parts, p.meet_mask, Hq};
        ap.plan = list;
        ap.bounds = p.bounds;
        if (adr::launch_kv_append(ap, fp8, (hipStream_t)stream) != hipSuccess)
            return ADR_ERR_LAUNCH;
    } else if (clear_ahead) {
        control_clear_kernel<<<1, 64, 0, (hipStream_t)stream>>>(p.control, plan.control_words());
        if (hipGetLastError() != hipSuccess)
            return ADR_ERR_LAUNCH;
    } else if (meets) {
        if (adr::launch_plan(list, (hipStream_t)stream) != hipSuccess)
            return ADR_ERR_LAUNCH;
    }
    hipError_t e = kernel == KERNEL_STREAM ? adr::launch_decode_stream(p, d, fp8, (hipStream_t)stream)
                   : kernel == KERNEL_GRID ? adr::launch_decode_mfma(p, d, fp8, (hipStream_t)stream)
                                           : adr::launch_decode_valu(p, d, fp8, (hipStream_t)stream);
    if (e != hipSuccess)
        return ADR_ERR_LAUNCH;
    if (split && !meets && !(flags & ADR_PARTIALS_ONLY)) {
        adr::MergeParams mp;
        mp.out = out;
        mp.lse_out = lse;
        mp.part_o = p.part_o;
        mp.part_lse = p.part_lse;
        mp.part_offsets = nullptr;
        mp.seq_lens = seq_lens;
        mp.partition_tokens = p.partition_tokens;
        mp.max_parts = p.max_parts;
        mp.max_seq_len = max_seq_len;
        mp.cut = p.cut;
        mp.cut_share = p.cut_share;
        mp.part_counts = list.items ? list.part_counts : nullptr;
        mp.B = B;
        mp.heads = Hq;
        mp.d = d;
        mp.out_f32 = p.out_f32;
        mp.status = kernel == KERNEL_STREAM ? p.control : nullptr; // the others have no wait that could expire
        e = adr::launch_lse_merge(mp, (hipStream_t)stream);
        if (e != hipSuccess)
            return ADR_ERR_LAUNCH;
    }
    return ADR_OK;
}

} // namespace

int adr_decode_attention(void *out, adr_dtype out_dtype, float *lse, const void *q,
                         int64_t q_row_stride, const adr_kv_cache *cache,
                         const int32_t *block_table, int max_pages_per_req,
                         const int32_t *seq_lens, int B, int Hq, float scale, int max_seq_len,
                         int partition_tokens, void *workspace, size_t workspace_bytes,
                         unsigned flags, void *stream)
{
    return decode_attention(out, out_dtype, lse, q, q_row_stride, cache, block_table, max_pages_per_req,
                            seq_lens, B, Hq, scale, max_seq_len, partition_tokens, workspace,
                            workspace_bytes, flags, stream, nullptr);
}

int adr_decode_attention_static(void *out, adr_dtype out_dtype, float *lse, const void *q, int64_t q_row_stride,
                                const adr_kv_cache *cache, const int32_t *block_table, int max_pages_per_req,
                                const int32_t *seq_lens, int B, int Hq, float scale, int max_seq_len,
                                int partition_tokens, unsigned flags, void *stream)
{
    return decode_attention(out, out_dtype, lse, q, q_row_stride, cache, block_table, max_pages_per_req,
                            seq_lens, B, Hq, scale, max_seq_len, partition_tokens, nullptr, 0, flags, stream,
                            nullptr, true);
}

int adr_decode_step(void *out, adr_dtype out_dtype, float *lse, const void *q, int64_t q_row_stride,
                    const void *k_new, const void *v_new, int64_t new_row_stride,
                    const adr_kv_cache *cache, const int32_t *block_table, int max_pages_per_req,
                    const int32_t *seq_lens, int B, int Hq, float scale, int max_seq_len,
                    int partition_tokens, void *workspace, size_t workspace_bytes, unsigned flags,
                    void *stream)
{
    const NewToken nt = {k_new, v_new, new_row_stride};
    return decode_attention(out, out_dtype, lse, q, q_row_stride, cache, block_table, max_pages_per_req,
                            seq_lens, B, Hq, scale, max_seq_len, partition_tokens, workspace,
                            workspace_bytes, flags, stream, &nt);
}

int adr_decode_merge(void *out, adr_dtype out_dtype, float *lse, const int32_t *seq_lens, int B,
                     int Hq, int d, int max_seq_len, int partition_tokens, const void *workspace,
                     size_t workspace_bytes, void *stream)
{
    if (!out || !seq_lens)
        return ADR_ERR_NULL;
    if (B < 0 || Hq <= 0 || max_seq_len < 0 || partition_tokens < 0 ||
        partition_tokens % adr::kPageSize != 0 || !aligned16(out))
        return ADR_ERR_SHAPE;
    if (d != 64 && d != 128)
        return ADR_ERR_UNSUPPORTED;
    if (out_dtype != ADR_BF16 && out_dtype != ADR_F32)
        return ADR_ERR_UNSUPPORTED;
    const int64_t max_parts = max_parts_for(max_seq_len, partition_tokens);
    if (partition_tokens == 0 || max_parts <= 1 || B == 0)
        return ADR_OK;
    const WorkspacePlan plan = plan_workspace(B, Hq, d, max_seq_len, partition_tokens);
    if (!workspace || ((uintptr_t)workspace & 255u) != 0 || workspace_bytes < plan.total())
        return ADR_ERR_WORKSPACE;
    adr::MergeParams mp;
    mp.out = out;
    mp.lse_out = lse;
    mp.part_o = (const float *)workspace;
    mp.part_lse = (const float *)((const char *)workspace + plan.part_o_bytes);
    mp.status = (const uint32_t *)((const char *)workspace + plan.part_o_bytes + plan.part_lse_bytes);
    mp.part_offsets = nullptr;
    mp.seq_lens = seq_lens;
    mp.partition_tokens = partition_tokens;
    mp.max_parts = (int)max_parts;
    mp.max_seq_len = max_seq_len;
    mp.cut = 0;
    mp.cut_share = 0;
    mp.part_counts = nullptr;
    mp.B = B;
    mp.heads = Hq;
    mp.d = d;
    mp.out_f32 = out_dtype == ADR_F32;
    return adr::launch_lse_merge(mp, (hipStream_t)stream) == hipSuccess ? ADR_OK : ADR_ERR_LAUNCH;
}

int adr_lse_merge(void *out, adr_dtype out_dtype, float *lse_out, const float *part_o,
                  const float *part_lse, const int32_t *part_offsets, int B, int heads, int d,
                  void *stream)
{
    if (!out || !part_o || !part_lse || !part_offsets)
        return ADR_ERR_NULL;
    if (B < 0 || heads <= 0)
        return ADR_ERR_SHAPE;
    if (d != 64 && d != 128)
        return ADR_ERR_UNSUPPORTED;
    if (out_dtype != ADR_BF16 && out_dtype != ADR_F32)
        return ADR_ERR_UNSUPPORTED;
    if (!aligned16(out) || !aligned16(part_o))
        return ADR_ERR_SHAPE;
    adr::MergeParams mp;
    mp.out = out;
    mp.lse_out = lse_out;
    mp.part_o = part_o;
    mp.part_lse = part_lse;
    mp.part_offsets = part_offsets;
    mp.seq_lens = nullptr;
    mp.partition_tokens = 0;
    mp.max_parts = 0;
    mp.max_seq_len = 0;
    mp.cut = 0;
    mp.cut_share = 0;
    mp.part_counts = nullptr;
    mp.B = B;
    mp.heads = heads;
    mp.d = d;
    mp.out_f32 = out_dtype == ADR_F32;
    mp.status = nullptr;
    return adr::launch_lse_merge(mp, (hipStream_t)stream) == hipSuccess ? ADR_OK : ADR_ERR_LAUNCH;
}

int adr_decode_kernel_choice(const adr_kv_cache *cache, int B, int Hq, int max_seq_len, int partition_tokens,
                             unsigned flags)
{
    const int rc = check_cache(cache);
    if (rc != ADR_OK)
        return -rc;
    if (B < 0 || Hq <= 0 || Hq % cache->Hkv != 0 || max_seq_len < 0 || partition_tokens < 0)
        return -ADR_ERR_SHAPE;
    return choose_kernel(cache, B, Hq, max_seq_len, partition_tokens, flags);
}

int adr_decode_step_kernel_choice(const adr_kv_cache *cache, int B, int Hq, int max_seq_len, int partition_tokens,
                                  unsigned flags)
{
    const int kernel = adr_decode_kernel_choice(cache, B, Hq, max_seq_len, partition_tokens, flags);
    adr::PlanParams list;
    return kernel > 0 && plan_pass(list, cache, kernel, B, Hq, max_seq_len, partition_tokens, flags, true) ? (int)KERNEL_GRID : kernel;
}

const char *adr_kernel_name(int kernel)
{
    switch (kernel) {
    case ADR_KERNEL_VALU: return "decode_valu_kernel";
    case ADR_KERNEL_MFMA: return "decode_stream_kernel";
    case ADR_KERNEL_MFMA_GRID: return "decode_mfma_kernel";
    default: return "";
    }
}

int adr_decode_read_status(const void *workspace, size_t workspace_bytes, int B, int Hq, int d, int max_seq_len,
                           int partition_tokens, uint32_t *expired_waits)
{
    if (!workspace || !expired_waits)
        return ADR_ERR_NULL;
    const WorkspacePlan plan = plan_workspace(B, Hq, d, max_seq_len, partition_tokens);
    if (plan.total() == 0 || ((uintptr_t)workspace & 255u) != 0 || workspace_bytes < plan.total())
        return ADR_ERR_WORKSPACE;
    const char *status = (const char *)workspace + plan.part_o_bytes + plan.part_lse_bytes;
    uint32_t word = 0;
    if (hipMemcpy(&word, status + 4 * adr::kStatusExpiredWaits, sizeof(word), hipMemcpyDeviceToHost) != hipSuccess)
        return ADR_ERR_LAUNCH;
    *expired_waits = word;
    return ADR_OK;
}

int adr_debug_bounds_status(adr_bounds_record *record, int reset)
{
#ifdef ADR_DEBUG_BOUNDS
    if (!record)
        return ADR_ERR_NULL;
    adr::BoundsRecord *dev = nullptr;
    if (bounds_record(&dev) != ADR_OK || !dev)
        return ADR_ERR_LAUNCH;
    adr::BoundsRecord host;
    if (hipMemcpy(&host, dev, sizeof(host), hipMemcpyDeviceToHost) != hipSuccess)
        return ADR_ERR_LAUNCH;
    record->count = host.count;
    record->kind = host.kind;
    record->row = host.row;
    record->index = host.index;
    record->value = host.value;
    if (reset && hipMemset(dev, 0, sizeof(host)) != hipSuccess)
        return ADR_ERR_LAUNCH;
    return ADR_OK;
#else
    (void)record;
    (void)reset;
    return ADR_ERR_UNSUPPORTED;
#endif
}

int adr_probe_stream_read(const void *src, size_t bytes, void *sink, void *stream)
{
    if (!src || !sink)
        return ADR_ERR_NULL;
    if (bytes % 16 != 0 || !aligned16(src))
        return ADR_ERR_SHAPE;
    return adr::launch_stream_read(src, bytes, sink, (hipStream_t)stream) == hipSuccess
               ? ADR_OK
               : ADR_ERR_LAUNCH;
}

int adr_probe_copy(void *dst, const void *src, size_t bytes, void *stream)
{
    if (!src || !dst)
        return ADR_ERR_NULL;
    if (bytes % 16 != 0 || !aligned16(src) || !aligned16(dst))
        return ADR_ERR_SHAPE;
    return adr::launch_copy(dst, src, bytes, (hipStream_t)stream) == hipSuccess ? ADR_OK
                                                                                : ADR_ERR_LAUNCH;
}

} // extern "C"
