"""GPU parity of the one-workgroup-per-item kernel where the library picks it by itself: two kv-heads of
64 elements taken side by side, rows cut finer or coarser than the caller's partitions, waves with more
tiles than one load of the page table brings, and the edges of tiles, waves and partitions in between."""
import types

import numpy as np
import pytest
import torch

import paper_2503_20552_amd as adr
import workloads as W
from gpu_util import ATOL, compare, dev, gpu_attention, oracle_attention, say

pytestmark = pytest.mark.gpu

# around the edges of a tile, of a workgroup's four waves, of partitions of 64, 128 and 512 tokens
EDGES = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1023, 1024, 1025]


def make(seed, Hq, Hkv, d, lens_after, page_size=16):
    lens_after = np.asarray(lens_after, dtype=np.int32)
    wl = W.Workload(96, "item", B=len(lens_after), Hq=Hq, Hkv=Hkv, d=d, lengths="given", page_size=page_size)
    b = W.make_batch(wl, device="cpu", headroom_tokens=1, seed_offset=seed, lens_before=np.maximum(lens_after - 1, 0))
    # (the slot of a row's last token, which no append has filled here, holds a value and not the poison)
    k, v = torch.nan_to_num(b.k_cache.float(), nan=0.25), torch.nan_to_num(b.v_cache.float(), nan=-0.5)
    return types.SimpleNamespace(wl=wl, q=b.q, k_cache=k.to(torch.bfloat16), v_cache=v.to(torch.bfloat16),
                                 block_table=b.block_table, seq_lens=lens_after, used=b.used)


def check(b, what, fp8=False, **kw):
    ref_kw = {}
    if fp8:     # pages no row owns keep NaN codes and NaN scales
        b.k_cache, ks = W.quantize_pool_fp8(b.k_cache, b.used)
        b.v_cache, vs = W.quantize_pool_fp8(b.v_cache, b.used)
        kw.update(k_scale=dev(ks), v_scale=dev(vs))
        ref_kw = dict(k_scale=W.bits(ks), v_scale=W.bits(vs))
    args = (dev(b.q), dev(b.k_cache), dev(b.v_cache), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    say(what)
    out, lse = gpu_attention(*args, **kw)
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale, **ref_kw)
    assert compare(out, lse, ref, ref_lse, what=what)[0] <= ATOL
    again, lse_again = gpu_attention(*args, **kw)
    assert torch.equal(out, again) and torch.equal(lse, lse_again)
    return out, lse


@pytest.mark.parametrize("G,Hkv", [(1, 2), (4, 8), (8, 2), (2, 6)])
@pytest.mark.parametrize("partition_tokens", [0, 64, 512])
@pytest.mark.parametrize("page_size", [16, 64])
def test_heads_of_64_in_pairs(G, Hkv, partition_tokens, page_size):
    b = make(G + Hkv, G * Hkv, Hkv, 64, EDGES, page_size)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    assert adr.adr_decode_kernel_choice(cache, len(EDGES), G * Hkv, 1025, partition_tokens) == adr.KERNEL_MFMA_GRID
    check(b, "pairs G=%d Hkv=%d part=%d page=%d" % (G, Hkv, partition_tokens, page_size),
          partition_tokens=partition_tokens)


@pytest.mark.parametrize("d,fp8", [(128, False), (128, True), (64, False), (64, True)])
def test_many_short_rows_are_items_as_they_are(d, fp8):
    # 2048 rows of the cache, bound 1025: not cut at all, whatever the caller's partitions
    Hkv = 32 if d == 128 else 64
    b = make(29, Hkv, Hkv, d, np.resize(EDGES, 64))
    out, _ = check(b, "short rows d=%d fp8=%s" % (d, fp8), fp8=fp8, partition_tokens=64)


def widen(b, bound):
    """The table has to describe as many tokens as the bound."""
    wide = np.zeros((b.block_table.shape[0], -(-bound // b.wl.page_size)), dtype=np.int32)
    wide[:, :b.block_table.shape[1]] = b.block_table
    b.block_table = wide


@pytest.mark.parametrize("d,G,fp8", [(128, 2, True), (128, 4, True), (64, 4, False)])
@pytest.mark.parametrize("partition_tokens", [0, 512])
def test_many_rows_under_an_ordinary_bound(d, G, fp8, partition_tokens):
    Hkv = 32 if d == 128 else 64                                   # 2048 rows of the cache
    b = make(37, G * Hkv, Hkv, d, np.resize(EDGES + [1500, 2100], 64))
    widen(b, 8192)
    check(b, "many rows d=%d G=%d fp8=%s part=%d" % (d, G, fp8, partition_tokens), fp8=fp8, partition_tokens=partition_tokens,
          max_seq_len=8192)


def test_a_kv_head_with_infinities_leaves_its_neighbour_alone():
    b = make(7, 8, 2, 64, [40, 700])
    k = b.k_cache.clone()
    k[:, :, 1, 5] = float("inf")
    args = (dev(b.q), dev(b.k_cache), dev(b.v_cache), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    say("infinities in the second of two kv-heads")
    clean, _ = gpu_attention(*args, partition_tokens=64)
    dirty, _ = gpu_attention(args[0], dev(k), *args[2:], partition_tokens=64)
    assert torch.equal(clean[:, :4], dirty[:, :4]) and not torch.equal(clean[:, 4:], dirty[:, 4:])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kernel", [adr.KERNEL_AUTO, adr.KERNEL_MFMA])
@pytest.mark.parametrize("partition_tokens", [0, 64])
def test_an_infinite_value_stays_infinite(d, kernel, partition_tokens):
    if d == 64 and kernel == adr.KERNEL_MFMA:
        pytest.skip("the resident kernel serves d = 128")
    b = make(9, 16, 4, d, [1, 40, 700, 1300])
    v = b.v_cache.clone()
    v[:, :, :, 5] = float("inf")            # every weight's every term meets one
    v[:, 3, :, 7] = -float("inf")
    args = (dev(b.q), dev(b.k_cache), dev(v), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    say("infinite values d=%d kernel=%d part=%d" % (d, kernel, partition_tokens))
    out, lse = gpu_attention(*args, partition_tokens=partition_tokens, flags=kernel)
    plain, plain_lse = gpu_attention(args[0], args[1], dev(b.v_cache), *args[3:], partition_tokens=partition_tokens, flags=kernel)
    assert (out[..., 5] == float("inf")).all() and (out[1:, :, 7] == -float("inf")).all()
    rest = [i for i in range(d) if i not in (5, 7)]
    assert torch.equal(out[..., rest], plain[..., rest]) and torch.equal(lse, plain_lse)


@pytest.mark.parametrize("Hkv,G", [(1, 4), (8, 2)])                # 1 .. 96 rows of the cache: partitions of 128
@pytest.mark.parametrize("bound", [None, 8192])                    # places of the workspace: 3 or 16 a row
def test_a_small_pass_is_cut_finer_than_the_callers_partitions(Hkv, G, bound):
    b = make(11 + Hkv, G * Hkv, Hkv, 128, [1, 128, 129, 2047, 2048, 2049, 0, 300, 1100][:9 if Hkv == 8 else 4])
    if bound:                                                     # the table has to describe that many tokens
        wide = np.zeros((b.block_table.shape[0], bound // 16), dtype=np.int32)
        wide[:, :b.block_table.shape[1]] = b.block_table
        b.block_table = wide
    out, _ = check(b, "finer Hkv=%d bound=%s" % (Hkv, bound), partition_tokens=1024, max_seq_len=bound)
    args = (dev(b.q), dev(b.k_cache), dev(b.v_cache), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    whole, _ = gpu_attention(*args, partition_tokens=1024, max_seq_len=bound, flags=adr.SINGLE_PARTITION_ITEMS)
    assert (not torch.equal(out, whole)) and (out - whole).abs().max().item() < 1e-4


def test_a_large_pass_is_cut_coarser_than_the_callers_partitions():
    b = make(13, 16, 16, 128, np.resize(EDGES + [1500, 2100], 64))       # 1024 rows of the cache
    out, _ = check(b, "coarser", partition_tokens=48)
    args = (dev(b.q), dev(b.k_cache), dev(b.v_cache), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    fine, _ = gpu_attention(*args, partition_tokens=48, flags=adr.SINGLE_PARTITION_ITEMS)
    assert (not torch.equal(out, fine)) and (out - fine).abs().max().item() < 1e-4


@pytest.mark.parametrize("d,G,Hkv", [(128, 1, 3), (128, 4, 8), (128, 16, 2), (64, 4, 8), (64, 8, 2), (64, 1, 2)])
@pytest.mark.parametrize("partition_tokens", [0, 64, 512])
@pytest.mark.parametrize("page_size", [16, 64])
def test_fp8_cache(d, G, Hkv, partition_tokens, page_size):
    b = make(19 + G + Hkv, G * Hkv, Hkv, d, EDGES, page_size)
    check(b, "fp8 d=%d G=%d Hkv=%d part=%d page=%d" % (d, G, Hkv, partition_tokens, page_size), fp8=True,
          partition_tokens=partition_tokens)


@pytest.mark.parametrize("B", [1, 7, 8, 9])        # (request, partition) units around whole turns of the eight chiplets
@pytest.mark.parametrize("Hkv", [1, 3, 8])
def test_fp8_every_item_is_done_once(B, Hkv):
    b = make(31 + B, 2 * Hkv, Hkv, 128, np.resize([1000, 17, 513, 0, 2100], B))
    check(b, "fp8 B=%d Hkv=%d" % (B, Hkv), fp8=True, partition_tokens=64)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("page_size", [16, 32])
@pytest.mark.parametrize("lens", [[2047, 33, 1], [4095, 4096, 4097, 3000], [8191, 8192, 8193, 8192 + 512, 8192 + 529, 33]])
def test_a_wave_with_more_tiles_than_one_load_of_the_table_brings(fp8, d, page_size, lens):
    # unsplit rows: 64 tiles of 16 tokens for each of four (a bound below 4096) or eight waves
    check(make(17, 4, 2, d, lens, page_size), "unsplit rows d=%d fp8=%s up to %d" % (d, fp8, max(lens)), fp8=fp8,
          partition_tokens=0)


@pytest.mark.parametrize("fp8", [False, True])
def test_four_waves_with_more_tiles_than_one_load_of_the_table_brings(fp8):
    # one partition of 4608 tokens: 72 tiles for each of four waves, and a ragged second partition
    b = make(23, 4, 2, 128, [4609, 4096, 4608, 100, 6000])
    check(b, "long partitions fp8=%s" % fp8, fp8=fp8, partition_tokens=4608, flags=adr.SINGLE_PARTITION_ITEMS)


# Workgroups per row: 33; what makes 68000 of them with 2061 rows or more; what makes 4096 with 124 or fewer.  Rows of one
# partition more or less than that, and of several times as many, under a bound that allows any number.
@pytest.mark.parametrize("B,Hkv,stride", [(40, 8, 33), (512, 8, 17), (1100, 8, 9), (2, 2, 1025)])
@pytest.mark.parametrize("fp8", [False, True])
def test_rows_with_more_partitions_than_workgroups(B, Hkv, stride, fp8):
    long = [16 * (stride + i) + j for i in (-1, 0, 1) for j in (0, 1)] + [16 * 3 * stride]
    lens = np.resize([1, 16, 17, 40, 300], B) if B > 8 else np.array(long[3:5])
    if B > 8:
        lens[np.arange(len(long)) * 5] = long
    b = make(43 + B, Hkv, Hkv, 128, lens)
    widen(b, 32768)
    flags = adr.SINGLE_PARTITION_ITEMS if fp8 else adr.KERNEL_MFMA_GRID       # the caller's partitions
    check(b, "looping workgroups B=%d Hkv=%d fp8=%s" % (B, Hkv, fp8), fp8=fp8, partition_tokens=16, max_seq_len=32768, flags=flags)


def partitions_of_a_pass(b, fp8, bound):
    """How many partitions a merging call with AUTO leaves in its workspace: the words of it that are written."""
    q, shape = dev(b.q), b.q.shape
    scales = [torch.ones(b.k_cache.shape[0], b.wl.Hkv, device="cuda:0") for _ in range(2)] if fp8 else (None, None)
    data = [dev(torch.randint(0, 0x40, x.shape, dtype=torch.uint8)) if fp8 else dev(x) for x in (b.k_cache, b.v_cache)]
    ws = torch.full((adr.adr_decode_workspace_bytes(*shape, bound, 512) // 4,), float("nan"), device="cuda:0")
    table = torch.zeros(shape[0], bound // 16, dtype=torch.int32, device="cuda:0")
    table[:, :b.block_table.shape[1]] = dev(b.block_table)
    adr.adr_decode_attention(torch.empty(shape, device="cuda:0"), q, adr.KVCache(*data, *scales), table, dev(b.seq_lens), b.wl.scale,
                             bound, 512, ws)
    torch.cuda.synchronize()
    control = 64 * (1 + -(-shape[0] // 512))
    return int((~torch.isnan(ws[:-control])).sum()) / (shape[1] * (shape[2] + 1))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("fp8", [False, True])
def test_a_bound_far_above_the_lengths_does_not_coarsen_the_cut(d, fp8):
    few = make(47, 8, 8, d, [2000, 1000, 1700])                # partitions of 128 tokens
    say("cut under loose bounds d=%d fp8=%s" % (d, fp8))
    assert [partitions_of_a_pass(few, fp8, n) for n in (8192, 32768, 131072, 1 << 20)] == [16 + 8 + 14] * 4
    for b in (make(48, 8, 8, d, [20000]), make(49, 8, 8, d, np.resize([1500, 3000], 40))):
        callers = int((-(-b.seq_lens // 512)).sum())
        for n in (32768, 131072, 1 << 20):
            assert partitions_of_a_pass(b, fp8, n) >= callers


@pytest.mark.parametrize("d,fp8", [(128, False), (128, True), (64, False)])
@pytest.mark.parametrize("bound", [8200, 32768, 1 << 20])
@pytest.mark.parametrize("lens", [[8191, 8192, 8193, 8320, 8321, 0, 1], [20000, 300], [16385, 12000] + [40] * 30])
def test_rows_around_the_length_from_which_they_are_cut_by_their_own(d, fp8, bound, lens):
    b = make(53, 8, 2, d, np.minimum(lens, bound))
    widen(b, bound)
    check(b, "long rows d=%d fp8=%s bound=%d %s" % (d, fp8, bound, lens[:3]), fp8=fp8, partition_tokens=512, max_seq_len=bound)


@pytest.mark.parametrize("bound,kernel", [(1024, adr.KERNEL_VALU), (1025, adr.KERNEL_MFMA_GRID)])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("partition_tokens", [0, 512])
def test_small_passes_of_single_heads_of_64(bound, kernel, fp8, partition_tokens):
    b = make(59, 8, 8, 64, [bound, 17, 0, 700])
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    assert adr.adr_decode_kernel_choice(cache, 4, 8, bound, partition_tokens) == kernel
    check(b, "single heads of 64, bound=%d fp8=%s part=%d" % (bound, fp8, partition_tokens), fp8=fp8, partition_tokens=partition_tokens)


VARIANTS = [(128, 4, 2, False), (128, 2, 3, True), (64, 4, 2, False), (64, 2, 4, True)]


@pytest.mark.parametrize("d,G,Hkv,fp8", VARIANTS)
@pytest.mark.parametrize("partition_tokens,page_size", [(16, 16), (48, 16), (64, 64), (512, 32)])
@pytest.mark.parametrize("apart", [False, True])
def test_the_callers_partitions(d, G, Hkv, fp8, partition_tokens, page_size, apart):
    """Calls that keep the caller's partitions (fewer tiles than waves among them): items of one partition each, and
    partials left in the workspace for adr_decode_merge."""
    b = make(61 + d, G * Hkv, Hkv, d, EDGES, page_size)
    scales = ()
    if fp8:
        b.k_cache, ks = W.quantize_pool_fp8(b.k_cache, b.used)
        b.v_cache, vs = W.quantize_pool_fp8(b.v_cache, b.used)
        scales = (ks, vs)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache), *map(dev, scales))
    bound, shape = int(b.seq_lens.max()), b.q.shape
    flags = adr.PARTIALS_ONLY if apart else adr.SINGLE_PARTITION_ITEMS
    assert adr.adr_decode_kernel_choice(cache, shape[0], shape[1], bound, partition_tokens, flags) == adr.KERNEL_MFMA_GRID
    out = torch.full(shape, float("nan"), device="cuda:0")
    lse = torch.full(shape[:2], float("nan"), device="cuda:0")
    ws = torch.full((adr.adr_decode_workspace_bytes(*shape, bound, partition_tokens) // 4,), float("nan"), device="cuda:0")
    say("callers' partitions d=%d fp8=%s part=%d page=%d apart=%s" % (d, fp8, partition_tokens, page_size, apart))
    table, lens = dev(b.block_table), dev(b.seq_lens)
    adr.adr_decode_attention(out, dev(b.q), cache, table, lens, b.wl.scale, bound, partition_tokens, ws, lse, flags)
    if apart:
        adr.adr_decode_merge(out, lens, bound, partition_tokens, ws, lse)
    torch.cuda.synchronize()
    ref_kw = dict(k_scale=W.bits(scales[0]), v_scale=W.bits(scales[1])) if fp8 else {}
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale, **ref_kw)
    assert compare(out, lse, ref, ref_lse, what="callers' partitions")[0] <= ATOL
    written = int((~torch.isnan(ws[:-64 * 2])).sum()) / (shape[1] * (d + 1))      # rows of one partition go to `out`
    counts = -(-b.seq_lens // partition_tokens)
    assert written == counts[counts > 1].sum()


@pytest.mark.parametrize("d,G,Hkv,fp8", VARIANTS[1:])
def test_debug_build_records_out_of_range_entries(d, G, Hkv, fp8):
    b = make(67, G * Hkv, Hkv, d, [40, 41, 201])
    table = b.block_table.copy()
    table[1, 0] = -5                               # clamps to page 0
    table[2, 3] = len(b.k_cache) + 1000            # clamps to the last page
    k, v, kw = b.k_cache, b.v_cache, {}
    if fp8:
        every = np.ones(len(b.k_cache), dtype=bool)    # (the clamped pages are read)
        k, ks = W.quantize_pool_fp8(b.k_cache, every)
        v, vs = W.quantize_pool_fp8(b.v_cache, every)
        kw = dict(k_scale=dev(ks), v_scale=dev(vs))
    args = (dev(b.q), dev(k), dev(v), dev(table), dev(b.seq_lens), b.wl.scale)
    say("debug build d=%d fp8=%s" % (d, fp8))
    release, release_lse = gpu_attention(*args, partition_tokens=64, **kw)
    with adr.debug_library():
        adr.adr_debug_bounds_status(reset=True)
        debug, debug_lse = gpu_attention(*args, partition_tokens=64, **kw)
        rec = adr.adr_debug_bounds_status(reset=True)
        assert rec["kind"] == 1 and rec["count"] >= 2
        assert (rec["row"], rec["index"], rec["value"]) in ((1, 0, -5), (2, 3, len(b.k_cache) + 1000))
        clean = dev(np.clip(table, 0, len(b.k_cache) - 1).astype(np.int32))
        again, _ = gpu_attention(*args[:3], clean, *args[4:], partition_tokens=64, **kw)
        assert adr.adr_debug_bounds_status()["count"] == 0
    assert torch.equal(release, debug) and torch.equal(release_lse, debug_lse) and torch.equal(release, again)
