"""Passes that are planned on the device (requests ordered by length, cut by the tokens the batch has, rows merged by the
wave that brings their last partition) and unplanned steps that merge the same way: against the oracle, on workspaces and
outputs full of NaN, at the edges of the rule, under bounds far above the lengths, and with `out` in q's place."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest
import torch

import paper_2503_20552_amd as adr
import oracle
import workloads as W
from gpu_util import ATOL, compare, dev, kernels_recorded, oracle_attention, say
from test_gpu_item_kernel import make, widen

gpu = pytest.mark.gpu
NAN = float("nan")


def run(b, cache, part, bound, entry="step", dtype=torch.float32, in_place=False, new=None):
    """(out, lse) of one call; a step appends the token that stands in the (bf16) cache already, unless `new` are given."""
    wl, q = b.wl, dev(b.q)
    out = q if in_place else torch.full(b.q.shape, NAN, dtype=dtype, device="cuda:0")
    lse = torch.full(b.q.shape[:2], NAN, device="cuda:0")
    ws = torch.full((adr.adr_decode_workspace_bytes(*b.q.shape, bound, part) // 4,), NAN, device="cuda:0")
    table, lens = dev(b.block_table), dev(b.seq_lens)
    if entry == "step":
        if new is None:
            at = np.maximum(b.seq_lens - 1, 0)
            page, slot = b.block_table[np.arange(wl.B), at // wl.page_size], at % wl.page_size
            new = [dev(t.cpu()[page, slot]) for t in (b.k_cache, b.v_cache)]
        adr.adr_decode_step(out, q, *new, cache, table, lens, wl.scale, bound, part, ws, lse)
    else:
        adr.adr_decode_attention(out, q, cache, table, lens, wl.scale, bound, part, ws, lse)
    torch.cuda.synchronize()
    assert adr.adr_decode_read_status(ws, *b.q.shape, bound, part) == 0
    return out, lse


def lengths(B, longest, kind):
    rng = np.random.default_rng(B + longest)
    n = {"mixed": rng.integers(0, min(200, longest + 1), B), "same": np.full(B, longest), "one": np.ones(B)}[kind].astype(np.int64)
    edges = [longest, 0, 1, 15, 16, 17, 127, 128, 129, 255, 256, 257, longest - 1, longest]
    if kind == "mixed":
        n[:len(edges)] = np.minimum(edges, longest)
    elif kind == "one":
        n[B // 2] = longest                        # a single long row among rows of one token
    return rng.permutation(n)


CASES = [(96, 8, 4, 128), (95, 8, 4, 128), (768, 1, 4, 128), (2048, 1, 2, 128), (2049, 1, 2, 128), (24, 32, 1, 128),
         (48, 16, 16, 128), (96, 16, 2, 64), (192, 8, 1, 64), (100, 8, 8, 128)]


@gpu
@pytest.mark.parametrize("B,Hkv,G,d", CASES)
@pytest.mark.parametrize("kind", ["mixed", "one"])
@pytest.mark.parametrize("entry", ["step", "attention"])
def test_planned_passes(B, Hkv, G, d, kind, entry):
    longest = 700
    b = make(71 + B, G * Hkv, Hkv, d, lengths(B, longest, kind))
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    say("planned B=%d Hkv=%d G=%d d=%d %s %s" % (B, Hkv, G, d, kind, entry))
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    for bound in (longest, 8192):
        if bound > longest:
            widen(b, bound)
        out, lse = run(b, cache, 128, bound, entry)
        assert compare(out, lse, ref, ref_lse, what="bound %d" % bound)[0] <= ATOL
        again, again_lse = run(b, cache, 128, bound, entry)
        assert torch.equal(out, again) and torch.equal(lse, again_lse)


@gpu
@pytest.mark.parametrize("B,Hkv,d", [(96, 8, 128), (64, 4, 128), (200, 4, 128), (100, 12, 128), (96, 16, 64)])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_heads_go_in_turn_from_so_many_tokens_on(B, Hkv, d, fp8, more):
    """A tile less than what the pass's heads go in turn from, as many, and one more; each head of each row once."""
    H = Hkv if d == 128 else Hkv // 2
    tiles = (65536 if fp8 else 131072) // (16 * H) + more
    per_row = np.full(B, tiles // B)
    per_row[:tiles % B] += 1
    b = make(113 + B + more, 2 * Hkv, Hkv, d, 16 * per_row - np.arange(B) % 7)
    widen(b, 4096)
    scales = [None, None]
    if fp8:
        b.k_cache, scales[0] = W.quantize_pool_fp8(b.k_cache, b.used)
        b.v_cache, scales[1] = W.quantize_pool_fp8(b.v_cache, b.used)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache), *(None if t is None else dev(t) for t in scales))
    new = [dev(torch.randn(B, Hkv, d, generator=torch.Generator().manual_seed(i)), torch.bfloat16) for i in range(2)]
    say("heads in turn B=%d Hkv=%d d=%d fp8=%s %+d" % (B, Hkv, d, fp8, more))
    out, lse = run(b, cache, 128, 4096, new=new)
    ref_kw = dict(k_scale=W.bits(cache.k_scale), v_scale=W.bits(cache.v_scale)) if fp8 else {}
    ref, ref_lse = oracle_attention(b.q, cache.k.cpu(), cache.v.cpu(), b.block_table, b.seq_lens, b.wl.scale, **ref_kw)
    assert compare(out, lse, ref, ref_lse, what="in turn")[0] <= ATOL


@gpu
@pytest.mark.parametrize("d,G,Hkv", [(128, 4, 8), (64, 2, 16)])
@pytest.mark.parametrize("places", [3, 4, 5, 33])
@pytest.mark.parametrize("entry", ["step", "attention"])
def test_planned_fp8_and_few_places(d, G, Hkv, places, entry):
    """Three partitions allowed: not planned; four: the list takes one's place and long rows have three."""
    part = 64
    b = make(73 + places, G * Hkv, Hkv, d, lengths(100, places * part, "mixed"))
    b.k_cache, ks = W.quantize_pool_fp8(b.k_cache, b.used)
    b.v_cache, vs = W.quantize_pool_fp8(b.v_cache, b.used)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache), dev(ks), dev(vs))
    say("planned fp8 d=%d places=%d %s" % (d, places, entry))
    new = [torch.randn(100, Hkv, d, generator=torch.Generator().manual_seed(i)).to(torch.bfloat16) for i in range(2)]
    if entry == "step":
        host = [W.bits(t).copy() for t in (b.k_cache, b.v_cache, ks, vs)]
        oracle.kv_append(*host[:2], *map(W.bits, new), b.block_table, b.seq_lens - 1, k_scale=host[2], v_scale=host[3])
    out, lse = run(b, cache, part, places * part, entry, new=[dev(t) for t in new])
    if entry == "step":
        for got, want in zip((cache.k, cache.v, cache.k_scale, cache.v_scale), host):
            assert np.array_equal(W.bits(got).view(np.uint8), want.view(np.uint8))
        b.k_cache, b.v_cache, ks, vs = (t.cpu() for t in (cache.k, cache.v, cache.k_scale, cache.v_scale))
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale,
                                    k_scale=W.bits(ks), v_scale=W.bits(vs))
    assert compare(out, lse, ref, ref_lse, what="fp8")[0] <= ATOL


@gpu
@pytest.mark.parametrize("B,kind", [(1, "same"), (3, "mixed"), (100, "mixed")])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("longest", [513, 1100, 1537, 5000])
def test_split_steps_small_and_planned(B, kind, dtype, longest):
    """Steps that append inside and are merged by the merge kernel, and planned ones whose rows meet; also with `out` in q's place."""
    b = make(79 + B, 32, 8, 128, lengths(max(B, 14), longest, kind)[:B] if kind == "mixed" else [longest] * B)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    say("split step B=%d %s %s longest=%d" % (B, kind, dtype, longest))
    bound = max(longest, int(b.seq_lens.max()))
    widen(b, bound)
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    out, lse = run(b, cache, 512, bound, dtype=dtype)
    compare(out, lse, ref, ref_lse, what="step")
    if B < 96:  # not planned: the two calls give the same bits
        two, two_lse = run(b, cache, 512, bound, "attention", dtype=dtype)
        assert torch.equal(out, two) and torch.equal(lse, two_lse)
    for entry in ("step", "attention"):
        out, lse = run(b, cache, 512, bound, entry, in_place=True)
        compare(out, lse, ref, ref_lse, what="in place, " + entry)


@gpu
@pytest.mark.parametrize("B,Hkv,G,d", [(32, 8, 4, 128), (31, 8, 4, 128), (95, 8, 8, 128), (256, 1, 4, 128), (64, 8, 4, 64)])
@pytest.mark.parametrize("kind", ["mixed", "same", "one"])
@pytest.mark.parametrize("allowed", [7, 8, 40])
def test_planned_steps_of_fewer_rows(B, Hkv, G, d, kind, allowed):
    """256 rows to 767, planned from eight partitions allowed on, merged by the merge kernel; rows of one length too."""
    longest = 128 * allowed
    b = make(89 + B, G * Hkv, Hkv, d, lengths(B, longest, kind))
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    say("planned step B=%d Hkv=%d G=%d d=%d %s allowed=%d" % (B, Hkv, G, d, kind, allowed))
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    out, lse = run(b, cache, 128, longest)
    assert compare(out, lse, ref, ref_lse, what="step")[0] <= ATOL
    again, again_lse = run(b, cache, 128, longest)
    assert torch.equal(out, again) and torch.equal(lse, again_lse)


@gpu
def test_a_plan_follows_the_lengths_of_each_replay():
    """One recorded step, replayed for other lengths; every replay against an eager call on other buffers."""
    longest = 900
    b = make(83, 32, 8, 128, lengths(100, longest, "same"))
    wl, part = b.wl, 128
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    q, table, new = dev(b.q), dev(b.block_table), [dev(torch.zeros(100, 8, 128), torch.bfloat16) for _ in range(2)]
    lens = dev(b.seq_lens)
    outs = [torch.full(b.q.shape, NAN, device="cuda:0") for _ in range(2)]
    wss = [torch.full((adr.adr_decode_workspace_bytes(*b.q.shape, longest, part) // 4,), NAN, device="cuda:0") for _ in range(2)]
    say("planned step recorded")
    def step(i):
        adr.adr_decode_step(outs[i], q, *new, cache, table, lens, wl.scale, longest, part, wss[i])
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        step(0)
    rng = np.random.default_rng(5)
    for replay in range(4):
        lens.copy_(dev(rng.integers(0, longest + 1, 100).astype(np.int32)))
        graph.replay()
        torch.cuda.synchronize()
        step(1)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]), "replay %d" % replay
        assert torch.isfinite(outs[0]).all()


@gpu
@pytest.mark.parametrize("page_size", [32, 64])
@pytest.mark.parametrize("B,Hkv,G,d,longest", [(100, 8, 4, 128, 700), (100, 16, 2, 64, 700), (40, 8, 4, 128, 1024), (3, 8, 4, 128, 900)])
@pytest.mark.parametrize("entry", ["step", "attention"])
def test_larger_pages(page_size, B, Hkv, G, d, longest, entry):
    """Pages of two and four tiles, whose partitions may begin inside a page, in every kind of pass."""
    b = make(107 + B, G * Hkv, Hkv, d, lengths(max(B, 14), longest, "mixed")[:B], page_size=page_size)
    b.seq_lens[0] = longest
    b = make(107 + B, G * Hkv, Hkv, d, b.seq_lens, page_size=page_size)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache))
    say("pages of %d B=%d d=%d %s" % (page_size, B, d, entry))
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    out, lse = run(b, cache, 128, longest, entry)
    assert compare(out, lse, ref, ref_lse, what="pages of %d" % page_size)[0] <= ATOL


@gpu
@pytest.mark.parametrize("B,Hkv,G,d,longest,part", [(100, 8, 4, 128, 700, 128), (100, 16, 2, 64, 700, 128), (40, 8, 4, 128, 1024, 128), (3, 8, 4, 128, 900, 128),
                                                    (3, 8, 2, 64, 900, 128), (80, 1, 2, 128, 900, 512), (100, 2, 4, 128, 900, 512)])
@pytest.mark.parametrize("where", [0, 1, -1])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_values_that_are_not_finite_meet(B, Hkv, G, d, longest, part, where, dtype):
    """Infinities and NaN in the values of one token, in a row's first, second or last partition: they come through the
    merge in their own columns and nowhere else."""
    b = make(109 + B, G * Hkv, Hkv, d, lengths(max(B, 14), longest, "mixed")[:B])
    b.seq_lens[0] = longest
    b = make(109 + B, G * Hkv, Hkv, d, b.seq_lens)
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    at = {0: 3, 1: longest // 3, -1: longest - 2}[where]
    b.v_cache[b.block_table[0, at // 16], at % 16, :, 5] = float("inf")
    b.v_cache[b.block_table[0, at // 16], at % 16, :, 6] = -float("inf")
    b.v_cache[b.block_table[0, at // 16], at % 16, :, 7] = NAN
    say("not finite B=%d d=%d at %d" % (B, d, at))
    out, lse = run(b, adr.KVCache(dev(b.k_cache), dev(b.v_cache)), part, longest, "step", dtype)
    assert (out[0, :, 5] == float("inf")).all() and (out[0, :, 6] == -float("inf")).all() and torch.isnan(out[0, :, 7]).all()
    out[0, :, 5:8] = torch.as_tensor(ref[0, :, 5:8]).to(out)
    # (bf16: half a unit in the last place of values below 8)
    assert compare(out, lse, ref, ref_lse, what="the rest")[0] <= (ATOL if dtype == torch.float32 else ATOL + 2.0 ** -6)


@gpu
@pytest.mark.parametrize("B,longest", [(2, 3000), (40, 4096), (100, 700)])
@pytest.mark.parametrize("entry", ["step", "attention"])
def test_out_in_the_place_of_an_input(B, longest, entry):
    """`out` in q's very place, over the new tokens, and in pinned host memory: the bits it has in memory of its own."""
    b = make(97 + B, 32, 8, 128, lengths(max(B, 14), longest, "mixed")[:B])
    b.seq_lens[0] = longest
    b = make(97 + B, 32, 8, 128, b.seq_lens)
    cache, part = adr.KVCache(dev(b.k_cache), dev(b.v_cache)), 128 if B == 100 else 512
    say("out in an input's place B=%d %s" % (B, entry))
    plain, lse = run(b, cache, part, longest, entry, dtype=torch.bfloat16)
    out, in_place_lse = run(b, cache, part, longest, entry, in_place=True)
    assert torch.equal(out, plain) and torch.equal(in_place_lse, lse)
    table, lens, ws = dev(b.block_table), dev(b.seq_lens), torch.empty(adr.adr_decode_workspace_bytes(*b.q.shape, longest, part), dtype=torch.uint8, device="cuda:0")
    host = torch.zeros(b.q.shape, dtype=torch.bfloat16, pin_memory=True)
    if entry == "attention":
        adr.adr_decode_attention(host, dev(b.q), cache, table, lens, b.wl.scale, longest, part, ws)
    else:
        at = np.maximum(b.seq_lens - 1, 0)
        page, slot = b.block_table[np.arange(B), at // 16], at % 16
        over = torch.zeros(b.q.shape, dtype=torch.bfloat16, device="cuda:0")
        new = over[:, 3:11], over[:, 17:25]
        for t, c in zip(new, (b.k_cache, b.v_cache)):
            t.copy_(dev(c.cpu()[page, slot]))
        adr.adr_decode_step(host, dev(b.q), *(t.clone() for t in new), cache, table, lens, b.wl.scale, longest, part, ws)
        adr.adr_decode_step(over, dev(b.q), *new, cache, table, lens, b.wl.scale, longest, part, ws)
        assert torch.equal(over, plain)
    torch.cuda.synchronize()
    assert torch.equal(host, plain.cpu())


# Steps that count arrivals: `over` has the new tokens in the memory of `out`, which keeps small ones from appending inside the
# attention pass; beyond 64 requests none does.  Kernels: append and attention, and the merge where they would be too many.
COUNTED = [(True, 1, 8, 16, 128, 16, 2), (True, 15, 8, 1, 128, 2, 2), (True, 16, 8, 1, 128, 2, 2), (True, 24, 8, 4, 128, 4, 2),
           (True, 31, 8, 4, 128, 3, 2), (True, 32, 8, 4, 128, 3, 3), (True, 15, 8, 8, 128, 4, 2), (True, 16, 8, 8, 128, 4, 3),
           (True, 15, 8, 8, 128, 6, 3), (True, 24, 16, 4, 64, 2, 2), (True, 48, 8, 1, 128, 2, 2), (True, 20, 8, 4, 64, 4, 2), (True, 3, 2, 1, 128, 7, 2),
           (False, 65, 1, 1, 128, 3, 2), (False, 80, 1, 2, 128, 2, 2), (False, 80, 2, 2, 64, 3, 2), (False, 127, 1, 1, 128, 2, 2),   # words
           (False, 128, 1, 1, 128, 2, 2), (False, 96, 1, 4, 128, 4, 2), (False, 97, 2, 1, 128, 3, 2), (False, 66, 3, 4, 128, 2, 2),  # bytes
           (False, 127, 2, 4, 128, 2, 2), (False, 128, 2, 4, 128, 2, 3), (False, 100, 4, 4, 64, 2, 3)]


@gpu
@pytest.mark.parametrize("over,B,Hkv,G,d,places,kernels", COUNTED)
@pytest.mark.parametrize("fp8", [False, True])
def test_small_steps_count_in_the_control_area(over, B, Hkv, G, d, places, kernels, fp8):
    """Up to 127 waves keep a word of the control area, up to 508 a byte; it is zero behind every call, vouched for or not, and
    the results are the two calls' bit for bit (also where they would be too many: 32 x 8 pairs, 16 x 8 in groups of eight)."""
    part = 512 if places == 2 else 256
    longest = part * places
    b = make(101 + B, G * Hkv, Hkv, d, [max(longest - 37 * i, 1 + i % 300) for i in range(B)])
    scales, new = [None, None], [torch.randn(B, Hkv, d, generator=torch.Generator().manual_seed(i)).to(torch.bfloat16) for i in range(2)]
    if fp8:
        b.k_cache, scales[0] = W.quantize_pool_fp8(b.k_cache, b.used)
        b.v_cache, scales[1] = W.quantize_pool_fp8(b.v_cache, b.used)
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache), *(None if t is None else dev(t) for t in scales))
    say("arrivals B=%d Hkv=%d G=%d d=%d fp8=%s" % (B, Hkv, G, d, fp8))
    q, table, lens, new = dev(b.q), dev(b.block_table), dev(b.seq_lens), [dev(t) for t in new]
    adr.adr_kv_append(cache, *new, table, lens - 1)
    two, two_lse = run(b, cache, part, longest, "attention")
    ws = torch.full((adr.adr_decode_workspace_bytes(*b.q.shape, longest, part) // 4,), NAN, device="cuda:0")
    for flags in (0, adr.WORKSPACE_READY, adr.WORKSPACE_READY, 0):
        out, lse = torch.full(b.q.shape, NAN, device="cuda:0"), torch.full(b.q.shape[:2], NAN, device="cuda:0")
        k_new = out.view(torch.bfloat16).view(-1)[:new[0].numel()].view(new[0].shape) if over else new[0]
        k_new.copy_(new[0])
        step = lambda: adr.adr_decode_step(out, q, k_new, new[1], cache, table, lens, b.wl.scale, longest, part, ws, lse, flags)
        step()
        torch.cuda.synchronize()
        assert torch.equal(out, two) and torch.equal(lse, two_lse)
        assert (ws[-128:].view(torch.int32) == 0).all()
    assert kernels_recorded(step) == kernels


@gpu
@pytest.mark.parametrize("entry,B,longest,part,kernels", [
    ("attention", 100, 400, 64, 1), ("attention", 128, 900, 128, 1), ("attention", 190, 1000, 128, 1),  # whole rows, short passes
    ("attention", 193, 1000, 128, 2), ("attention", 96, 700, 128, 2),                                   # a plan ahead
    ("step", 100, 400, 64, 2), ("step", 96, 700, 128, 2), ("step", 96, 700, 256, 3), ("step", 48, 1024, 128, 3)])
def test_launches_of_a_call(entry, B, longest, part, kernels):
    """The kernels a call records: no plan of its own for an attention pass whose rows stay whole anyway and are short."""
    cache = adr.KVCache(*(torch.zeros(longest // 16 + 1, 16, 8, 128, dtype=torch.bfloat16, device="cuda:0") for _ in range(2)))
    q = torch.zeros(B, 32, 128, dtype=torch.bfloat16, device="cuda:0")
    out, new = torch.zeros_like(q), torch.zeros(B, 8, 128, dtype=torch.bfloat16, device="cuda:0")
    table = torch.zeros(B, longest // 16 + 1, dtype=torch.int32, device="cuda:0")
    lens = torch.full((B,), longest, dtype=torch.int32, device="cuda:0")
    ws = torch.zeros(adr.adr_decode_workspace_bytes(B, 32, 128, longest, part), dtype=torch.uint8, device="cuda:0")
    say("launches of %s B=%d" % (entry, B))
    graph, stream = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        if entry == "step":
            adr.adr_decode_step(out, q, new, new, cache, table, lens, 0.1, longest, part, ws)
        else:
            adr.adr_decode_attention(out, q, cache, table, lens, 0.1, longest, part, ws)
    nodes = ctypes.c_size_t(0)
    count = adr.load_library().hipGraphGetNodes  # (the HIP runtime that the library itself is bound to)
    assert count(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0 and nodes.value == kernels


def test_the_step_choice_names_the_planned_passes():
    from test_abi_host import FAKE, cache
    lib = adr.load_library()
    def both(c, B, Hq, part=512, bound=8192, flags=0):
        return tuple(f(ctypes.byref(c), B, Hq, bound, part, flags) for f in (lib.adr_decode_kernel_choice, lib.adr_decode_step_kernel_choice))
    R, I, V = adr.KERNEL_MFMA, adr.KERNEL_MFMA_GRID, adr.KERNEL_VALU
    gqa = cache(Hkv=8)
    assert both(gqa, 256, 32) == both(gqa, 2048, 32) == (R, I) and both(gqa, 2049, 32) == (R, R)
    assert both(gqa, 256, 32, bound=1 << 20) == (R, I) and both(gqa, 256, 32, part=4096) == (R, R)
    assert both(gqa, 256, 32, flags=R) == (R, R) and both(gqa, 256, 32, flags=adr.GRID_CUS(64)) == (R, R)
    assert both(gqa, 256, 32, flags=adr.PARTIALS_ONLY) == both(gqa, 256, 32, flags=adr.SINGLE_PARTITION_ITEMS) == (R, R)
    assert both(gqa, 95, 32) == both(gqa, 96, 32) == (I, I) and both(cache(Hkv=1, d=64), 2000, 8) == (V, V)
    assert both(gqa, 256, 31)[1] < 0


SHIM = r"""
#include "plan_cut.h"
// The rows of a pass as plan.h cuts them: partitions and tokens of each, and the places of the list.
extern "C" long cut_rows(int few, int even_tiles, int fill_rounds, int whole, int max_parts, int H, int B, int bound, const int *L, int *parts, int *tokens)
{
    const adr::PlanRule rule = {few, even_tiles, fill_rounds, max_parts, (uint32_t)whole, (float)H / adr::kSlots};
    uint32_t all = 0, longest = 0;
    int rows = 0;
    for (int b = 0; b < B; ++b) {
        all += adr::plan_tiles(L[b]);
        rows += L[b] > 0;
        longest = adr::larger(longest, adr::plan_tiles(L[b]));
    }
    const adr::PlanCut cut = adr::plan_cut(rule, rows, all, longest);
    for (int b = 0; b < B; ++b)
        parts[b] = adr::plan_parts(L[b], cut, max_parts, tokens[b]);
    return (long)adr::plan_places(B, H, bound, rule);
}
"""


@pytest.fixture(scope="module")
def cut_rows(tmp_path_factory):
    """plan_cut.h compiled for the host: (rule, lengths) -> (partitions and tokens of each row, places of the list)."""
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(os.path.abspath(adr.__file__)), "csrc")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-I" + csrc, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    fn = ctypes.CDLL(str(d / "shim.so")).cut_rows
    fn.restype = ctypes.c_long
    def call(few, even_tiles, fill_rounds, max_parts, H, bound, L, whole=256):
        L = np.ascontiguousarray(L, dtype=np.int32)
        n, tokens = np.zeros_like(L), np.zeros_like(L)
        at = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        places = fn(int(few), int(even_tiles), int(fill_rounds), int(whole), int(max_parts), int(H), len(L), int(bound), at(L), at(n), at(tokens))
        return n.astype(np.int64), tokens.astype(np.int64), places
    return call


def test_planned_lists_fit_their_places(cut_rows):
    """Items never outnumber the places of their list; every row's partitions cover it, at most as many as it has places for."""
    rng = np.random.default_rng(11)
    for case in range(4000):
        few = case % 2 == 1
        H = int(rng.choice([1, 2, 4, 8, 32, 64]))
        B = int(rng.integers(-(-256 // H), -(-768 // H))) if few else int(np.clip(int(np.exp(rng.uniform(0, np.log(2048)))), -(-768 // H), 2048))
        bound = int(np.exp(rng.uniform(np.log(128), np.log((1 << int(rng.integers(10, 32))) - 1))))
        kind = rng.integers(6)
        L = (np.full(B, bound) if kind == 0 else rng.integers(0, bound + 1, B) if kind == 1 else
             np.exp(rng.uniform(0, math.log(bound), B)).astype(np.int64) if kind == 2 else
             np.full(B, rng.integers(1, bound + 1)) if kind == 3 else np.where(np.arange(B) % 10, 1, bound) if kind == 4 else
             np.where(np.arange(B) % 3, bound, 0)).astype(np.int64)
        places = min(max(-(-bound // 16) - 1, 3), 4096) if rng.integers(2) else int(rng.integers(3, 40))
        n, tokens, room = cut_rows(few, rng.integers(8, 65), rng.integers(2), places, H, bound, L, whole=256 << rng.integers(2))
        assert (n >= 1).all() and (n <= places).all(), (few, H, B, bound, kind)
        assert (n * tokens >= L).all() and ((n - 1) * tokens <= np.maximum(L - 1, 0)).all(), (few, H, B, bound, kind)
        assert n.sum() <= room and room % 8 == 0, (few, H, B, bound, kind)


@pytest.mark.parametrize("fill_rounds", [0, 1])
def test_rows_that_fill_up_a_batch_do_not_change_its_cut(cut_rows, fill_rounds):
    """Rows of one length in a recorded batch that is partly filled are cut as in a batch of their own: rows without tokens
    are no part of the mean that tells rows of one length from others."""
    for rows, length, even_tiles in [(33, 6000, 24), (40, 6000, 24), (48, 6000, 32), (33, 5900, 16), (60, 1000, 48), (64, 300, 56)]:
        for padding in (1, 15, 31):
            alone = cut_rows(1, even_tiles, fill_rounds, 63, 8, 8192, [length] * rows)
            padded = cut_rows(1, even_tiles, fill_rounds, 63, 8, 8192, [length] * rows + [0] * padding)
            assert np.array_equal(padded[0][:rows], alone[0]) and np.array_equal(padded[1][:rows], alone[1])
            assert (padded[0][rows:] == 1).all()
    # as without a plan where the larger partitions' last round is less than half full, or they are no larger; a bf16 cache
    tokens = lambda rows, length, even_tiles: int(cut_rows(1, even_tiles, fill_rounds, 63, 8, 8192, [length] * rows)[1][0])
    assert tokens(33, 6000, 24) == 384 and tokens(60, 1000, 48) == 512
    assert tokens(48, 6000, 32) == (2048 if fill_rounds else 512)


def test_rows_of_passes_that_the_resident_kernel_served_stay_whole(cut_rows):
    """512 requests of 5000 tokens and 256 of 8000, 8 kv-heads: whole rows up to 512 tiles there, halves elsewhere."""
    for rows, length in ((512, 5000), (256, 8000)):
        for whole, parts in ((256, 2), (512, 1)):
            n, tokens, _ = cut_rows(0, 0, 1, 15, 8, length, [length] * rows, whole=whole)
            assert (n == parts).all() and (n * tokens >= length).all()
