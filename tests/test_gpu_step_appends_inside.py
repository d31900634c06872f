"""Steps that append the new tokens inside the attention pass (up to 64 requests): against the two calls, bit for bit, with
requests that share pages in every way a table allows: a page some request appends to read by others before, at and behind the
new token's slot, a row's own page in its table twice, entries outside the pool, rows beyond the bound."""
import numpy as np
import pytest
import torch

import paper_2503_20552_amd as adr
import workloads as W
from gpu_util import dev, kernels_recorded, say

pytestmark = pytest.mark.gpu


def shared_pages(seed, B, page, longest, pages):
    """Lengths and a table over a small pool.  No two requests append to one slot, and none beside a token that sets its page's scales."""
    rng = np.random.default_rng(seed)
    L = rng.integers(0, longest + 1, B)
    edges = [1, page, page + 1, longest, 0, 2 * page, longest - 1, 17]
    L[:len(edges)] = np.minimum(edges, longest)[:B]
    table = rng.integers(0, pages, (B, -(-longest // page)))
    first, slots = set(), set()
    for b in range(B):
        if L[b] == 0:
            continue
        at, slot = divmod(int(L[b]) - 1, page)
        free = [p for p in rng.permutation(pages) if p not in first and (p, slot) not in slots and (slot or not any(q == p for q, _ in slots))]
        if not free:
            L[b] = 0
            continue
        table[b, at] = free[0]
        slots.add((free[0], slot))
        if slot == 0:
            first.add(free[0])
        if b % 3 == 1 and at:
            table[b, rng.integers(0, at)] = free[0]      # the page it appends to, earlier in its own table
    if B > 4:
        table[4, 0] = -3                                 # clamped to page 0, and nothing is appended where the last one is
        table[2, (max(int(L[2]), 1) - 1) // page] = pages + 9
    return L.astype(np.int32), table.astype(np.int32)


@pytest.mark.parametrize("d,G,Hkv,fp8", [(128, 4, 2, False), (64, 2, 4, False), (128, 4, 2, True), (64, 2, 4, True), (128, 16, 1, False)])
@pytest.mark.parametrize("B,longest", [(1, 40), (3, 700), (64, 300), (65, 300)])
@pytest.mark.parametrize("page,part", [(16, 0), (16, 64), (64, 512)])
def test_requests_that_share_pages(d, G, Hkv, fp8, B, longest, page, part):
    pages, Hq, scale = 2 * B + 9, G * Hkv, d ** -0.5
    gen = torch.Generator().manual_seed(B + longest)
    data = [torch.randn(pages, page, Hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    scales = [None, None]
    if fp8:
        data, scales = map(list, zip(*(W.quantize_pool_fp8(t, np.ones(pages, dtype=bool)) for t in data)))
    q, k_new, v_new = (dev(torch.randn(B, h, d, generator=gen), torch.bfloat16) for h in (Hq, Hkv, Hkv))
    for seed in range(3):
        L, table = shared_pages(seed, B, page, longest, pages)
        bound = longest - 3 if seed == 2 else longest    # rows beyond it are cut short and append nothing
        lens, entries = dev(L), dev(table)
        say("shared pages B=%d d=%d fp8=%s page=%d part=%d seed=%d" % (B, d, fp8, page, part, seed))
        got = []
        for one_call in (True, False):
            cache = adr.KVCache(*([dev(t) for t in data] + [None if s is None else dev(s) for s in scales]))
            out, lse = torch.full((B, Hq, d), float("nan"), device="cuda:0"), torch.full((B, Hq), float("nan"), device="cuda:0")
            ws = torch.full((max(adr.adr_decode_workspace_bytes(B, Hq, d, bound, part), 4) // 4,), float("nan"), device="cuda:0")
            if one_call:
                adr.adr_decode_step(out, q, k_new, v_new, cache, entries, lens, scale, bound, part, ws, lse)
            else:
                adr.adr_kv_append(cache, k_new, v_new, entries, dev(np.where(L > bound, -1, L - 1).astype(np.int32)))
                adr.adr_decode_attention(out, q, cache, entries, lens, scale, bound, part, ws, lse)
            torch.cuda.synchronize()
            got.append([out, lse, cache.k, cache.v] + ([cache.k_scale, cache.v_scale] if fp8 else []))
        for a, b in zip(*got):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), "seed %d" % seed
        assert torch.isfinite(got[0][0]).all()


@pytest.mark.parametrize("d,G,Hkv,fp8", [(128, 4, 2, False), (64, 2, 4, False), (128, 4, 2, True), (64, 2, 4, True)])
@pytest.mark.parametrize("page,part", [(16, 0), (16, 64), (64, 512)])
def test_requests_that_append_to_one_slot(d, G, Hkv, fp8, page, part):
    """Rows that fill up a batch may all be one token on one page: the last one's token stands for all, in the cache and in what
    every row attends, as if each had brought that token."""
    B, longest = 64, 700
    rng = np.random.default_rng(page + d)
    L = np.where(np.arange(B) % 8 == 3, rng.integers(page + 2, longest + 1, B), 1)
    L[[5, 21, 62]] = page + 2                            # three rows behind a page that all of them share
    L[0] = longest
    need = -(-L // page)
    table = np.zeros((B, -(-longest // page)), dtype=np.int64)
    at = 3
    for b in range(B):
        if L[b] == 1:
            table[b] = 0
        elif b in (5, 21, 62):
            table[b, :2] = 1, 2
        else:
            table[b, :need[b]] = at + np.arange(need[b])
            at += need[b]
    gen = torch.Generator().manual_seed(d)
    data = [torch.randn(at, page, Hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    scales = [None, None]
    if fp8:
        data, scales = map(list, zip(*(W.quantize_pool_fp8(t, np.ones(at, dtype=bool)) for t in data)))
    q, k_new, v_new = (dev(torch.randn(B, h, d, generator=gen), torch.bfloat16) for h in (G * Hkv, Hkv, Hkv))
    bring = np.arange(B)
    bring[L == 1] = np.nonzero(L == 1)[0][-1]
    bring[[5, 21, 62]] = 62
    lens, entries, scale = dev(L.astype(np.int32)), dev(table.astype(np.int32)), d ** -0.5
    say("one slot d=%d fp8=%s page=%d part=%d" % (d, fp8, page, part))
    got = []
    for one_call in (True, False):
        cache = adr.KVCache(*([dev(t) for t in data] + [None if s is None else dev(s) for s in scales]))
        out, lse = torch.full((B, G * Hkv, d), float("nan"), device="cuda:0"), torch.full((B, G * Hkv), float("nan"), device="cuda:0")
        ws = torch.full((max(adr.adr_decode_workspace_bytes(B, G * Hkv, d, longest, part), 4) // 4,), float("nan"), device="cuda:0")
        if one_call:
            adr.adr_decode_step(out, q, k_new, v_new, cache, entries, lens, scale, longest, part, ws, lse)
        else:
            adr.adr_kv_append(cache, k_new[bring].contiguous(), v_new[bring].contiguous(), entries, lens - 1)
            adr.adr_decode_attention(out, q, cache, entries, lens, scale, longest, part, ws, lse)
        torch.cuda.synchronize()
        got.append([out, lse, cache.k, cache.v] + ([cache.k_scale, cache.v_scale] if fp8 else []))
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("B,part,over,kernels", [
    (64, 0, None, 1), (65, 0, None, 2), (64, 256, None, 2), (65, 256, None, 3),   # with the append inside and, from 65 on, without
    (64, 0, "out", 2), (64, 256, "out", 3), (64, 0, "lse", 2), (64, 256, "lse", 3), (64, 256, "workspace", 3)])
def test_which_steps_append_inside(B, part, over, kernels):
    """The kernels of a step, and its results where they take the place of the new tokens, which must all be read before."""
    Hkv, G, d, page, bound = 2, 16, 128, 16, 300 if part == 0 else 1000
    rng = np.random.default_rng(B)
    L = rng.integers(1, bound + 1, B).astype(np.int32)
    wide = -(-bound // page)
    table = rng.permutation(B * wide).reshape(B, wide).astype(np.int32)
    gen = torch.Generator().manual_seed(B + part)
    data = [torch.randn(B * wide, page, Hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    q, k_new, v_new = (dev(torch.randn(B, h, d, generator=gen), torch.bfloat16) for h in (G * Hkv, Hkv, Hkv))
    lens, entries, ws_bytes = dev(L), dev(table), max(adr.adr_decode_workspace_bytes(B, G * Hkv, d, bound, part), 256)
    say("step route B=%d part=%d over=%s" % (B, part, over))
    got = []
    for apart in (True, False):
        cache = adr.KVCache(*(dev(t) for t in data))
        ws = torch.full((ws_bytes // 4,), float("nan"), device="cuda:0")
        out, lse = torch.zeros(B, G * Hkv, d, dtype=torch.bfloat16, device="cuda:0"), torch.zeros(B, G * Hkv, device="cuda:0")
        new = [k_new.clone(), v_new.clone()]
        if not apart and over:
            memory = {"out": out.view(-1), "lse": torch.zeros(B * Hkv * d, dtype=torch.bfloat16, device="cuda:0"), "workspace": ws.view(torch.bfloat16)}[over]
            if over == "lse":
                lse = memory.view(torch.float32)[:lse.numel()].view(lse.shape)
            new[1] = memory[:v_new.numel()].view(v_new.shape)
            new[1].copy_(v_new)
        call = lambda: adr.adr_decode_step(out, q, *new, cache, entries, lens, d ** -0.5, bound, part, ws, lse)
        call()
        torch.cuda.synchronize()
        got.append([out, lse, cache.k, cache.v])
        nodes = kernels_recorded(call)
    assert nodes == kernels
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("d,Hkv,fp8,bound,part,kernels", [
    (128, 8, True, 4095, 0, 1), (128, 8, True, 4096, 0, 2), (128, 8, False, 4096, 0, 1), (64, 16, True, 4096, 0, 2), (64, 16, False, 9000, 0, 1),
    (128, 8, True, 4094, 2048, 2), (128, 8, True, 4096, 2048, 3), (128, 8, False, 4096, 2048, 2), (64, 16, True, 2046, 1024, 2), (64, 16, True, 2048, 1024, 3),
    (64, 16, False, 2048, 1024, 2), (128, 8, True, 40000, 8000, 2), (128, 8, True, 49152, 8192, 3), (64, 16, True, 5120, 1024, 2)])
def test_long_partitions_of_an_fp8_cache_keep_the_append_kernel(d, Hkv, fp8, bound, part, kernels):
    """By what a partition may have at most; so many rows that none merge inside the pass."""
    B, G = 48, 16 if d == 128 else 8
    shape = (bound // 16 + 1, 16, Hkv, d)
    if fp8:
        cache = adr.KVCache(*(torch.zeros(shape, dtype=torch.uint8, device="cuda:0") for _ in range(2)), *(torch.ones(shape[0], Hkv, device="cuda:0") for _ in range(2)))
    else:
        cache = adr.KVCache(*(torch.zeros(shape, dtype=torch.bfloat16, device="cuda:0") for _ in range(2)))
    q, new = (torch.zeros(B, h, d, dtype=torch.bfloat16, device="cuda:0") for h in (G * Hkv, Hkv))
    out, lens = torch.zeros_like(q), torch.full((B,), 17, dtype=torch.int32, device="cuda:0")
    table = torch.arange(shape[0], dtype=torch.int32, device="cuda:0").repeat(B, 1)
    ws = torch.zeros(max(adr.adr_decode_workspace_bytes(B, G * Hkv, d, bound, part), 256), dtype=torch.uint8, device="cuda:0")
    say("append kernel of long partitions d=%d fp8=%s bound=%d part=%d" % (d, fp8, bound, part))
    assert kernels_recorded(lambda: adr.adr_decode_step(out, q, new, new, cache, table, lens, d ** -0.5, bound, part, ws)) == kernels


@pytest.mark.parametrize("d,G,Hkv,fp8", [(128, 4, 2, False), (64, 2, 4, False), (128, 4, 2, True), (64, 2, 4, True)])
@pytest.mark.parametrize("page,part", [(16, 0), (64, 128)])
def test_new_tokens_that_are_not_finite(d, G, Hkv, fp8, page, part):
    """Infinities and NaN among the new tokens' elements, as the first token of a page and later in it: the two calls' bits."""
    L = np.array([1, 5, page + 1, 3 * page + 7, 600, 40 * page // page + 1], dtype=np.int32)
    B, wide = len(L), -(-600 // page)
    table = np.arange(B * wide).reshape(B, wide).astype(np.int32)
    gen = torch.Generator().manual_seed(d + page)
    data = [torch.randn(B * wide, page, Hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    scales = [None, None]
    if fp8:
        data, scales = map(list, zip(*(W.quantize_pool_fp8(t, np.ones(B * wide, dtype=bool)) for t in data)))
    q, k_new, v_new = (dev(torch.randn(B, h, d, generator=gen), torch.bfloat16) for h in (G * Hkv, Hkv, Hkv))
    for i, x in enumerate((float("inf"), -float("inf"), float("nan"))):
        k_new[i::4, i % Hkv, 3 + i], v_new[i::4, (i + 1) % Hkv, 9 + i] = x, x
    lens, entries = dev(L), dev(table)
    say("new tokens not finite d=%d fp8=%s page=%d part=%d" % (d, fp8, page, part))
    got = []
    for one_call in (True, False):
        cache = adr.KVCache(*([dev(t) for t in data] + [None if s is None else dev(s) for s in scales]))
        out, lse = torch.zeros(B, G * Hkv, d, device="cuda:0"), torch.zeros(B, G * Hkv, device="cuda:0")
        ws = torch.full((max(adr.adr_decode_workspace_bytes(B, G * Hkv, d, 600, part), 4) // 4,), float("nan"), device="cuda:0")
        if one_call:
            adr.adr_decode_step(out, q, k_new, v_new, cache, entries, lens, d ** -0.5, 600, part, ws, lse)
        else:
            adr.adr_kv_append(cache, k_new, v_new, entries, lens - 1)
            adr.adr_decode_attention(out, q, cache, entries, lens, d ** -0.5, 600, part, ws, lse)
        torch.cuda.synchronize()
        got.append([out, lse, cache.k, cache.v] + ([cache.k_scale, cache.v_scale] if fp8 else []))
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert torch.isfinite(got[0][0][3]).all() and not torch.isfinite(got[0][0][:3]).all()


@pytest.mark.parametrize("d,G,Hkv,fp8,bound,part", [(128, 4, 2, False, 16384, 8192), (64, 2, 4, False, 16384, 8192), (128, 4, 2, True, 40000, 8000),
                                                    (64, 2, 4, True, 40000, 8000), (128, 4, 2, False, 9000, 0)])
@pytest.mark.parametrize("page", [16, 64])
def test_waves_of_more_tiles_than_a_load_of_the_table_brings(d, G, Hkv, fp8, bound, part, page):
    """More than 64 tiles a wave (the next ids, and an fp8 cache's scales, arrive beside the new token): the two calls' bits."""
    L = np.array([bound, bound - page, bound // 2 + 1, 4 * 64 * 16 * max(bound // part, 1) + 1 if part else 8193, 4097, 17], dtype=np.int32)
    B, wide = len(L), -(-bound // page)
    need = -(-L // page)
    table = np.zeros((B, wide), dtype=np.int32)
    start = np.concatenate([[0], np.cumsum(need)])
    for b in range(B):
        table[b, :need[b]] = start[b] + np.random.default_rng(b).permutation(need[b])
    gen = torch.Generator().manual_seed(d + page)
    data = [torch.randn(start[-1], page, Hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    scales = [None, None]
    if fp8:
        data, scales = map(list, zip(*(W.quantize_pool_fp8(t, np.ones(start[-1], dtype=bool)) for t in data)))
    q, k_new, v_new = (dev(torch.randn(B, h, d, generator=gen), torch.bfloat16) for h in (G * Hkv, Hkv, Hkv))
    lens, entries = dev(L), dev(table)
    say("many tiles a wave d=%d fp8=%s bound=%d part=%d page=%d" % (d, fp8, bound, part, page))
    got = []
    for one_call in (True, False):
        cache = adr.KVCache(*([dev(t) for t in data] + [None if s is None else dev(s) for s in scales]))
        out, lse = torch.full((B, G * Hkv, d), float("nan"), device="cuda:0"), torch.full((B, G * Hkv), float("nan"), device="cuda:0")
        ws = torch.full((max(adr.adr_decode_workspace_bytes(B, G * Hkv, d, bound, part), 4) // 4,), float("nan"), device="cuda:0")
        step = lambda: adr.adr_decode_step(out, q, k_new, v_new, cache, entries, lens, d ** -0.5, bound, part, ws, lse)
        if one_call:
            step()
        else:
            adr.adr_kv_append(cache, k_new, v_new, entries, lens - 1)
            adr.adr_decode_attention(out, q, cache, entries, lens, d ** -0.5, bound, part, ws, lse)
        torch.cuda.synchronize()
        got.append([out, lse, cache.k, cache.v] + ([cache.k_scale, cache.v_scale] if fp8 else []))
        if one_call:
            assert kernels_recorded(step) == (2 if part else 1)
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert torch.isfinite(got[0][0]).all()


@pytest.mark.parametrize("d,G,Hkv,fp8", [(128, 4, 2, False), (64, 2, 4, True)])
def test_debug_build_records_what_is_not_appended(d, G, Hkv, fp8):
    """A step whose request 1 would append to a page outside the pool: recorded as often as by the two calls, nothing is written
    for it, and the results are the release build's."""
    page, L, table = 16, np.array([40, 41, 180], dtype=np.int32), np.arange(3 * 13).reshape(3, 13).astype(np.int32)
    pages = table.size
    table[1, 2] = pages + 7
    gen = torch.Generator().manual_seed(d)
    data = [torch.randn(pages, page, Hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    scales = [None, None]
    if fp8:
        data, scales = map(list, zip(*(W.quantize_pool_fp8(t, np.ones(pages, dtype=bool)) for t in data)))
    q, k_new, v_new = (dev(torch.randn(3, h, d, generator=gen), torch.bfloat16) for h in (G * Hkv, Hkv, Hkv))
    lens, entries = dev(L), dev(table)

    def call(one_call):
        cache = adr.KVCache(*([dev(t) for t in data] + [None if s is None else dev(s) for s in scales]))
        out = torch.full((3, G * Hkv, d), float("nan"), device="cuda:0")
        if one_call:
            adr.adr_decode_step(out, q, k_new, v_new, cache, entries, lens, d ** -0.5, 208, 0, None)
        else:
            adr.adr_kv_append(cache, k_new, v_new, entries, lens - 1)
            adr.adr_decode_attention(out, q, cache, entries, lens, d ** -0.5, 208, 0, None)
        torch.cuda.synchronize()
        return out, cache

    say("debug record of a step d=%d fp8=%s" % (d, fp8))
    release, _ = call(True)
    with adr.debug_library():
        records = []
        for one_call in (True, False):
            adr.adr_debug_bounds_status(reset=True)
            out, cache = call(one_call)
            records.append(adr.adr_debug_bounds_status(reset=True))
            assert torch.equal(out, release)
            assert torch.equal(cache.k[pages - 1].cpu(), data[0][pages - 1])      # (the page its entry is clamped to)
        for r in records:
            assert (r["row"], r["index"], r["value"]) == (1, 2, pages + 7) and r["kind"] in (1, 3)
        assert records[0]["count"] == records[1]["count"] > 1
