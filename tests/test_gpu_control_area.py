"""Every call leaves its workspace's control area zero, whichever kernel serves it: on a workspace of 0xFF
bytes the status reads 0 behind the call, partials taken by a call that vouches for the area merge to
the right result, and the resident kernel may start on it."""
import numpy as np
import pytest
import torch

import paper_2503_20552_amd as adr
import workloads as W
from gpu_util import compare, dev, oracle_attention, say
from test_gpu_item_kernel import make

pytestmark = pytest.mark.gpu

LENS = [700, 1, 64, 65, 513, 1300]


def call(entry, b, cache, ws, part, flags):
    t = dict(out=torch.full(b.q.shape, float("nan"), device="cuda:0"), q=dev(b.q), cache=cache, block_table=dev(b.block_table),
             seq_lens=dev(b.seq_lens), scale=b.wl.scale, max_seq_len=int(b.seq_lens.max()), partition_tokens=part, workspace=ws,
             lse=torch.full(b.q.shape[:2], float("nan"), device="cuda:0"), flags=flags)
    if entry is adr.adr_decode_step:
        rng = torch.Generator().manual_seed(3)
        new = [dev(torch.randn(b.wl.B, b.wl.Hkv, b.wl.d, generator=rng), torch.bfloat16) for _ in range(2)]
        t.update(k_new=new[0], v_new=new[1])
    entry(**t)
    return t


@pytest.mark.parametrize("entry", [adr.adr_decode_attention, adr.adr_decode_step])
@pytest.mark.parametrize("d,Hkv,fp8,flags,kernel", [
    (128, 2, False, adr.KERNEL_AUTO, adr.KERNEL_MFMA_GRID), (128, 2, True, adr.KERNEL_AUTO, adr.KERNEL_MFMA_GRID),
    (64, 2, False, adr.KERNEL_AUTO, adr.KERNEL_MFMA_GRID), (64, 2, True, adr.KERNEL_AUTO, adr.KERNEL_MFMA_GRID),
    (64, 1, False, adr.KERNEL_AUTO, adr.KERNEL_VALU), (128, 2, False, adr.KERNEL_VALU, adr.KERNEL_VALU),
    (128, 2, False, adr.KERNEL_MFMA, adr.KERNEL_MFMA)])
@pytest.mark.parametrize("part,rows", [(64, 1), (0, 1), (64, 100)])       # 100: 600 rows, three blocks of the area
def test_a_call_leaves_the_control_area_zero(entry, d, Hkv, fp8, flags, kernel, part, rows):
    b = make(41 + d, 4 * Hkv, Hkv, d, LENS if rows == 1 else np.resize([16, 1, 100, 40], 6 * rows))
    scales = ()
    if fp8:
        b.k_cache, ks = W.quantize_pool_fp8(b.k_cache, b.used)
        b.v_cache, vs = W.quantize_pool_fp8(b.v_cache, b.used)
        scales = (dev(ks), dev(vs))
    cache = adr.KVCache(dev(b.k_cache), dev(b.v_cache), *scales)
    wl, bound = b.wl, int(b.seq_lens.max())
    assert adr.adr_decode_kernel_choice(cache, wl.B, wl.Hq, bound, part, flags) == kernel
    size = (wl.B, wl.Hq, d, bound, part)
    ws = torch.full((adr.adr_decode_workspace_bytes(*size),), 0xFF, dtype=torch.uint8, device="cuda:0")
    words = 64 * (1 + -(-wl.B // 512))
    say("%s d=%d fp8=%s kernel %d part=%d rows=%d" % (entry.__name__, d, fp8, kernel, part, wl.B))
    first = call(entry, b, cache, ws, part, flags)
    torch.cuda.synchronize()
    assert not ws[-4 * words:].any()
    assert adr.adr_decode_read_status(ws, *size) == 0

    kw = dict(k_scale=W.bits(cache.k_scale.cpu()), v_scale=W.bits(cache.v_scale.cpu())) if fp8 else {}
    ref, ref_lse = oracle_attention(b.q, cache.k.cpu(), cache.v.cpu(), b.block_table, b.seq_lens, wl.scale, **kw)
    compare(first["out"], first["lse"], ref, ref_lse, what="first call")
    if part == 0:
        return
    again = call(adr.adr_decode_attention, b, cache, ws, part, flags | adr.PARTIALS_ONLY | adr.WORKSPACE_READY)
    adr.adr_decode_merge(again["out"], again["seq_lens"], bound, part, ws, again["lse"])
    torch.cuda.synchronize()
    compare(again["out"], again["lse"], ref, ref_lse, what="partials and merge")
    if d == 128:
        third = call(adr.adr_decode_attention, b, cache, ws, part, adr.KERNEL_MFMA | adr.WORKSPACE_READY)
        torch.cuda.synchronize()
        compare(third["out"], third["lse"], ref, ref_lse, what="resident kernel")
    assert adr.adr_decode_read_status(ws, *size) == 0
