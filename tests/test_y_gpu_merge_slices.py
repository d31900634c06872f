"""The merge of a split pass with one, two, four and eight slices per row (the number follows from the
bound on the lengths): partition counts around the edges of slices and rounds, against the fp64 oracle,
and the NaN that a broken hand-shake must leave in every row whatever the number of slices."""
import numpy as np
import pytest
import torch

import paper_2503_20552_amd as adr
import workloads as W
from gpu_util import ATOL, compare, dev, gpu_attention, oracle_attention, say

pytestmark = pytest.mark.gpu


def case(seed, Hq, Hkv, d, lens):
    wl = W.Workload(95, "slices", B=len(lens), Hq=Hq, Hkv=Hkv, d=d, lengths="given")
    return W.make_batch(wl, device="cpu", headroom_tokens=1, seed_offset=seed, lens_before=np.asarray(lens, dtype=np.int32))


def run(b, **kw):
    args = (dev(b.q), dev(b.k_cache), dev(b.v_cache), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    return gpu_attention(*args, partition_tokens=16, flags=kw.pop("flags"), **kw)


# partitions of 16 tokens: the bound gives 11, 12, 24, 48 and 150 places a row, i.e. 1, 2, 4, 8 and 8 slices
@pytest.mark.parametrize("places", [11, 12, 24, 48, 150])
@pytest.mark.parametrize("d,kernel", [(128, adr.KERNEL_MFMA_GRID), (128, adr.KERNEL_MFMA), (64, adr.KERNEL_VALU)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_partition_counts_around_slices_and_rounds(places, d, kernel, out_dtype):
    counts = [c for c in (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 128, 129, 149) if c < places] + [places]
    lens = [16 * c - 1 - (c % 3) for c in counts] + [0]           # (before the append: one token more is attended)
    b = case(places + d, 6, 2, d, lens) if kernel != adr.KERNEL_VALU else case(places, 4, 2, d, lens)
    say("merge of %d places, d=%d kernel=%d" % (places, d, kernel))
    out, lse = run(b, flags=kernel, out_dtype=out_dtype, max_seq_len=16 * places)
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    max_abs, _ = compare(out, lse, ref, ref_lse, what="places %d" % places)
    assert out_dtype == torch.bfloat16 or max_abs <= ATOL
    again, lse_again = run(b, flags=kernel, out_dtype=out_dtype, max_seq_len=16 * places)
    assert torch.equal(out, again) and torch.equal(lse, lse_again)


@pytest.mark.parametrize("places", [11, 24, 64])
def test_expired_waits_reach_every_row(places):
    b = case(places, 8, 2, 128, [16 * places - 1, 3, 40, 16 * (places // 2)])
    say("expired waits, %d places" % places)
    out, lse = run(b, flags=adr.KERNEL_MFMA | adr.DEBUG_EXPIRE_WAITS, max_seq_len=16 * places)
    assert torch.isnan(out).all() and torch.isnan(lse).all()
    clean, _ = run(b, flags=adr.KERNEL_MFMA, max_seq_len=16 * places)
    assert torch.isfinite(clean).all()
