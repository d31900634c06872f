"""Weights are handed to the matrix instructions as sums of bf16 terms; the terms must not make up weight
that is not there.  Values up to the largest bf16 number under weights that underflow to zero, and values
of about 2^g under weights of 2^-g, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2503_20552_amd as adr
from gpu_util import ATOL, compare, dev, gpu_attention, oracle_attention, say
from test_gpu_item_kernel import make

pytestmark = pytest.mark.gpu


def batch(d, gaps, top_v, v_of_gap):
    """Token 16 i has score 0 for every head, the others -g (base 2) for g of `gaps` in turn.  (One in every
    tile, so that no wave's own maximum is the low score: its sums would leave the range of fp32.)"""
    b = make(3, 8, 2, d, [1, 40, 700, 1300])
    q = torch.zeros_like(b.q)
    q[:, :, 0] = 1
    n = b.k_cache.shape[0] * 16
    g = torch.tensor(gaps)[torch.arange(n) % len(gaps)].reshape(-1, 16)
    g[:, 0] = 0
    k = torch.zeros_like(b.k_cache)
    k[..., 0] = (-g / (b.wl.scale * np.log2(np.e))).to(torch.bfloat16)[:, :, None]
    v = b.v_cache.double() * v_of_gap(g.double())[:, :, None, None]
    v[:, 0] = b.v_cache[:, 0].double() * top_v
    b.q, b.k_cache, b.v_cache = q, k, v.clamp(-3.3e38, 3.3e38).to(torch.bfloat16)
    return b


@pytest.mark.parametrize("d,kernel", [(64, adr.KERNEL_AUTO), (128, adr.KERNEL_MFMA_GRID), (128, adr.KERNEL_MFMA)])
@pytest.mark.parametrize("partition_tokens", [0, 64])
@pytest.mark.parametrize("what,gaps,v_of_gap", [
    ("weights that are zero", [160, 300, 1000], lambda g: torch.full_like(g, 3e38)),
    # 2^-122 of a weight has 4 bits above the smallest normal number; the second term may then be lost (2^-8)
    ("tiny weights", [20, 60, 90, 101, 113, 122], lambda g: 2.0 ** g)])
def test_terms_add_up_to_the_weight(d, kernel, partition_tokens, what, gaps, v_of_gap):
    b = batch(d, gaps, 1.0, v_of_gap)
    args = (dev(b.q), dev(b.k_cache), dev(b.v_cache), dev(b.block_table), dev(b.seq_lens), b.wl.scale)
    say("%s d=%d kernel=%d part=%d" % (what, d, kernel, partition_tokens))
    out, lse = gpu_attention(*args, partition_tokens=partition_tokens, flags=kernel)
    ref, ref_lse = oracle_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.wl.scale)
    worst, _ = compare(out, lse, ref, ref_lse, what=what)
    assert what != "weights that are zero" or worst <= ATOL
