"""GPU parity of whole rows by item on both sides of the line between eight and four waves: fewer rows of the cache than
compute units, as many, and more."""
import numpy as np
import pytest

from test_gpu_item_kernel import EDGES, check, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,d", [(17, 2, 128), (51, 5, 128), (64, 4, 128), (65, 4, 128), (85, 6, 64), (64, 8, 64)])
@pytest.mark.parametrize("longest", [300, 2100])
@pytest.mark.parametrize("fp8", [False, True])
def test_whole_rows_by_item(B, Hkv, d, longest, fp8):
    lens = np.minimum(np.resize(EDGES + [longest, longest - 1, 255, 256, 257], B), longest)
    check(make(B + longest, 2 * Hkv, Hkv, d, lens), "whole rows %d x %d d=%d up to %d fp8=%s" % (B, Hkv, d, longest, fp8),
          fp8=fp8, partition_tokens=0)


@pytest.mark.parametrize("B,Hkv,d", [(3, 8, 128), (223, 1, 128), (28, 8, 128), (31, 8, 64)])
@pytest.mark.parametrize("longest", [128, 129])
@pytest.mark.parametrize("fp8", [False, True])
def test_short_whole_rows_by_item(B, Hkv, d, longest, fp8):
    """A tile for each of eight waves, and the first of a second round; fewer fp8 rows than leave some compute units to spare."""
    lens = np.minimum(np.resize([longest, 1, 0, 127, 16, 17, longest - 1, 65], B), longest)
    check(make(B + longest, 2 * Hkv, Hkv, d, lens), "short whole rows %d x %d d=%d up to %d fp8=%s" % (B, Hkv, d, longest, fp8),
          fp8=fp8, partition_tokens=0)
