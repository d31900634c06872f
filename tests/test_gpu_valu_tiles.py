"""GPU parity of the vector-ALU kernel around the edges of its turns: one or two tiles a turn of four or eight waves, the 64
tiles of a wave that one load of the page table brings, partitions of one page and of more tiles than a load brings."""
import pytest

import paper_2503_20552_amd as adr
from test_gpu_item_kernel import check, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G,waves", [(64, 1, 8), (64, 2, 4), (128, 1, 4)])
@pytest.mark.parametrize("page_size,fp8", [(16, False), (64, True), (16, True)])
def test_whole_rows(d, G, waves, page_size, fp8):
    turn, load = 16 * waves, 64 * 16 * waves            # tokens of a turn of one tile, of the tiles one load brings
    lens = [0, 1, 16, 17, turn - 1, turn, turn + 1, 2 * turn - 16, 2 * turn, 2 * turn + 1, 3 * turn + 5,
            load - turn, load - 1, load, load + 1, load + turn + 1, 2 * load + 33]
    b = make(d + G, 3 * G, 3, d, lens, page_size)
    check(b, "valu whole rows d=%d G=%d page=%d fp8=%s" % (d, G, page_size, fp8), fp8=fp8, partition_tokens=0,
          flags=adr.KERNEL_VALU)


@pytest.mark.parametrize("page_size,pages", [(16, 1), (16, 3), (16, 17), (16, 513), (64, 1), (64, 3), (64, 129)])
def test_partitions(page_size, pages):
    n = page_size * pages
    b = make(7, 4, 4, 64, [0, 1, n, n + 1, 2 * n + 17, 1000], page_size)
    check(b, "valu partitions of %d page=%d" % (n, page_size), partition_tokens=n, flags=adr.KERNEL_VALU)


@pytest.mark.parametrize("longest", [1, 63, 64, 65])
@pytest.mark.parametrize("page_size,fp8", [(16, False), (64, True), (16, True)])
def test_rows_of_a_tile_a_wave(longest, page_size, fp8):
    """Both sides of the line between four waves and eight, in whole rows and in partitions of 64 tokens."""
    b = make(11 + longest, 6, 6, 64, [min(n, longest) for n in (longest, 0, 1, 15, 16, 17, 33, 48, 49, longest - 1)], page_size)
    check(b, "valu rows of up to %d page=%d fp8=%s" % (longest, page_size, fp8), fp8=fp8, partition_tokens=0, flags=adr.KERNEL_VALU)


@pytest.mark.parametrize("fp8", [False, True])
def test_partitions_of_a_tile_a_wave(fp8):
    b = make(13, 6, 6, 64, [0, 1, 63, 64, 65, 127, 129, 1000])
    check(b, "valu partitions of 64 fp8=%s" % fp8, fp8=fp8, partition_tokens=64, flags=adr.KERNEL_VALU)
