"""Binary16 block-pruned products of every width on the matrix cores: few columns (the reduction split over wavefronts),
widths that are no multiple of 8 (pieces that straddle rows, the last one of x), many columns; against the CPU checker with
the binary16 gate."""
import pytest

import synth
from test_gpu_block_gemm import check

pytestmark = pytest.mark.gpu


# widths around the pieces of 8, the 32-, 64- and 128-column tiles and the 512-column one
@pytest.mark.parametrize("n", [1, 2, 7, 9, 31, 33, 65, 127, 129, 511, 513, 1030])
@pytest.mark.parametrize("mk", [(1, 1, 1), (65, 17, 16), (130, 700, 16), (64, 2600, 64)], ids=lambda v: "x".join(str(i) for i in v))
def test_widths(mk, n):
    m, k, b = mk                          # lists of one chunk up to more than two segments of 128 entries per wavefront
    check(synth.random_block_layer("w", m, k, n, b, b, "f16", 1.0 if k < 20 else 0.6, 1.0 if k < 20 else 0.6, seed=m + n, relu=bool(n & 2)))


@pytest.mark.parametrize("n", [4099, 8200])
def test_wide_tiles_with_ragged_rows(n):
    check(synth.random_block_layer("wide", 500, 300, n, 64, 64, "f16", 0.6, 0.6, seed=n))


def test_empty_and_uneven_lists():
    check(synth.random_block_layer("empty", 128, 256, 5, 64, 64, "f16", 0.5, 0.0, seed=1))
    check(synth.random_block_layer("uneven", 192, 400, 13, 64, 400, "f16", 0.02, 0.5, seed=2))


def test_the_generic_kernel_takes_more_rows_than_its_lists_have_in_one_grid():
    # 65 536 lists of 32 rows, one more than a grid has rows
    check(synth.random_block_layer("tall", 65535 * 32 + 1, 1, 2, 64, 1, "f16", 0.6, 1.0, seed=3), variant=1)
