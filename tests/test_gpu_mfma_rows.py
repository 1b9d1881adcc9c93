"""The row-stacked matrix-core kernel of 3x3 binary16 layers: every shape, by request and replayed from what the plan reports, on images smaller than
a tile, widths that end inside a group of eight pixels and inside a tile, channels that fill no chunk, one chunk, several tiles for
each workgroup with a number of chunks that doesn't divide the kernel's unrolling, with and without a fused pool; and a NaN."""
import numpy as np
import pytest

import synth
import paper_2206_10620_amd as pp
from gpu_util import check_layer, run_layer, to_device

pytestmark = pytest.mark.gpu

SHAPES = [(2, 16, 2), (2, 32, 1), (2, 32, 2), (2, 64, 1), (2, 64, 2), (4, 64, 1)]       # rows of a wavefront, columns of a tile, groups of four wavefronts
# n, c_in, c_out, h, w
LAYERS = [(1, 17, 3, 2, 2), (5, 32, 70, 14, 14), (3, 30, 64, 20, 24), (2, 130, 33, 34, 66), (1, 16, 65, 10, 128), (40, 40, 10, 130, 38), (60, 64, 20, 132, 12)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda v: "x".join(map(str, v)))
@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "x".join(map(str, v)))
def test_shapes(layer, shape):
    n, c_in, c_out, h, w = layer
    t, tc, groups = shape
    asked = pp.Tuning(variant=3, mfma_kind=2, tiles_per_wave=t, tile_cols=tc, wg_waves=4 * groups)
    for pool in (False, True):
        print(f"rows {layer} {shape} {pool}", flush=True)
        lay = synth.random_pruned_layer_k("rows", n, c_in, c_out, h, w, "f16", 3, synth.PSET8, 0.5, 0.1, seed=c_in + w, pool=pool)
        if (tc == 16 and w > 16) or ((c_in + 15) // 16) % groups:
            with pytest.raises(pp.PPError):
                pp.plan_from_layer(lay, tuning=asked, host_only=True)
            continue
        rep, y = check_layer(lay, tuning=asked, relu=pool, label=f"rows{layer}{shape}{pool}")
        chosen = rep["chosen"]
        assert (chosen["mfma_kind"], chosen["tiles_per_wave"], chosen["tile_cols"], chosen["tile_rows"], chosen["wg_waves"]) == (2, t, tc, 128 * t // tc, 4 * groups)
        same, again = run_layer(lay, lay.make_input(), tuning=pp.Tuning(**chosen), relu=pool)
        assert again == chosen and np.array_equal(y, same)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda v: "x".join(map(str, v)))
def test_a_nan_without_relu_stays_one(shape):
    # the general kernel, which ran such layers before, stores it too; the product is dense, so it reaches every filter of its window
    t, tc, groups = shape
    lay = synth.random_pruned_layer_k("nan", 2, 32, 70, 14, 14 if tc == 16 else 38, "f16", 3, synth.PSET8, 0.5, 0.1, seed=9)
    x = lay.make_input()
    clean, _ = run_layer(lay, x, tuning=pp.Tuning(variant=3, mfma_kind=2, tiles_per_wave=t, tile_cols=tc, wg_waves=4 * groups), relu=False)
    x[1, 17, 6, 9] = np.nan
    for kind in (dict(mfma_kind=1), dict(mfma_kind=2, tiles_per_wave=t, tile_cols=tc, wg_waves=4 * groups)):
        y, _ = run_layer(lay, x, tuning=pp.Tuning(variant=3, **kind), relu=False)
        nan = np.zeros(y.shape, bool)
        nan[1, :, 5:8, 8:11] = True
        assert np.array_equal(np.isnan(y), nan)
    assert np.array_equal(y[~nan], clean[~nan])


def test_the_tuner_times_every_shape():
    lay = synth.random_pruned_layer("tune", 4, 32, 64, 14, 14, "f16", synth.PSET8, 0.5, 0.3, seed=5)
    x = lay.make_input()
    _, report = pp.autotune(lay, to_device(x), to_device(np.zeros((4, 64, 14, 14), np.float16)), steps=2, rounds=1)
    timed = {(c["tiles_per_wave"], c["tile_cols"], c["wg_waves"] // 4) for _, c, _ in report if c["mfma_kind"] == 2}
    assert set(SHAPES) <= timed
