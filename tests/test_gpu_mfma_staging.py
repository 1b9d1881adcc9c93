"""The general binary16 matrix-core kernel where its staging and its weight ring can go wrong: images one, two and three
pixels wide, odd widths whose last column is loaded one column early, single-pixel images, one to four chunks of channels
(whole and partial), tiles at both ends of the staging registers, both workgroup shapes.  Tolerance: the binary16 gate of
2e-3, four units in the last place of the stored type."""
import numpy as np
import pytest

import synth
import paper_2206_10620_amd as pp
from gpu_util import check_layer, run_layer

pytestmark = pytest.mark.gpu

# n, c_in, c_out, h, w, ksize, stride, pool
LAYERS = [(1, 1, 1, 1, 1, 1, 1, False), (3, 17, 65, 1, 1, 3, 2, False), (2, 33, 64, 9, 1, 5, 1, False), (70, 16, 20, 2, 1, 3, 2, False),
          (2, 32, 40, 6, 2, 3, 2, False), (5, 31, 70, 3, 3, 7, 1, False), (2, 48, 64, 17, 29, 3, 2, False), (1, 49, 130, 15, 57, 5, 2, False),
          (4, 64, 64, 12, 12, 1, 2, False), (2, 40, 72, 21, 57, 5, 1, False), (2, 3, 64, 30, 31, 7, 2, False), (1, 20, 33, 1, 200, 3, 2, False),
          (3, 18, 64, 12, 20, 5, 1, True), (2, 16, 33, 8, 9, 1, 1, False), (4, 24, 64, 75, 57, 5, 1, False), (1, 65, 64, 5, 7, 3, 2, False)]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "x".join(str(int(i)) for i in v))
def test_layers(layer):
    n, c_in, c_out, h, w, ksize, stride, pool = layer
    print(f"mfma staging {layer}", flush=True)
    pset = synth.random_pattern_set(ksize, {1: 1, 3: 4, 5: 6, 7: 9}[ksize], 1 if ksize == 1 else 5, seed=2)
    lay = synth.random_pruned_layer_k("staging", n, c_in, c_out, h, w, "f16", ksize, pset, 0.6, 0.3, seed=n + c_in, stride=stride, pool=pool)
    for ntw in (0, 1, 2, 4):
        rep, _ = check_layer(lay, tuning=pp.Tuning(variant=3, mfma_kind=1, tiles_per_wave=ntw), relu=bool(ntw & 1), label=f"staging{layer}")
        assert rep["chosen"]["mfma_kind"] == 1 and rep["chosen"]["tiles_per_wave"] in ((ntw,) if ntw else (1, 2))


def test_the_rule_takes_both_shapes():
    def chosen(n, hw):
        pset = synth.random_pattern_set(5, 5, 6, seed=2)
        lay = synth.random_pruned_layer_k("shape", n, 16, 64, hw, hw, "f16", 5, pset, 0.6, 0.3, seed=1)
        rep, _ = check_layer(lay, tuning=pp.Tuning(variant=3, mfma_kind=1), label=f"shape{hw}")
        return rep["chosen"]["tiles_per_wave"]
    assert chosen(1, 20) == 1 and chosen(3, 120) == 2


# n, c_in, c_out, h, w, pool, whether the general kernel runs it: small and odd maps, padded channels, pools; and large whole-chunk layers
AUTO = [(1, 1, 1, 2, 2, False, True), (1, 97, 33, 64, 53, False, True), (4, 40, 20, 7, 7, False, True), (2, 64, 96, 33, 29, False, True), (3, 30, 70, 20, 24, True, True),
        (9, 64, 256, 14, 14, False, True), (2, 20, 64, 113, 111, False, True), (8, 16, 64, 112, 112, True, False), (2, 64, 64, 224, 224, False, False)]


@pytest.mark.parametrize("layer", AUTO, ids=lambda v: "x".join(str(int(i)) for i in v))
def test_the_rule_between_the_matrix_core_kernels(layer):
    n, c_in, c_out, h, w, pool, general = layer
    print(f"mfma auto {layer}", flush=True)
    lay = synth.random_pruned_layer_k("auto", n, c_in, c_out, h, w, "f16", 3, synth.PSET8, 0.5, 0.1, seed=n + c_in, pool=pool)
    rep, _ = check_layer(lay, n_hint=1, label=f"auto{layer}-hint")
    assert rep["chosen"]["mfma_kind"] in (1, 2)
    rep, y = check_layer(lay, label=f"auto{layer}")
    assert rep["chosen"]["mfma_kind"] == (1 if general else 2)
    same, chosen = run_layer(lay, lay.make_input(), tuning=pp.Tuning(**rep["chosen"]))
    assert chosen == rep["chosen"] and np.array_equal(y, same)
    other, _ = run_layer(lay, lay.make_input(), tuning=pp.Tuning(variant=3, mfma_kind=2 if general else 1))
    assert n * c_out * h * w < 100 or not np.array_equal(y, other)      # the other kernel sums in another order: enough outputs round differently
