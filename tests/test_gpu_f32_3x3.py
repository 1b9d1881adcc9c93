"""Binary32 3x3 layers left to the library's choice (the small matrix instruction, or the dense product where the work is
little) against the CPU checker with the binary32 gate of 1e-5 (a sum of K products in any order errs by about sqrt(K) *
2^-24 of its rms: 3e-6 for the 2304 longest one here)."""
import numpy as np
import pytest

import synth
from gpu_util import check_layer

pytestmark = pytest.mark.gpu

# n, c_in, c_out, h, w, keep: widths around the four-pixel pieces and the 64-piece wavefronts (pieces that divide 64 and
# others), batches whose images a wavefront straddles, filter counts around 16 and its quads, channels around the shares of
# 4, 8 and 16 wavefronts; sizes on both sides of the choice between the kernels
LAYERS = [(1, 1, 1, 1, 1, 1.0), (2, 3, 5, 4, 3, 0.6), (64, 16, 33, 7, 7, 0.5), (40, 17, 16, 9, 13, 0.5), (8, 31, 20, 16, 64, 0.5), (4, 40, 50, 33, 62, 0.3),
          (16, 64, 64, 28, 28, 0.5), (2, 256, 144, 30, 57, 0.3), (3, 100, 77, 33, 45, 0.4), (32, 130, 64, 14, 14, 0.5), (1, 20, 16, 300, 261, 0.5), (1, 256, 256, 56, 56, 0.3)]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "x".join(str(i) for i in v[:5]))
def test_layers(layer):
    n, c_in, c_out, h, w, keep = layer
    print(f"f32 3x3 layer {layer}", flush=True)
    lay = synth.random_pruned_layer("quads", n, c_in, c_out, h, w, "f32", synth.PSET16, keep, 0.3, seed=c_in + w)
    for relu in (True, False):
        rep, _ = check_layer(lay, relu=relu, label=f"quads{layer}")
        assert rep["chosen"]["variant"] == 2


@pytest.mark.parametrize("taps", [1, 2, 7, 9])
def test_any_pattern_table(taps):
    pset = synth.random_pattern_set(3, taps, 1 if taps in (1, 9) else 6, seed=taps)
    lay = synth.random_pruned_layer_k("quads", 24, 40, 50, 28, 30, "f32", 3, pset, 0.5, 0.3, seed=4)
    check_layer(lay, label=f"quads-taps{taps}")


def test_no_kernel_kept_and_no_bias():
    import copy
    base = synth.random_pruned_layer("quads", 16, 48, 80, 28, 28, "f32", synth.PSET8, 0.5, 0.3, seed=3)
    lay = copy.copy(base)
    lay.conn_mask = np.zeros_like(base.conn_mask)
    _, y = check_layer(lay, relu=False, label="quads-empty")
    assert np.array_equal(y, np.broadcast_to(base.bias[None, :, None, None], y.shape))
    lay = copy.copy(base)
    lay.bias = None
    check_layer(lay, label="quads-no-bias")
