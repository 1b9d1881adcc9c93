"""Binary32 3x3 layers on the kernel of the small matrix instruction (mfma_kind 4) and as dense products (5), each by name and
left to the library's choice, against the oracle with the binary32 gate of 1e-5 (a sum of K products in any order errs by about sqrt(K) *
2^-24 of its rms: 3e-6 for the 2304 longest one here)."""
import numpy as np
import pytest

import synth
import paper_2206_10620_amd as pp
from gpu_util import check_layer, run_layer, to_device

pytestmark = pytest.mark.gpu

# n, c_in, c_out, h, w, keep: widths around the four-pixel pieces and the 64-piece wavefronts (pieces that divide 64 and
# others), batches whose images a wavefront straddles, filter counts around 16 and its quads, channels around the shares of
# 4, 8 and 16 wavefronts; which kernel the library takes
LAYERS = [(1, 1, 1, 1, 1, 1.0, 5), (2, 3, 5, 4, 3, 0.6, 5), (64, 16, 33, 7, 7, 0.5, 5), (40, 17, 16, 9, 13, 0.5, 5), (8, 31, 20, 16, 64, 0.5, 5), (4, 40, 50, 33, 62, 0.3, 5),
          (16, 64, 64, 28, 28, 0.4, 4), (2, 256, 144, 30, 57, 0.3, 4), (3, 100, 77, 33, 45, 0.4, 5), (32, 130, 64, 14, 14, 0.5, 5), (1, 20, 16, 300, 261, 0.5, 4),
          (1, 256, 256, 56, 56, 0.3, 4)]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "x".join(str(i) for i in v[:5]))
def test_layers(layer):
    n, c_in, c_out, h, w, keep, kind = layer
    print(f"f32 3x3 layer {layer}", flush=True)
    lay = synth.random_pruned_layer("quads", n, c_in, c_out, h, w, "f32", synth.PSET16, keep, 0.3, seed=c_in + w)
    for relu in (True, False):
        y = {}
        for asked in (4, 5):
            rep, y[asked] = check_layer(lay, tuning=pp.Tuning(variant=2, mfma_kind=asked), relu=relu, label=f"quads{layer}-{asked}")
            assert rep["chosen"] == pp.Tuning(variant=2, mfma_kind=asked).as_dict()
        rep, auto = check_layer(lay, relu=relu, label=f"quads{layer}")
        assert rep["chosen"] == pp.Tuning(variant=2, mfma_kind=kind).as_dict() and np.array_equal(auto, y[kind])


@pytest.mark.parametrize("w", [4, 12, 13, 16, 64, 67])
@pytest.mark.parametrize("n,c_in,c_out,h,keep", [(1, 3, 16, 5, 0.5), (3, 9, 70, 7, 0.5), (40, 33, 64, 20, 0.5), (3, 200, 64, 40, 0.5), (1, 250, 40, 9, 0.2)])
def test_every_instantiation(n, c_in, c_out, h, keep, w):
    # pieces that divide 64 and others, whole pieces and not, with 4, 8 and 16 wavefronts on a tile's channels
    lay = synth.random_pruned_layer("quads", n, c_in, c_out, h, w, "f32", synth.PSET16, keep, 0.3, seed=c_in + w)
    check_layer(lay, tuning=pp.Tuning(variant=2, mfma_kind=4), label=f"quads{(n, c_in, c_out, h, w)}")


@pytest.mark.parametrize("kind", [0, 4, 5])
@pytest.mark.parametrize("taps", [1, 2, 7, 9])
def test_any_pattern_table(taps, kind):
    pset = synth.random_pattern_set(3, taps, 1 if taps in (1, 9) else 6, seed=taps)
    lay = synth.random_pruned_layer_k("quads", 24, 40, 50, 28, 30, "f32", 3, pset, 0.5, 0.3, seed=4)
    check_layer(lay, tuning=pp.Tuning(variant=2, mfma_kind=kind) if kind else None, label=f"quads-taps{taps}")


@pytest.mark.parametrize("kind", [4, 5])
def test_no_kernel_kept_and_no_bias(kind):
    import copy
    base = synth.random_pruned_layer("quads", 16, 48, 80, 28, 28, "f32", synth.PSET8, 0.5, 0.3, seed=3)
    lay = copy.copy(base)
    lay.conn_mask = np.zeros_like(base.conn_mask)
    tuning = pp.Tuning(variant=2, mfma_kind=kind)
    _, y = check_layer(lay, tuning=tuning, relu=False, label="quads-empty")
    assert np.array_equal(y, np.broadcast_to(base.bias[None, :, None, None], y.shape))
    lay = copy.copy(base)
    lay.bias = None
    check_layer(lay, tuning=tuning, label="quads-no-bias")


@pytest.mark.parametrize("dtype,shape", [("f32", (2, 24, 32, 28, 28)), ("f32", (16, 64, 64, 28, 28)), ("f16", (1, 97, 33, 64, 53)), ("f16", (4, 16, 64, 112, 112))])
def test_tuners_time_every_kernel_and_what_they_report_runs_again(dtype, shape):
    lay = synth.random_pruned_layer("tune", *shape, dtype, synth.PSET8, 0.5, 0.3, seed=5)
    x = lay.make_input()
    _, report = pp.autotune(lay, to_device(x), to_device(np.zeros((shape[0], shape[2], *shape[3:]), dtype=x.dtype)), steps=2, rounds=1)
    kinds = {(c["variant"], c["mfma_kind"]) for _, c, _ in report}
    assert kinds == ({(1, 6), (2, 0), (2, 4), (2, 5)} if dtype == "f32" else {(2, 0), (3, 1), (3, 2)})
    for tuning in [pp.Tuning(autotune=1)] + [pp.Tuning(**c) for _, c, _ in report]:
        y, chosen = run_layer(lay, x, tuning=tuning)
        chosen["autotune"] = 0
        again, same = run_layer(lay, x, tuning=pp.Tuning(**chosen))
        assert same == chosen and np.array_equal(again, y), chosen


@pytest.mark.parametrize("n,c_in,c_out,h,w,keep", [(32, 64, 64, 56, 56, 0.1), (19, 77, 500, 43, 32, 0.008), (4, 64, 64, 224, 224, 0.2)])
def test_large_layers_with_few_kernels_left_run_on_the_vector_kernel(n, c_in, c_out, h, w, keep):
    lay = synth.random_pruned_layer("few", n, c_in, c_out, h, w, "f32", synth.PSET16, keep, 0.3, seed=3)
    rep, y = check_layer(lay, label=f"few{(n, c_in, c_out, h, w)}")
    assert rep["chosen"]["variant"] == 2 and rep["chosen"]["mfma_kind"] == 0 and rep["chosen"]["filters_per_wave"] > 0
    again, chosen = run_layer(lay, lay.make_input(), tuning=pp.Tuning(**rep["chosen"]))
    assert chosen == rep["chosen"] and np.array_equal(again, y)
