"""The dense binary32 convolution in bfloat16 parts and on the binary32 instruction: every workgroup shape, in parts with each remainder of
its loop over four reduction units and shares shorter than that loop, partial filter and pixel tiles, 1x1 to 5x5, stride 1 and 2, a fused
pool; inputs of every size, and sums of one product, against the oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2206_10620_amd as pp
from gpu_util import check_layer, run_layer

pytestmark = pytest.mark.gpu

# n, c_in, c_out, h, w, ksize, stride, pool; in parts the workgroup (filter tiles, pixel tiles, reduction shares) and the reduction units of a
# share; on the binary32 instruction the workgroup (filter tiles, pixel tiles, shares, wavefronts on different pixels).  test_host_rules.py holds the
# rules to these.
LAYERS = [((1, 3, 3, 7, 7, 1, 2, False), (1, 4, 1), 1, (1, 1, 4, 1)), ((1, 64, 3, 5, 7, 1, 2, False), (2, 1, 4), 1, (1, 1, 4, 1)), ((1, 77, 3, 7, 5, 3, 2, False), (2, 1, 4), 12, (1, 1, 4, 1)),
          ((1, 17, 3, 5, 7, 5, 2, False), (2, 1, 4), 13, (1, 1, 4, 1)), ((4, 33, 3, 64, 33, 1, 1, False), (1, 4, 1), 3, (1, 2, 4, 1)),
          ((32, 3, 3, 9, 57, 1, 1, False), (1, 4, 1), 1, (1, 2, 1, 4)), ((32, 17, 3, 57, 9, 1, 1, False), (1, 4, 1), 2, (1, 2, 4, 1)), ((32, 33, 3, 9, 57, 1, 1, False), (1, 4, 1), 3, (1, 2, 4, 1)),
          ((16, 64, 3, 57, 28, 1, 1, False), (1, 4, 1), 4, (1, 2, 4, 1)), ((16, 64, 3, 58, 28, 1, 1, True), (1, 4, 1), 4, (1, 2, 4, 1)),
          ((2, 64, 33, 33, 64, 3, 1, False), (2, 1, 4), 9, (1, 2, 4, 1)), ((2, 64, 33, 34, 64, 3, 1, True), (2, 1, 4), 9, (1, 2, 4, 1)), ((32, 48, 33, 15, 33, 3, 2, False), (2, 1, 4), 7, (1, 2, 4, 1)),
          ((8, 77, 33, 9, 57, 3, 1, False), (2, 1, 4), 12, (1, 2, 4, 1)),
          ((1, 17, 300, 57, 57, 1, 1, False), (2, 2, 2), 1, (2, 2, 4, 1)), ((32, 200, 33, 57, 7, 1, 1, False), (2, 2, 2), 7, (2, 2, 4, 1)), ((32, 33, 33, 28, 14, 3, 1, False), (2, 2, 2), 14, (2, 2, 4, 1)),
          ((32, 33, 33, 28, 14, 3, 1, True), (2, 2, 2), 14, (2, 2, 4, 1)),
          ((16, 17, 33, 28, 28, 5, 1, False), (2, 2, 4), 13, (2, 2, 4, 1)), ((16, 33, 33, 28, 28, 5, 1, False), (2, 2, 4), 19, (2, 2, 4, 1)), ((16, 17, 33, 28, 28, 5, 1, True), (2, 2, 4), 13, (2, 2, 4, 1)),
          ((8, 3, 33, 64, 57, 1, 1, False), (2, 4, 1), 1, (1, 2, 1, 4)), ((32, 100, 33, 14, 57, 1, 1, False), (2, 4, 1), 7, (1, 2, 1, 4)), ((32, 100, 33, 14, 58, 1, 1, True), (2, 4, 1), 7, (1, 2, 1, 4)),
          ((16, 33, 77, 15, 57, 3, 1, False), (4, 2, 4), 7, (1, 2, 1, 4)), ((16, 300, 77, 33, 28, 1, 1, False), (4, 2, 4), 5, (2, 2, 2, 2)), ((16, 300, 77, 34, 28, 1, 1, True), (4, 2, 4), 5, (2, 2, 2, 2)),
          ((32, 17, 200, 57, 33, 1, 2, False), (4, 4, 1), 2, (2, 2, 1, 4)), ((16, 3, 77, 28, 57, 3, 1, False), (4, 4, 1), 9, (2, 2, 1, 4)), ((16, 3, 77, 28, 58, 3, 1, True), (4, 4, 1), 9, (2, 2, 1, 4)),
          ((32, 256, 77, 14, 57, 1, 1, False), (4, 4, 2), 8, (1, 2, 4, 1)), ((16, 33, 130, 57, 57, 3, 2, False), (4, 4, 2), 14, (2, 2, 4, 1)), ((32, 256, 77, 14, 58, 1, 1, True), (4, 4, 2), 8, (1, 2, 4, 1))]


def dense(layer, staging):
    """The tuning that asks for a kernel of the dense product by name: 1 the binary32 instruction, 3 parts."""
    return pp.Tuning(variant=2 if layer[5] == 3 and layer[6] == 1 and not layer[7] else 1, mfma_kind=5, staging=staging)


@pytest.mark.parametrize("staging", [1, 3])
@pytest.mark.parametrize("layer", [row[0] for row in LAYERS], ids=lambda v: "x".join(str(int(i)) for i in v))
def test_shapes_and_remainders(layer, staging):
    n, c_in, c_out, h, w, ks, stride, pool = layer
    print(f"split layer {layer} {staging}", flush=True)
    lay = synth.random_pruned_layer_k("split", n, c_in, c_out, h, w, "f32", ks, synth.random_pattern_set(ks, 1 if ks == 1 else 4, 1 if ks == 1 else 6, seed=2), 0.8, 0.3,
                                      seed=c_in + w, stride=stride, pool=pool)
    # A sum is rounded once per 16 products, in binary32, in each of two accumulators and once per share (on the binary32 instruction once per two
    # products): a walk of `units` steps of 2^-24 of the sum, of which four deviations cover 10^5 outputs, and the operands' three parts leave
    # nothing out above 2^-24.
    units = ks * ks * ((c_in + 15) // 16)
    tol = 4 * 2.0 ** -24 * (2 * math.sqrt(units if staging == 3 else 8 * units) + 2)
    rep, _ = check_layer(lay, tuning=dense(layer, staging), tol=tol, label=f"split{layer}")
    assert rep["chosen"] == dense(layer, staging).as_dict()


@pytest.mark.parametrize("layer", [(2, 64, 33, 33, 64, 3, 1), (32, 256, 77, 14, 57, 1, 1)], ids=lambda v: "x".join(map(str, v)))
@pytest.mark.parametrize("scale", [0, 100, -100, -112, -126, -140, -145])
@pytest.mark.parametrize("staging", [1, 3])
def test_inputs_of_every_size(layer, staging, scale):
    # 64 bits say what a sum is; each of its K roundings in binary32 is 2^-24 of it or half the smallest subnormal
    n, c_in, c_out, h, w, ks, stride = layer
    lay = synth.random_pruned_layer_k("size", n, c_in, c_out, h, w, "f32", ks, synth.PSET8 if ks == 3 else np.array([1], np.uint16), 0.8, 0.3, seed=3, stride=stride)
    lay.bias = None
    x = np.ldexp(lay.make_input().astype(np.float64), scale).astype(np.float32)
    y, chosen = run_layer(lay, x, tuning=pp.Tuning(variant=2 if ks == 3 else 1, mfma_kind=5, staging=staging), relu=False)
    pts = np.stack([np.random.RandomState(1).randint(m, size=4096) for m in y.shape], axis=1).astype(np.int32)
    conv_at = oracle.conv_at if ks == 3 else lambda x, w, p, b, r: oracle.conv_k_at(x, w, p, stride, b, r)
    ref, _, sc = conv_at(x, oracle.layer_dense_weights(lay), pts, None, False)
    err = np.abs(y[tuple(pts.T)].astype(np.float64) - ref)
    assert chosen["mfma_kind"] == 5 and np.all(err <= 4 * math.sqrt(ks * ks * c_in) * (2.0 ** -24 * sc + 2.0 ** -150))

def test_a_sum_of_one_product_is_rounded_once():
    # (such a layer is not split, and large enough that no two wavefronts share its reduction)
    lay = synth.random_pruned_layer_k("one", 8, 1, 64, 224, 224, "f32", 1, np.array([1], np.uint16), 1.0, 0.3, seed=3)
    x = lay.make_input()
    y, chosen = run_layer(lay, x, relu=False)
    ref = lay.weights.reshape(-1).astype(np.float64)[None, :, None, None] * x.astype(np.float64) + lay.bias.astype(np.float64)[None, :, None, None]
    assert chosen["mfma_kind"] == 5 and np.all(np.abs(y - ref) <= 2.0 ** -24 * (1 + 1e-6) * np.abs(ref))


@pytest.mark.parametrize("staging", [0, 3])
def test_a_batch_just_below_two_to_the_31_pixels(staging):
    # 128 pixels to 256 lanes: a single launch would be of 2^32 lanes
    n, h, w = 7613, 51, 5531
    st, handle = pp.pp_conv_plan(c_in=1, c_out=1, h=h, w=w, pattern_masks=np.array([1], np.uint16), pattern_id=np.zeros(1, np.int32), conn_mask=None, weights=np.array([2.0], np.float32),
                                 bias=np.array([1.0], np.float32), kernel_size=1, n_hint=n, tuning=pp.Tuning(variant=1, mfma_kind=5, staging=staging))
    assert st == pp.PP_OK
    x = torch.full((n * h * w,), 3.0, device="cuda")
    y = torch.full_like(x, float("nan"))
    assert pp.pp_conv_run(handle, x.data_ptr(), y.data_ptr(), n, torch.cuda.current_stream().cuda_stream) == pp.PP_OK
    for i in range(0, x.numel(), 1 << 28):
        assert bool((y[i:i + (1 << 28)] == 7.0).all())
    pp.pp_conv_destroy(handle)
