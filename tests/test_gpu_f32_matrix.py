"""Binary32 layers on the matrix cores (every kernel size, stride and fused pool the tiled kernel has no code for, and
block-pruned products) against the CPU checker.  Tolerance: the binary32 gate of 1e-5; a sum of K products in any order
errs by at most about sqrt(K) * 2^-24 of its rms, 2e-6 for the 1152 terms of the longest one here."""
import numpy as np
import pytest
import torch

import synth
import paper_2206_10620_amd as pp
from gpu_util import check_layer
from test_gpu_block_gemm import check as check_block

pytestmark = pytest.mark.gpu

# n, c_in, c_out, h, w, ksize, stride, pool: channel counts around the groups of eight and the pairs, filters around the
# 32-row tiles, pixels around the 32- and 64-wide tiles, maps so small that a wavefront's pixels span many images
LAYERS = [(1, 1, 1, 1, 1, 1, 1, False), (1, 2, 31, 1, 32, 1, 1, False), (2, 3, 33, 5, 13, 1, 2, False), (70, 7, 32, 1, 1, 3, 2, False),
          (3, 8, 65, 8, 11, 3, 2, False), (40, 9, 5, 2, 2, 3, 1, True), (2, 17, 40, 10, 14, 3, 1, True), (1, 15, 70, 9, 7, 5, 1, False),
          (2, 5, 12, 12, 20, 7, 2, True), (2, 64, 128, 28, 28, 1, 1, False), (4, 128, 64, 29, 31, 3, 2, False), (8, 64, 256, 32, 33, 1, 1, False),
          (16, 24, 100, 40, 40, 5, 2, False)]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "x".join(str(int(i)) for i in v))
def test_conv(layer):
    n, c_in, c_out, h, w, ksize, stride, pool = layer
    print(f"f32 layer {layer}", flush=True)
    pset = synth.random_pattern_set(ksize, {1: 1, 3: 4, 5: 6, 7: 9}[ksize], 1 if ksize == 1 else 5, seed=2)
    lay = synth.random_pruned_layer_k("f32mc", n, c_in, c_out, h, w, "f32", ksize, pset, 0.6, 0.3, seed=n + c_in, stride=stride, pool=pool)
    for relu in (True, False):
        for kind in (5, 6):                  # the dense product and the kernel lists
            rep, _ = check_layer(lay, tuning=pp.Tuning(variant=1, mfma_kind=kind), relu=relu, label=f"f32mc{layer}-{kind}")
            assert rep["chosen"] == pp.Tuning(variant=1, mfma_kind=kind).as_dict()
        check_layer(lay, relu=relu, label=f"f32mc{layer}")


def test_conv_batches_beyond_the_hint():
    lay = synth.random_pruned_layer_k("hint", 9, 12, 40, 6, 7, "f32", 1, np.array([1], dtype=np.uint16), 0.6, 0.3, seed=8)
    check_layer(lay, n_hint=1, label="f32mc-hint")


def test_the_largest_batch_a_call_takes():
    # 2^31 - 2 pixels of one channel: no room behind them in 32 bits for the rest of a tile
    n, h, w = 42966, 151, 331
    plan_args = dict(c_in=1, c_out=1, h=h, w=w, pattern_masks=np.array([1], dtype=np.uint16), pattern_id=np.zeros(1, np.int32), conn_mask=None,
                     weights=np.array([2.0], np.float32), bias=np.array([1.0], np.float32), kernel_size=1, n_hint=n, tuning=pp.Tuning(variant=1, mfma_kind=5))
    st, handle = pp.pp_conv_plan(**plan_args)
    assert st == pp.PP_OK
    x = torch.empty(n * h * w, device="cuda")
    for i in range(0, x.numel(), 1 << 28):
        x[i:i + (1 << 28)] = torch.arange(i % 8191, i % 8191 + min(1 << 28, x.numel() - i), device="cuda").remainder_(8191)
    y = torch.full_like(x, float("nan"))
    assert pp.pp_conv_run(handle, x.data_ptr(), y.data_ptr(), n, torch.cuda.current_stream().cuda_stream) == pp.PP_OK
    for i in range(0, x.numel(), 1 << 28):
        assert torch.equal(y[i:i + (1 << 28)], 2 * x[i:i + (1 << 28)] + 1)
    pp.pp_conv_destroy(handle)


# m, k, n, block, row keep, column keep
PRODUCTS = [(1, 1, 1, 1, 1.0, 1.0), (31, 7, 31, 8, 1.0, 1.0), (32, 8, 32, 16, 1.0, 1.0), (33, 9, 33, 16, 0.6, 0.6), (100, 200, 65, 16, 0.5, 0.5),
            (64, 64, 40, 32, 0.0, 0.5), (200, 1000, 1, 64, 0.5, 0.5), (300, 520, 197, 50, 0.5, 0.5), (1000, 600, 700, 16, 0.5, 0.5)]


@pytest.mark.parametrize("product", PRODUCTS, ids=lambda v: "x".join(str(i) for i in v[:4]))
def test_block_product(product):
    m, k, n, b, rk, ck = product
    lay = synth.random_block_layer("f32mc", m, k, n, b, b, "f32", rk, ck, seed=m + n, relu=bool(n & 1))
    check_block(lay)


@pytest.mark.parametrize("dtype,variant", [("f32", 0), ("f16", 1)])
@pytest.mark.parametrize("k", [1, 8, 9, 15])
def test_block_product_with_an_infinite_last_column(k, dtype, variant):
    # the list's padding is no column: an infinity in its last one meets each row's own weight there and nothing else
    lay = synth.random_block_layer("inf", 64, k, 37, 16, 16, dtype, 1.0, 1.0, seed=k, relu=False)
    x = lay.make_input()
    x[k - 1, 5] = np.inf
    plan = pp.block_plan_from_layer(lay, variant=variant)
    y = plan.run(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
    plan.close()
    assert np.all(y[:, 5] == np.sign(lay.weights[:, k - 1]) * np.inf)
    assert np.all(np.isfinite(np.delete(y, 5, axis=1)))
