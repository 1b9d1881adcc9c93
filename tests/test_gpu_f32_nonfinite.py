"""Infinities and NaN in the input of binary32 layers: a pruned tap is skipped, so they reach the outputs whose kept taps read
them and no other, on every kernel (what mfma_kind 5 means by itself is mostly the binary32 instruction for layers as small as the first
ones); against the oracle's gather evaluation, which walks the masks' bits."""
import numpy as np
import pytest

import oracle
import synth
import paper_2206_10620_amd as pp
from gpu_util import run_layer

pytestmark = pytest.mark.gpu

# n, c_in, c_out, h, w, ksize, stride, pool, mfma_kind and variant: every epilogue (shares of the reduction or not, pooled or
# not), ragged widths, odd channel counts (the last pair is read twice)
LAYERS = [(2, 9, 21, 8, 12, 3, 1, False, 4, 2), (3, 40, 33, 13, 29, 3, 1, False, 4, 2), (2, 200, 16, 20, 64, 3, 1, False, 4, 2), (2, 9, 21, 8, 12, 3, 1, False, 5, 2),
          (2, 40, 33, 13, 29, 3, 1, False, 0, 2), (1, 1, 5, 6, 7, 1, 1, False, 5, 1), (3, 31, 70, 9, 14, 1, 2, False, 5, 1), (2, 8, 40, 8, 12, 3, 1, True, 5, 1),
          (2, 17, 33, 12, 16, 5, 2, True, 5, 1), (1, 12, 64, 15, 17, 7, 1, False, 5, 1), (40, 64, 128, 16, 16, 1, 1, False, 5, 1)]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "x".join(str(int(i)) for i in v))
def test_layers(layer):
    n, c_in, c_out, h, w, ksize, stride, pool, kind, variant = layer
    pset = synth.PSET8 if ksize == 3 else synth.random_pattern_set(ksize, {1: 1, 5: 6, 7: 9}[ksize], 1 if ksize == 1 else 5, seed=2)
    lay = synth.random_pruned_layer_k("inf", n, c_in, c_out, h, w, "f32", ksize, pset, 1.0 if c_in == 1 else 0.4, 0.3, seed=7, stride=stride, pool=pool)
    x = lay.make_input()
    flat, rs = x.reshape(-1), np.random.RandomState(3)
    at = np.unique(np.concatenate([[0, flat.size - 1], rs.choice(flat.size, size=min(12, flat.size // 4), replace=False)]))
    flat[at] = np.resize([np.inf, np.nan, -np.inf], len(at))
    with np.errstate(all="ignore"):
        pre = oracle.brute_k(x, ksize, stride, lay.taps, lay.pattern_masks, lay.pattern_id, lay.conn_mask, lay.weights, c_out, lay.bias, False)
    assert np.isnan(pre).any() and np.isinf(pre).any() and np.isfinite(pre).any()
    for relu in (False, True):
        ref = np.where(pre > 0, pre, 0.0) if relu else pre                       # a NaN is not above 0
        if pool:
            q = [ref[:, :, i::2, j::2] for i in (0, 1) for j in (0, 1)]
            ref = q[0]
            for v in q[1:]:
                ref = np.where(v > ref, v, ref)
        y, chosen = run_layer(lay, x, tuning=pp.Tuning(variant=variant, mfma_kind=kind), relu=relu)
        assert chosen["mfma_kind"] == kind
        assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isposinf(y), np.isposinf(ref)) and np.array_equal(np.isneginf(y), np.isneginf(ref))
        fin = np.isfinite(ref)
        scale = np.sqrt(np.mean(ref[fin] ** 2)) + 1e-6                           # the binary32 gate: 1e-5 of the value or of the rms
        assert np.all(np.abs(y[fin] - ref[fin]) <= 1e-5 * np.maximum(np.abs(ref[fin]), scale))


# The dense product in bfloat16 parts, where an infinity and what is beyond that type's largest value have to survive the splitting: workgroups
# without reduction shares and with two and four, one, two and four filter tiles, pooled or not.
PARTS = [(5, 64, 33, 58, 28, 1, 1, True), (2, 64, 33, 33, 64, 3, 1, False), (32, 33, 33, 28, 14, 3, 1, True), (16, 17, 33, 28, 28, 5, 1, False), (16, 17, 33, 28, 28, 5, 1, True), (16, 33, 77, 15, 57, 3, 1, False),
         (16, 300, 77, 34, 28, 1, 1, True), (16, 33, 130, 57, 57, 3, 2, False), (32, 256, 77, 14, 58, 1, 1, True)]


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("layer", PARTS, ids=lambda v: "x".join(str(int(i)) for i in v))
def test_layers_in_parts(layer, relu):
    n, c_in, c_out, h, w, ksize, stride, pool = layer
    pset = synth.PSET8 if ksize == 3 else synth.random_pattern_set(ksize, {1: 1, 5: 6}[ksize], 1 if ksize == 1 else 5, seed=2)
    lay = synth.random_pruned_layer_k("inf", n, c_in, c_out, h, w, "f32", ksize, pset, 0.4, 0.3, seed=7, stride=stride, pool=pool)
    lay.weights = np.clip(lay.weights, -0.9, 0.9)                                # the largest value times one weight stays finite
    x = lay.make_input()
    rs = np.random.RandomState(3)
    images = [0, n - 1]                                                          # (the others are compared as they are)
    for img in images:
        flat = x[img].reshape(-1)
        at = np.unique(np.concatenate([[0, flat.size - 1], rs.choice(flat.size, size=12, replace=False)]))
        flat[at] = np.resize(np.array([np.inf, np.nan, -np.inf, np.finfo(np.float32).max, -3.395e38], np.float32), len(at))
    y, chosen = run_layer(lay, x, tuning=pp.Tuning(variant=2 if ksize == 3 and stride == 1 and not pool else 1, mfma_kind=5, staging=3), relu=relu)
    assert chosen["mfma_kind"] == 5 and chosen["staging"] == 3
    with np.errstate(all="ignore"):
        pre = oracle.brute_k(x[images], ksize, stride, lay.taps, lay.pattern_masks, lay.pattern_id, lay.conn_mask, lay.weights, c_out, lay.bias, False)
    assert np.isnan(pre).any() and np.isinf(pre).any() and (np.isfinite(pre) & (np.abs(pre) > 1e36)).any()
    ref = np.where(pre > 0, pre, 0.0) if relu else pre
    if pool:
        q = [ref[:, :, i::2, j::2] for i in (0, 1) for j in (0, 1)]
        ref = q[0]
        for v in q[1:]:
            ref = np.where(v > ref, v, ref)
    got = y[images].astype(np.float64)
    edge = np.isfinite(ref) & (np.abs(ref) > 3.4e38)                             # a sum at the end of the range may round to infinity
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got)[~edge], np.isinf(ref)[~edge])
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    fin = np.isfinite(ref) & ~edge
    small = fin & (np.abs(ref) < 1e30)
    scale = np.sqrt(np.mean(ref[small] ** 2)) + 1e-6
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-5 * np.maximum(np.abs(ref[fin]), scale))
    assert np.all(np.isfinite(np.delete(y, images, axis=0)))
