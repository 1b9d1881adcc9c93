"""Sums beyond the binary16 range without ReLU: every kernel stores the infinity that rounding to nearest gives, so a column's
value does not depend on how many columns or images the call has."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2206_10620_amd as pp
from gpu_util import run_layer

pytestmark = pytest.mark.gpu

MAX, TIE = 65504.0, 65520.0                 # the largest binary16 value; from the tie on, rounding gives infinity


def compare(y, ref):
    y = y.astype(np.float64)
    assert (ref > 1.2 * TIE).any() and (ref < -1.2 * TIE).any() and (np.abs(ref) < 0.8 * MAX).any()
    assert np.all(y[ref > 1.2 * TIE] == np.inf) and np.all(y[ref < -1.2 * TIE] == -np.inf)
    near = np.abs(ref) < 0.8 * MAX          # products of binary16 values in binary32: off by far less than their rounding, 2^-11
    assert np.all(np.abs(y[near] - ref[near]) <= 2e-3 * np.maximum(np.abs(ref[near]), 1e4))


# the split tile and, where there are many columns, the 512-column one; whole pieces and not
@pytest.mark.parametrize("m,k,n", [(128, 256, 8), (128, 256, 13), (64, 64, 131080), (64, 64, 131075)])
def test_block_product(m, k, n):
    lay = synth.random_block_layer("big", m, k, n, 64, 64, "f16", 0.8, 0.8, seed=n, relu=False)
    lay.weights = lay.weights * np.float32(600.0)
    x = (lay.make_input(n).astype(np.float32) * 300.0).astype(np.float16)
    plan = pp.block_plan_from_layer(lay)
    y = plan.run(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.close()
    w = oracle.widen_f16(oracle.round_f16(lay.weights.astype(np.float64)))
    wd = oracle.block_expand(lay.m, lay.k, lay.bm, lay.bk, lay.row_keep, lay.col_keep, w)
    compare(y, wd @ x.astype(np.float64) + (0.0 if lay.bias is None else lay.bias.astype(np.float64)[:, None]))


KERNELS = [(dict(variant=2), False), (dict(variant=3, mfma_kind=1), False), (dict(variant=3, mfma_kind=1), True), (dict(variant=3, mfma_kind=2), False),
           (dict(variant=3, mfma_kind=2), True), (dict(variant=3, mfma_kind=2, split_k=2), False)]


@pytest.mark.parametrize("tuning,pool", KERNELS, ids=lambda t: "-".join(f"{k}{v}" for k, v in t.items()) if isinstance(t, dict) else f"pool{int(t)}")
def test_convolution(tuning, pool):
    lay = synth.random_pruned_layer_k("big", 2, 64, 40, 14, 20, "f16", 3, synth.PSET8, 0.5, 0.3, seed=3, pool=pool)
    lay.weights = lay.weights * np.float32(600.0)
    x = (lay.make_input().astype(np.float32) * 300.0).astype(np.float16)
    y, _ = run_layer(lay, x, tuning=pp.Tuning(**tuning), relu=False)
    ref, _, _ = oracle.layer_reference(lay, x.astype(np.float64), relu=False)
    compare(y, ref)
