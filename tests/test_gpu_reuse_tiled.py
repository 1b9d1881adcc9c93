"""Deep reuse on its tiled path (neuron vectors and outputs in multiples of 4) against the CPU checker: signatures and
representatives bit-exact, outputs within the binary32 gate; sizes around the 64- and 128-row tiles, the 512-row rounds, the
2048-row padding, the 64-column blocks; every vector length; segments with more clusters than fit in LDS."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.compare import TOL, error_report
import paper_2206_10620_amd as pp
from test_gpu_reuse import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [4, 8, 12, 16, 20, 24, 28, 32])
@pytest.mark.parametrize("n", [1, 127, 513])
def test_vector_lengths(L, n):
    check(synth.random_reuse_layer("L", n, 5 * L, 12, L, 7, seed=L + n, prototypes=9, noise=0.02))


@pytest.mark.parametrize("m", [4, 60, 64, 68, 132])
@pytest.mark.parametrize("n", [64, 1025, 4100])
def test_output_blocks_and_row_counts(m, n):
    check(synth.random_reuse_layer("m", n, 48, m, 16, 9, seed=m + n, prototypes=20, noise=0.02, relu=bool(n & 1)))


@pytest.mark.parametrize("m", [12, 28, 60])
@pytest.mark.parametrize("n", [2041, 2048, 6144])
def test_workgroups_that_end_behind_the_last_whole_2048_rows(m, n):
    # 680, 292 and 544 rows a workgroup; the table of numbers is as short as the plan makes it, and a longer run came before
    check(synth.random_reuse_layer("end", n, 48, m, 16, 9, seed=m + n, prototypes=20, noise=0.02))


@pytest.mark.parametrize("hash_bits", [1, 6, 12])
def test_many_clusters(hash_bits):
    # unrelated vectors: up to 4096 clusters in a segment, read from memory instead of LDS
    check(synth.random_reuse_layer("c", 6000, 64, 64, 16, hash_bits, seed=3, prototypes=6000, noise=0.0))


def test_runs_of_different_lengths_in_turn():
    lay = synth.random_reuse_layer("t", 5000, 96, 32, 8, 10, seed=6, prototypes=40)
    plan = pp.reuse_plan_from_layer(lay)
    try:
        for n in (5000, 70, 513, 2048, 2049, 5000, 2048):      # each run finds the tables as the one before left them
            x = lay.make_input(n)
            y = plan.run(torch.from_numpy(x).cuda())
            torch.cuda.synchronize()
            sig, rep = plan.clusters(n)
            ref, pre, sc, rsig, rrep = oracle.reuse_layer(x, lay.weights, lay.hyperplanes, lay.seg_len, lay.hash_bits, lay.bias, lay.relu)
            assert np.array_equal(sig, rsig) and np.array_equal(rep, rrep), n
            assert error_report(y.cpu().numpy(), ref, pre, sc)["E"] <= TOL["f32"]
    finally:
        plan.close()


def test_a_pass_that_stopped_behind_its_hash_leaves_nothing_to_the_next():
    """A pass recorded into a graph from which the last two kernels are taken (what a failed launch leaves: the
    representatives elected, nothing after that), then an ordinary pass on other rows."""
    import ctypes as C
    lay = synth.random_reuse_layer("stop", 3000, 96, 32, 8, 10, seed=6, prototypes=40)
    plan = pp.reuse_plan_from_layer(lay)
    hip = pp.lib()                                  # the HIP runtime the library itself is linked to
    try:
        x0, x1 = lay.make_input(3000), np.ascontiguousarray(lay.make_input(3000)[::-1])
        d0, d1 = torch.from_numpy(x0).cuda(), torch.from_numpy(x1).cuda()
        y = torch.empty((3000, 32), device="cuda")
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        graph, execg, count = C.c_void_p(), C.c_void_p(), C.c_size_t()
        s = C.c_void_p(side.cuda_stream)
        assert hip.hipStreamBeginCapture(s, C.c_int(2)) == 0
        st = pp.pp_reuse_run(plan.handle, d0.data_ptr(), y.data_ptr(), 3000, side.cuda_stream)
        assert hip.hipStreamEndCapture(s, C.byref(graph)) == 0 and st == pp.PP_OK
        chain, node, one = [], C.c_void_p(), C.c_size_t(1)
        assert hip.hipGraphGetRootNodes(graph, C.byref(node), C.byref(one)) == 0 and one.value == 1
        while one.value:
            chain.append(C.c_void_p(node.value))
            assert hip.hipGraphNodeGetDependentNodes(chain[-1], None, C.byref(count)) == 0 and count.value <= 1
            one = C.c_size_t(count.value)
            if one.value:
                assert hip.hipGraphNodeGetDependentNodes(chain[-1], C.byref(node), C.byref(one)) == 0
        for last in chain[:-3:-1]:
            assert hip.hipGraphDestroyNode(last) == 0
        assert hip.hipGraphInstantiate(C.byref(execg), graph, None, None, C.c_size_t(0)) == 0
        assert hip.hipGraphLaunch(execg, s) == 0
        torch.cuda.synchronize()
        plan.run(d1, y)
        torch.cuda.synchronize()
        sig, rep = plan.clusters(3000)
        ref, pre, sc, rsig, rrep = oracle.reuse_layer(x1, lay.weights, lay.hyperplanes, lay.seg_len, lay.hash_bits, lay.bias, lay.relu)
        assert np.array_equal(sig, rsig) and np.array_equal(rep, rrep)
        assert error_report(y.cpu().numpy(), ref, pre, sc)["E"] <= TOL["f32"]
        assert hip.hipGraphExecDestroy(execg) == 0 and hip.hipGraphDestroy(graph) == 0
    finally:
        plan.close()
