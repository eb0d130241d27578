"""The samplet transform at the edges of what it takes: infinities, a tree's first call,
capture of a transform after another call on the tree.
"""
import time

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2211_11681_amd import spm
    spm._lib.load()
    assert torch.cuda.is_available()
    return spm


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("leaf", [16, 17, 18, 19, 33])
def test_transform_of_an_infinity(S, leaf, inverse):
    # an infinity in a leaf's last input gives infinities of the unit vector's signs there,
    # not the NaN of an infinity times a padding zero
    t = S.Tree(synth.workload_points("cube2", 16 * leaf, 5), leaf, 1)
    arr = t.arrays()
    leaf_c = np.nonzero(arr["level"] == t.depth)[0][5]
    assert arr["pt_size"][leaf_c] == leaf
    pts = arr["perm"][arr["pt_start"][leaf_c]:arr["pt_start"][leaf_c] + leaf]
    fun = np.arange(arr["cluster_start"][leaf_c], arr["cluster_start"][leaf_c + 1])
    src, dst = (fun, pts) if inverse else (pts, fun)
    x = torch.zeros(3, t.n, dtype=torch.float64, device="cuda")
    x[0, src[-1]], x[1, src[-1]] = 1.0, float("inf")
    y = S.fst(t, x, inverse=inverse).cpu().numpy()
    unit = y[0, dst]
    live = np.abs(unit) > 1e-10
    assert live.sum() >= len(dst) // 2
    assert np.array_equal(y[1, dst][live], np.where(unit[live] > 0, np.inf, -np.inf))
    assert not y[2].any()


def test_first_transform_of_a_tree(S):
    # the tables of 60000 points: 1 ms for their copies; 15 ms with the matrices laid out on the host
    n = 60000
    pts = synth.workload_points("sphere", n, 3)
    x = torch.ones(4, n, dtype=torch.float64, device="cuda")
    took = []
    for _ in range(4):
        t = S.Tree(pts, 32, 1)
        torch.cuda.synchronize()
        start = time.perf_counter()
        S.fst(t, x)
        torch.cuda.synchronize()
        took.append(time.perf_counter() - start)
    assert min(took) < 5e-3, took


def test_inverse_is_capturable_after_a_forward_transform(S):
    # the first call on a tree uploads its tables; every later one is launches alone
    n, r = 5000, 3
    t = S.Tree(synth.workload_points("cube2", n, 12), 32, 2)
    x = torch.from_numpy(2 * synth.uniform(53, np.arange(r * n)).reshape(r, n) - 1).cuda()
    y = S.fst(t, x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        back = S.fst(t, y, inverse=True)
    for k in range(4):
        y.copy_(S.fst(t, (k + 1) * x))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(back, S.fst(t, y, inverse=True))
        assert (back - (k + 1) * x).abs().max().item() <= 1e-11


def test_forward_is_capturable_after_a_construction(S):
    n, r = 2000, 3
    t = S.Tree(synth.workload_points("cube2", n, 12), 32, 1)
    pat = S.Pattern.from_tree(t, 1.0)
    S.kernel_compress(pat, t, 1, 0.3, 1.0 / n)
    x = torch.from_numpy(2 * synth.uniform(53, np.arange(r * n)).reshape(r, n) - 1).cuda()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = S.fst(t, x)
    for k in range(4):
        x.mul_(1.5)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, S.fst(t, x))
        assert (S.fst(t, y, inverse=True) - x).abs().max().item() <= 1e-11
