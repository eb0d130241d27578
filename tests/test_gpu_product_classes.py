"""The masked product on every kind of unit class, against the FP64 oracle.

The kernel of a unit is chosen by the blocks of 16 rows on its two sides and by the
functions of its clusters, so the leaf sizes below give leaf groups of 2 to 8 blocks: 17
to 32 functions per leaf (of a degree-1 basis, leaf points - m), with all sizes even or
with odd ones, one or several leaves in the last group.  Tolerances as in the other
product tests: 1e-12 for FP64 (a sum of at most N terms), 1e-8 and 1e-6 for the FP32 forms.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import ops, pattern

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2211_11681_amd import spm
    spm._lib.load()
    assert torch.cuda.is_available()
    return spm


def to_dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# (cloud, N, leaf, eta, block counts of the leaf groups)
CASES = [("cube2", 20 * 32, 20, 1.2, {5}),        # 17 functions: odd
         ("cube3", 24 * 32, 24, 1.0, {5}),        # 20: four leaves are 80 rows
         ("cube3", 28 * 64, 28, 1.0, {6}),        # 24: one wave per leaf, six blocks
         ("cube3", 32 * 16, 32, 1.0, {7}),        # 28
         ("cube3", 36 * 32, 36, 1.0, {8}),        # 32: the largest cluster
         ("cube3", 1500, 32, 1.0, {5}),           # 23 and 24 points: odd sizes
         ("sphere", 1000, 32, 1.0, {7}),          # 31 and 32 points: 27 and 28 functions
         ("cube3", 60, 32, 5.0, {4}),             # two leaves, one group, full pattern
         ("cube3", 54, 28, 5.0, {3}),             # two leaves of 23
         ("cube2", 39, 20, 5.0, {2})]             # a leaf of 17 beside one of 16


@pytest.mark.parametrize("kind,n,leaf,eta,blocks", CASES)
def test_product_of_every_class(S, kind, n, leaf, eta, blocks):
    t = S.Tree(synth.workload_points(kind, n, 6), leaf, 1)
    pat = S.Pattern.from_tree(t, eta)
    sides = {c["row_blocks"] for c in pat.classes()}
    print(f"case: classes {kind} n={n} leaf={leaf} eta={eta} sides={sorted(sides)}", flush=True)
    assert blocks <= sides
    mask = pattern.dense_mask(*pat.download_csr(), n)
    i, j = np.nonzero(mask)
    a, b = np.zeros((n, n)), np.zeros((n, n))
    a[i, j] = 2 * synth.pair_uniform(41, i, j, n) - 1
    b[i, j] = 2 * synth.pair_uniform(42, i, j, n) - 1
    A, B = pat.values_from_csr(to_dev(a[mask])), pat.values_from_csr(to_dev(b[mask]))
    for ta, tb in [(0, 0), (1, 1)]:
        ref = ops.masked_product(a.T if ta else a, b.T if tb else b, mask)[mask]
        for prec, tol in (("f64", 1e-12), ("f32split", 1e-8), ("f32acc", 1e-6)):
            X, Y = (S.convert(pat, v, "f64", prec) for v in (A, B))
            C = S.convert(pat, S.masked_gemm(pat, X, Y, transA=bool(ta), transB=bool(tb), prec=prec), prec, "f64")
            err = np.linalg.norm(pat.values_to_csr(C).cpu().numpy() - ref) / np.linalg.norm(ref)
            assert err <= tol, (prec, ta, tb, err)


def test_result_rows_depend_on_their_own_rows_only(S):
    # rows past a cluster's end are filled with its last row, and absent tiles with zeros:
    # an infinity in one row of A may reach the results of that row alone
    n = 28 * 32
    t = S.Tree(synth.workload_points("cube3", n, 6), 28, 1)
    pat = S.Pattern.from_tree(t, 1.0)
    mask = pattern.dense_mask(*pat.download_csr(), n)
    i, j = np.nonzero(mask)
    a, b = np.zeros((n, n)), np.zeros((n, n))
    a[i, j] = 2 * synth.pair_uniform(43, i, j, n) - 1
    b[i, j] = 2 * synth.pair_uniform(44, i, j, n) - 1
    rows = [3, n // 2, n - 1]
    bad = a.copy()
    bad[rows] = np.where(mask[rows], np.inf, 0.0)
    B = pat.values_from_csr(to_dev(b[mask]))
    good = pat.values_to_csr(S.masked_gemm(pat, pat.values_from_csr(to_dev(a[mask])), B)).cpu().numpy()
    got = pat.values_to_csr(S.masked_gemm(pat, pat.values_from_csr(to_dev(bad[mask])), B)).cpu().numpy()
    own = np.isin(i, rows)
    assert np.array_equal(got[~own], good[~own])
    assert not np.isfinite(got[own]).all()
