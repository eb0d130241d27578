"""The staged samplet transform and the construction of K^eta where their stages can go wrong:
one to three stages, clusters with more than 32 inputs, leaves smaller than the number of
moments (their functions are all handed up, so a cluster's inputs are not two runs), sizes
of a block's edge, ragged clusters, single and many vectors.  Against the oracle: the
transform to 1e-13 of the vector norm (log N orthogonal steps of at most 64 terms each),
the compressed matrix to 1e-12 relative Frobenius as in the other construction tests.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import compress, ops, pattern, samplets, tree

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2211_11681_amd import spm
    spm._lib.load()
    assert torch.cuda.is_available()
    return spm


# (cloud, N, leaf, q, vectors)
CASES = [("cube2", 12, 16, 1, 1),        # one leaf
         ("cube3", 64, 32, 1, 3),        # exactly one block
         ("cube2", 65, 32, 1, 17),       # two stages, blocks of 32 and 33 points
         ("cube3", 1344, 42, 2, 16),     # 42 inputs per leaf
         ("cube2", 47 * 16, 47, 4, 5),   # 47 inputs, 15 moments
         ("cube3", 700, 6, 2, 2),        # leaves below the 10 moments
         ("sphere", 3001, 32, 1, 10),    # ragged
         ("cube2", 20000, 32, 2, 33)]    # three stages, three groups of vectors


@pytest.mark.parametrize("kind,n,leaf,q,r", CASES)
def test_transform_stages_vs_oracle(S, kind, n, leaf, q, r):
    print(f"case: transform {kind} n={n} leaf={leaf} q={q} r={r}", flush=True)
    pts = synth.workload_points(kind, n, 12)
    basis = samplets.build_samplets(tree.build_tree(pts, leaf), q)
    x = 2 * synth.uniform(51, np.arange(r * n)).reshape(r, n) - 1
    t = S.Tree(pts, leaf, q)
    X = torch.from_numpy(x).cuda()
    ref = ops.fst(basis, x.T).T
    for _ in range(2):                            # the second call finds the tables in place
        Y = S.fst(t, X)
        err = np.linalg.norm(Y.cpu().numpy() - ref, axis=1) / np.linalg.norm(x, axis=1)
        assert err.max() <= 1e-13, err.max()
    back = S.fst(t, torch.from_numpy(np.ascontiguousarray(ref)).cuda(), inverse=True).cpu().numpy()
    err = np.linalg.norm(back - x, axis=1) / np.linalg.norm(x, axis=1)
    assert err.max() <= 1e-13, err.max()


def test_transform_keeps_vectors_and_clusters_apart(S):
    # a NaN in one vector stays in it, and there in the functions over that point
    n, leaf, q = 300, 20, 1
    pts = synth.workload_points("cube3", n, 13)
    basis = samplets.build_samplets(tree.build_tree(pts, leaf), q)
    t = S.Tree(pts, leaf, q)
    x = 2 * synth.uniform(52, np.arange(4 * n)).reshape(4, n) - 1
    good = S.fst(t, torch.from_numpy(x).cuda()).cpu().numpy()
    bad = x.copy()
    bad[2, 17] = np.nan
    got = S.fst(t, torch.from_numpy(bad).cuda()).cpu().numpy()
    touched = np.zeros((4, n), bool)
    pos = int(np.nonzero(basis.tree.perm == 17)[0][0])
    for c in range(basis.tree.n_clusters):
        if basis.tree.start[c] <= pos < basis.tree.start[c] + basis.tree.size[c]:
            touched[2, basis.cluster_start[c]:basis.cluster_start[c + 1]] = True
    assert np.array_equal(got[~touched], good[~touched])
    assert np.isnan(got[touched]).all()


@pytest.mark.parametrize("kind,n,leaf,q,eta,p,ell,deriv", [("cube2", 12, 16, 1, 1.0, 0, 0.5, False),
                                                           ("cube3", 64, 32, 1, 1.0, 1, 0.5, False),
                                                           ("cube3", 1344, 42, 2, 1.0, 2, 0.3, False),
                                                           ("cube2", 47 * 16, 47, 4, 1.0, 3, 0.4, True),
                                                           ("cube3", 700, 6, 2, 1.0, 1, 0.3, False),
                                                           ("sphere", 3001, 32, 1, 1.0, 1, 0.3, True)])
def test_construction_stages_vs_oracle(S, kind, n, leaf, q, eta, p, ell, deriv):
    print(f"case: construction {kind} n={n} leaf={leaf} q={q} deriv={deriv}", flush=True)
    pts = synth.workload_points(kind, n, 14)
    ot = tree.build_tree(pts, leaf)
    ob = samplets.build_samplets(ot, q)
    t = S.Tree(pts, leaf, q)
    pat = S.Pattern.from_tree(t, eta)
    mask = pattern.dense_mask(*pat.download_csr(), n)
    ref = compress.compress_dense(ob, p, ell, 1.0 / n, deriv=deriv)[mask]
    for _ in range(2):
        got = pat.values_to_csr(S.kernel_compress(pat, t, p, ell, 1.0 / n, deriv=deriv)).cpu().numpy()
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert err <= 1e-12, err
