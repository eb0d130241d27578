"""The masked product over patterns with enough one-block units for the two-by-two kernel
(4096 pairs of row group pairs), against the FP64 oracle: clusters of 0 to 9 functions, so
that the 32 k rows of a stage cut clusters, hold eight small ones or one kind of them only,
odd numbers of groups, masked positions.  Tolerance 1e-12 as in the other product tests (a
sum of at most N terms).
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


# cloud, N, leaf, degree, eta
CASES = [("cube2", 2000, 4, 1, 0.25),    # 0 to 6 functions, just above the smallest number of quads
         ("sphere", 2500, 4, 0, 2.0),    # 1 to 3: eight clusters do not fill a stage
         ("cube2", 3000, 16, 1, 1.0),    # 3 to 9
         ("cube3", 2500, 9, 1, 0.4)]     # 1 to 8


def operands(pat, mask, n, seed):
    i, j = np.nonzero(mask)
    out = []
    for s in (seed, seed + 1):
        x = np.zeros((n, n))
        x[i, j] = 2 * synth.pair_uniform(s, i, j, n) - 1
        out.append(x)
    return out + [pat.values_from_csr(to_dev(x[mask])) for x in out]


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("kind,n,leaf,q,eta", CASES)
def test_product_of_quads(S, kind, n, leaf, q, eta, masked):
    print(f"case: quads {kind} n={n} leaf={leaf} q={q} eta={eta} masked={masked}", flush=True)
    t = S.Tree(synth.workload_points(kind, n, 6), leaf, q)
    pat = S.Pattern.from_tree(t, eta)
    mask = pattern.dense_mask(*pat.download_csr(), n)
    if masked:                           # a symmetric tenth of the positions dropped, the diagonal kept
        i, j = np.nonzero(mask)
        drop = synth.pair_uniform(45, np.minimum(i, j), np.maximum(i, j), n) < 0.1
        mask[i[drop & (i != j)], j[drop & (i != j)]] = False
        rp = np.concatenate([[0], np.cumsum(mask.sum(1))])
        pat = S.Pattern.from_csr(n, rp, np.nonzero(mask)[1], t.arrays()["cluster_start"])
    a, b, A, B = operands(pat, mask, n, 51)
    for ta, tb in [(0, 0), (1, 0), (0, 1)]:
        ref = ops.masked_product(a.T if ta else a, b.T if tb else b, mask)[mask]
        C = S.masked_gemm(pat, A, B, transA=bool(ta), transB=bool(tb))
        err = np.linalg.norm(pat.values_to_csr(C).cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-12, (ta, tb, err)


def test_infinities_stay_where_a_tile_meets_them(S):
    # entries without an infinity in any product of stored tiles keep their value
    kind, n, leaf, q, eta = CASES[2]
    t = S.Tree(synth.workload_points(kind, n, 6), leaf, q)
    pat = S.Pattern.from_tree(t, eta)
    mask = pattern.dense_mask(*pat.download_csr(), n)
    a, b, A, B = operands(pat, mask, n, 61)
    cs = np.asarray(t.arrays()["cluster_start"])
    k = int(cs[len(cs) // 2])            # one row of B, in the pattern's columns
    bad = b.copy()
    bad[k] = np.where(mask[k], np.inf, 0.0)
    good = pat.values_to_csr(S.masked_gemm(pat, A, B)).cpu().numpy()
    got = pat.values_to_csr(S.masked_gemm(pat, A, pat.values_from_csr(to_dev(bad[mask])))).cpu().numpy()
    # the rows of a group of up to 16 rows share their middle clusters
    i, j = np.nonzero(mask)
    rows = np.zeros(n, bool)
    for c in np.nonzero([mask[cs[c], k] if cs[c + 1] > cs[c] else False for c in range(len(cs) - 1)])[0]:
        rows[max(0, cs[c] - 16):min(n, cs[c + 1] + 16)] = True
    clean = ~rows[i] | ~mask[k, j]
    assert clean.any() and np.array_equal(got[clean], good[clean])
    assert not np.isfinite(got[~clean]).all()
