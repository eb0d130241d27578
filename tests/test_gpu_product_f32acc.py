"""The FP32-accumulate product on the classes of the kernels that load four rows at a time
(every cluster size a multiple of four), against the FP64 oracle: one block by 4 to 7, and
5 to 7 blocks by 5 to 7, both orders, full and masked patterns; with 8 blocks the product
runs on the per-tile kernel.  Tolerance 1e-6 as in the
other FP32 product tests: operands and the sums of 32 k rows are rounded to 2^-24.
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


# N, leaf, eta, blocks of the leaf groups
CASES = [(72, 36, 5.0, 4),        # two leaves of 32 functions
         (24 * 32, 24, 1.0, 5),   # 20 each: members end inside a block and inside a wave's 64 rows
         (28 * 32, 28, 1.0, 6),   # 24
         (32 * 32, 32, 0.6, 7),   # 28
         (36 * 16, 36, 1.0, 8)]   # 32: per-tile kernel


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("n,leaf,eta,blocks", CASES)
def test_f32acc_product_of_four_row_classes(S, n, leaf, eta, blocks, masked):
    print(f"case: f32acc n={n} leaf={leaf} eta={eta} masked={masked}", flush=True)
    t = S.Tree(synth.workload_points("cube3", n, 6), leaf, 1)
    cs = np.asarray(t.arrays()["cluster_start"])
    assert not (np.diff(cs) % 4).any()
    pat = S.Pattern.from_tree(t, eta)
    sides = {(c["row_blocks"], c["col_blocks"]) for c in pat.classes()}
    assert {(1, blocks), (blocks, 1), (blocks, blocks)} <= sides
    mask = pattern.dense_mask(*pat.download_csr(), n)
    i, j = np.nonzero(mask)
    if masked:                           # a symmetric tenth of the positions dropped, the diagonal kept
        drop = (synth.pair_uniform(45, np.minimum(i, j), np.maximum(i, j), n) < 0.1) & (i != j)
        mask[i[drop], j[drop]] = False
        rp = np.concatenate([[0], np.cumsum(mask.sum(1))])
        pat = S.Pattern.from_csr(n, rp, np.nonzero(mask)[1], cs)
        i, j = np.nonzero(mask)
    a, b = np.zeros((n, n)), np.zeros((n, n))
    a[i, j] = 2 * synth.pair_uniform(71, i, j, n) - 1
    b[i, j] = 2 * synth.pair_uniform(72, i, j, n) - 1
    X, Y = (S.convert(pat, pat.values_from_csr(to_dev(v[mask])), "f64", "f32acc") for v in (a, b))
    for ta, tb in [(0, 0), (1, 0), (0, 1)]:
        ref = ops.masked_product(a.T if ta else a, b.T if tb else b, mask)[mask]
        C = S.convert(pat, S.masked_gemm(pat, X, Y, transA=bool(ta), transB=bool(tb), prec="f32acc"), "f32acc", "f64")
        err = np.linalg.norm(pat.values_to_csr(C).cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-6, (ta, tb, err)
