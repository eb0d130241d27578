"""S x dense on every kind of block row: at most 4, 8, 16 and 32 functions, one column of X to
three passes, pieces shorter and longer than a step of 64 columns.  Against the dense
product in double precision; a row sums at most N terms, 1e-13 of ||A_i|| ||x|| each."""
import numpy as np
import pytest
import torch

import synth
from oracle import pattern

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,leaf,q,eta", [("cube3", 2048, 32, 1, 1.0),     # 4 and 28 functions
                                               ("cube2", 2000, 32, 2, 1.6),     # 6 and 25, 26
                                               ("sphere", 1001, 16, 1, 0.8),    # 4 and 11, 12
                                               ("cube2", 700, 9, 1, 1.0)])      # 3 and 2 to 6
@pytest.mark.parametrize("r", [1, 4, 5, 8, 12, 13, 16, 17, 35])
def test_spmm_block_rows(kind, n, leaf, q, eta, r):
    from paper_2211_11681_amd import spm as S
    print(f"case: spmm {kind} n={n} leaf={leaf} r={r}", flush=True)
    t = S.Tree(synth.workload_points(kind, n, 8), leaf, q)
    pat = S.Pattern.from_tree(t, eta)
    mask = pattern.dense_mask(*pat.download_csr(), n)
    i, j = np.nonzero(mask)
    a = np.zeros((n, n))
    a[i, j] = 2 * synth.pair_uniform(61, i, j, n) - 1
    x = 2 * synth.uniform(62, np.arange(r * n)).reshape(r, n) - 1
    A = pat.values_from_csr(torch.from_numpy(a[mask]).cuda())
    y = S.spmm(pat, A, torch.from_numpy(x).cuda()).cpu().numpy()
    bound = 1e-13 * np.linalg.norm(a, axis=1)[None, :] * np.linalg.norm(x, axis=1)[:, None]
    assert (np.abs(y - x @ a.T) <= bound).all()
