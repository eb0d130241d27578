"""S x dense with 10 to 12 columns of X in a pass, where block rows of at most 8 functions take
one form or the other by their length (a 2^13th of the stored values): a band of clusters and
eight clusters next to everything.  Against the product in double precision, 1e-13 of
||A_i|| ||x|| as a row sums at most N terms.
"""
import numpy as np
import pytest
import scipy.sparse
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [10, 11, 12, 27, 28])
def test_rows_of_both_lengths(r):
    from paper_2211_11681_amd import spm as S
    nc = 3000
    size = np.array([4, 3, 8, 5])[np.arange(nc) % 4]
    cs = np.concatenate([[0], np.cumsum(size)])
    n = int(cs[-1])
    near = [np.arange(nc) if c < 8 else np.unique(np.concatenate([np.arange(8), np.arange(c - 4, min(nc, c + 5))]))
            for c in range(nc)]
    pat = S.Pattern.from_blocks(n, cs, np.cumsum([0] + [len(x) for x in near]), np.concatenate(near))
    cols = np.array([size[x].sum() for x in near])
    assert cols[8:].max() < 0.75 * (pat.n_stored >> 13) and cols[:8].min() > 1.5 * (pat.n_stored >> 13)
    rp, col = pat.download_csr()
    row = np.repeat(np.arange(n), np.diff(rp))
    v = 2 * synth.pair_uniform(61, row, col, n) - 1
    a = scipy.sparse.csr_matrix((v, col, rp), shape=(n, n))
    x = 2 * synth.uniform(62, np.arange(r * n)).reshape(r, n) - 1
    A = pat.values_from_csr(torch.from_numpy(v).cuda())
    y = S.spmm(pat, A, torch.from_numpy(x).cuda()).cpu().numpy()
    norms = np.sqrt(np.asarray(a.multiply(a).sum(axis=1)).ravel())
    bound = 1e-13 * norms[None, :] * np.linalg.norm(x, axis=1)[:, None]
    assert (np.abs(y - (a @ x.T).T) <= bound).all()
