"""An infinity in one operand of the FP64 product, where units of one block by five have
waves over two clusters of 20 functions: a result whose clusters do not both have a tile at
the infinity's cluster keeps its value.  Four clusters of 4 functions next to everything and
two groups of four clusters of 20, cluster k of one next to cluster k of the other, so that a
stage of 32 k rows holds one of the large clusters (all but the last one, which the small
ones join).
"""
import numpy as np
import pytest
import torch

from oracle import pattern

pytestmark = pytest.mark.gpu

SIZES = [4] * 4 + [20] * 8


@pytest.fixture(scope="module")
def S():
    from paper_2211_11681_amd import spm
    spm._lib.load()
    assert torch.cuda.is_available()
    return spm


@pytest.mark.parametrize("wide_rows", [True, False])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_infinity_beside_absent_tiles(S, wide_rows, value):
    nc, n = len(SIZES), sum(SIZES)
    cs = np.concatenate([[0], np.cumsum(SIZES)])
    near = np.eye(nc, dtype=bool)
    near[:4], near[:, :4] = True, True
    near[range(4, 8), range(8, 12)] = near[range(8, 12), range(4, 8)] = True
    pat = S.Pattern.from_blocks(n, cs, np.concatenate([[0], np.cumsum(near.sum(1))]), np.nonzero(near)[1])
    assert {(1, 5), (5, 1)} <= {(c["row_blocks"], c["col_blocks"]) for c in pat.classes()}
    mask = pattern.dense_mask(*pat.download_csr(), n)
    rng = np.random.RandomState(3)
    a, b = (np.where(mask, rng.uniform(0.1, 1.0, (n, n)), 0.0) for _ in range(2))

    def product(x, y):
        x, y = (pat.values_from_csr(torch.from_numpy(v[mask]).cuda()) for v in (x, y))
        out = np.zeros((n, n))
        out[mask] = pat.values_to_csr(S.masked_gemm(pat, x, y)).cpu().numpy()
        return out if wide_rows else out.T               # rows: the large clusters

    good = product(a, b)
    for mu in range(4, nc - 1):
        k = int(cs[mu]) + 7
        bad = b.copy() if wide_rows else a.T.copy()
        bad[k] = np.where(mask[k], value, 0.0)
        got = product(a, bad) if wide_rows else product(bad.T, b)
        for c in range(4, nc):
            rows = slice(int(cs[c]), int(cs[c + 1]))
            if near[c, mu]:
                assert not np.isfinite(got[rows, :16]).any(), (mu, c)
            else:
                assert np.array_equal(got[rows, :16], good[rows, :16]), (mu, c)
