"""The construction's temporary device memory (a panel of rows of K, here 168 MB) is given back
when the call returns, without a further synchronisation.
"""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def test_panel_memory_is_given_back():
    from paper_2211_11681_amd import spm as S
    n = 32768
    t = S.Tree(synth.workload_points("cube2", n, 3), 32, 1)
    pat = S.Pattern.from_tree(t, 1.0)
    out = pat.empty()
    S.kernel_compress(pat, t, 1, 0.3, 1.0 / n, out=out)     # the tree's tables stay
    torch.cuda.synchronize()
    for _ in range(3):
        before = torch.cuda.mem_get_info()[0]
        S.kernel_compress(pat, t, 1, 0.3, 1.0 / n, out=out)
        assert before - torch.cuda.mem_get_info()[0] < 32 << 20
