"""The product kernels that the patterns of the GPU tests reach, from the plan (no GPU): pairs
of row group pairs at or above the smallest number for k_mgemm_quad, and the classes of the
FP32-accumulate kernels.  The groups of one 16-row block are formed here as the planner forms
them, which its number of one-block units confirms.
"""
import os
import re

import numpy as np
import pytest

import synth
import test_gpu_product_f32acc as f32acc
import test_gpu_product_quads as quads
from oracle import pattern
from paper_2211_11681_amd import spm as S


def constant(name):
    path = os.path.join(os.path.dirname(S.__file__), "csrc", "spm_internal.h")
    return int(re.search(rf"constexpr int(?:64_t)? {name} = (\d+);", open(path).read()).group(1))


def quad_count(cs, near):
    """One-block units and quads of a pattern whose clusters have at most 16 functions."""
    slot = -(-np.diff(cs) // 4) * 4
    group, g, k = np.full(len(slot), -1), -1, 0
    for c in range(len(slot)):
        if slot[c] == 0:                                # ends a group as any other change of slot
            k = 0
            continue
        if k == 0 or slot[c] != slot[c - 1] or k == 16 // slot[c]:
            g, k = g + 1, 0
        group[c] = g
        k += 1
    i, j = np.nonzero(near)
    i, j = group[i], group[j]
    i, j = i[(i >= 0) & (j >= 0)], j[(i >= 0) & (j >= 0)]
    return len(np.unique(i * (g + 1) + j)), len(np.unique((i // 2) * (g + 1) + j // 2))


def plan(kind, n, leaf, q, eta, masked):
    t = S.Tree(synth.workload_points(kind, n, 6), leaf, q)
    cs = np.asarray(t.arrays()["cluster_start"])
    rp, col = t.block_pattern(eta)
    near = np.zeros((len(cs) - 1, len(cs) - 1), bool)
    near[np.repeat(np.arange(len(cs) - 1), np.diff(rp)), col] = True
    if not masked:
        return S.Pattern.plan_blocks(n, cs, rp, col), cs, near
    mask = pattern.dense_mask(*S.Pattern.plan_blocks(n, cs, rp, col).download_csr(), n)
    i, j = np.nonzero(mask)
    drop = synth.pair_uniform(45, np.minimum(i, j), np.maximum(i, j), n) < 0.1
    mask[i[drop & (i != j)], j[drop & (i != j)]] = False
    pat = S.Pattern.plan_csr(n, np.concatenate([[0], np.cumsum(mask.sum(1))]), np.nonzero(mask)[1], cs)
    own = np.repeat(np.arange(len(cs) - 1), np.diff(cs))
    i, j = np.nonzero(mask)
    near[:] = False
    near[own[i], own[j]] = True
    return pat, cs, near


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("kind,n,leaf,q,eta", quads.CASES)
def test_quad_cases_reach_quads(kind, n, leaf, q, eta, masked):
    pat, cs, near = plan(kind, n, leaf, q, eta, masked)
    units, nq = quad_count(cs, near)
    assert [c["units"] for c in pat.classes() if c["row_blocks"] == c["col_blocks"] == 1] == [units]
    assert nq >= constant("kQuadMin"), nq


def test_a_small_pattern_keeps_single_units():
    pat, cs, near = plan("cube2", 1000, 12, 1, 0.5, False)
    units, nq = quad_count(cs, near)
    assert [c["units"] for c in pat.classes() if c["row_blocks"] == c["col_blocks"] == 1] == [units]
    assert 0 < nq < constant("kQuadMin"), nq


@pytest.mark.parametrize("n,leaf,eta,blocks", f32acc.CASES)
def test_f32acc_cases_and_the_side_kernel(n, leaf, eta, blocks):
    # units of one block by 4 to 7 take the side kernel; a group of 8 blocks has a class of
    # 8 x 8, and a pattern with a class above 7 blocks takes the per-tile kernel throughout
    pat, cs, _ = plan("cube3", n, leaf, 1, eta, False)
    assert not (np.diff(cs) % 4).any()
    sides = {(c["row_blocks"], c["col_blocks"]) for c in pat.classes()}
    assert {(1, blocks), (blocks, 1)} <= sides
    assert (max(max(s) for s in sides) > 7) == (blocks == 8)
