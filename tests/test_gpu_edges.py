"""GPU kernels at the sizes where their splits of the work change: the edges
of tiles and lane groups, remainders, and the smallest and largest of a
range, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1010_1482_amd import workloads as W
from tests.gpu_util import assert_close, host, need_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()
    from paper_1010_1482_amd import hfmm
    hfmm.library()


def H():
    from paper_1010_1482_amd import hfmm
    return hfmm


# ---------------------------------------------------------------- FMM lists
def _points(kind):
    """Particle sets whose lists take many rounds of the traversals."""
    rng = np.random.default_rng(7)
    if kind == "corner":  # cells down to the last level beside coarse leaves
        d = 2.0 ** -np.arange(1, 23)
        near = np.concatenate([0.3 + np.outer(d, v) for v in
                               ((1, 1, 1), (-0.9, 0.7, 0.5), (0.6, -0.8, 0.9))])
        return np.concatenate([near, rng.random((150, 3))])
    # a fine layer beside a few coarse leaves: long U and W lists
    flat = rng.random((2500, 3))
    flat[:, 0] = 0.5 + 1e-5 * flat[:, 0]
    return np.concatenate([flat, rng.random((40, 3))])


@pytest.mark.parametrize("kind,leaf", [("corner", 1), ("layer", 2)])
def test_list_traversals_deep(kind, leaf):
    x, y, z = (np.ascontiguousarray(a) for a in _points(kind).T)
    T = O.Tree(x, y, z, leaf)
    say(f"lists {kind} n={len(x)} leaf={leaf}: {T.ncells} cells, depth {T.depth}")
    t = H().Tree(*to_dev(x, y, z), leaf_max=leaf)
    t.upward(to_dev(np.ones(len(x)))[0], 2, H().FMM, H().FP64)
    for w in range(4):
        off, it = T.list(w)
        goff, git = (a.cpu().numpy() for a in t.fmm_list(w))
        assert np.array_equal(goff, off), w
        for b in range(T.ncells):
            assert np.array_equal(np.sort(git[goff[b]:goff[b + 1]]),
                                  np.sort(it[off[b]:off[b + 1]])), (w, b)
