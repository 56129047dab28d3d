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


# ---------------------------------------------------------------- sort
# Around the runs of a wave (256 keys) and the tiles of a block (4096), on a
# lattice with about ten particles a site: each leaf's particles, and those of
# a site in their order (the order inside a leaf is free otherwise).
@pytest.mark.parametrize("n", [2, 63, 65, 255, 257, 511, 4095, 4096, 4097, 5121, 8193])
def test_sort_tiles(n):
    rng = np.random.default_rng(n)
    x, y, z = (np.ascontiguousarray(a) for a in (rng.integers(0, 10, (3, n)) / 9.0))
    say(f"sort n={n}")
    T = O.Tree(x, y, z, 64)
    t = H().Tree(*to_dev(x, y, z), leaf_max=64)
    gp, op = t.perm().cpu().numpy(), T.perm()
    cells = T.cells()
    for a, k, nchild in zip(cells["first"], cells["count"], cells["nchild"]):
        if nchild == 0:
            assert np.array_equal(np.sort(gp[a:a + k]), np.sort(op[a:a + k]))
    site = (9 * x + 100 * 9 * y + 10000 * 9 * z).round().astype(int)[gp]
    for v in np.unique(site):
        assert np.all(np.diff(gp[site == v]) > 0)


# ---------------------------------------------------------------- direct sum
# FP64: every term is good to a few 2^-53 and at most 257 of one sign are
# added, so 257 * 2^-53 < 1e-13 bounds phi; the acceleration's terms cancel by
# less than 10 in a uniform cube.  FP32: coordinates rounded to 2^-25 of the
# cube against separations above 1e-3 for all but a few pairs.
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-3)])
@pytest.mark.parametrize("nt,ns", [(1, 1), (7, 64), (9, 257), (64, 63), (65537, 65),
                                   (131075, 257), (262145, 3)])
def test_direct_target_tiles(nt, ns, prec, tol):
    say(f"direct nt={nt} ns={ns} {prec}")
    x, y, z, m = W.uniform(ns, 51)
    tx, ty, tz, _ = W.uniform(nt, 52)
    ref = O.direct_points(x, y, z, m, tx, ty, tz)
    out = host(H().direct(*to_dev(x, y, z, m), precision=prec, targets=to_dev(tx, ty, tz)))
    torch.cuda.synchronize()
    assert_close(out, ref, tol, f"direct {prec}")


# More targets than one launch of 64 a block holds (2^30), on a line beside
# three sources; around the seams and the end.  FP32: coordinates below 7 rounded
# to 2^-24 of themselves and separations above 3, so a few 1e-7 per term.
def test_direct_beyond_one_launch():
    nt = (1 << 30) + 5
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    say(f"direct nt={nt}")
    line = torch.arange(nt, dtype=torch.float64, device="cuda").mul_(2.0 ** -28)
    src = [np.array(v) for v in ([-1.0, -2.0, -1.5], [-1.0, 5.0, 6.0], [-3.0, -1.0, 7.0],
                                 [0.5, 1.0, 0.25])]
    ids = np.r_[0:3, (1 << 29) - 3:(1 << 29) + 3, (1 << 30) - 3:nt]
    out = H().direct(*to_dev(*src), precision="fp32", targets=(line, line, line))
    out = host([o[torch.from_numpy(ids).cuda()] for o in out])
    c = ids * 2.0 ** -28
    assert_close(out, O.direct_points(*src, c, c, c), 1e-5, "beyond one launch")


# ---------------------------------------------------------------- FP32 M2L
# FP32 against the FP64 evaluation of the same approximation: the bar of the
# other FP32 tests.  Small leaves give many cells: 32 and more 256-target tiles
# per octant (tile groups); the flat layer fills four octants (no groups).
@pytest.mark.parametrize("kind,n,leaf,p", [("uniform", 5000, 16, 9), ("uniform", 150000, 2, 8),
                                           ("plummer", 150000, 2, 11), ("layer", 60000, 4, 10)])
def test_fp32_m2l_split_orders_and_tile_groups(kind, n, leaf, p):
    x, y, z, m = W.make("uniform" if kind == "layer" else kind, n, 61)
    if kind == "layer":
        z = 0.25 + 0.0 * z
    tg = W.sample_targets(n, 64, 62)
    ref = O.fmm(x, y, z, m, p, leaf, targets=tg)
    say(f"fmm fp32 {kind} n={n} leaf={leaf} p={p}")
    out = [o[tg] for o in host(H().solve(*to_dev(x, y, z, m), p=p, method="fmm",
                                         precision="fp32", leaf_max=leaf))]
    if kind == "layer":  # the field lies in the plane: its third component is rounding
        out, ref = out[:3], ref[:3]
    assert_close(out, ref, 1e-5, "vs oracle fmm")


# The potential of both signs cancels to a few percent, so that the M2L's own
# rounding shows in it: 2.8e-7 to 5.4e-7 over seeds with FP32 matrix products,
# 1.6e-6 and more when the sources' third BF16 part is lost, 2.2e-6 and more when
# the operator's is too.
@pytest.mark.parametrize("p", [8, 9, 10, 11])
def test_fp32_m2l_split_accuracy(p):
    n = 100003
    x, y, z, _ = W.make("uniform", n, 63)
    m = W.masses(n, 563, "mixed")
    tg = W.sample_targets(n, 2048, 64)
    ref = O.fmm(x, y, z, m, p, 64, targets=tg)
    out = host(H().solve(*to_dev(x, y, z, m), p=p, method="fmm", precision="fp32", leaf_max=64))
    err = O.rel_l2(out[0][tg], ref[0])
    say(f"fmm fp32 mixed n={n} p={p}: phi {err:.2e}")
    assert err < 1e-6


# ---------------------------------------------------------------- P2P
# One leaf of n targets against itself (n at and around the lane splits, and
# above the 64 of one pass), and two-level trees whose lists pack cells into
# partly filled chunks.  FP64: sums of at most 130 (3000) terms of one sign;
# FP32: positions rounded to 2^-24 of the leaf against separations above 1e-4.
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 2e-3)])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 8, 9, 12, 13, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49,
                               64, 65, 130])
def test_p2p_single_leaf(n, prec, tol):
    say(f"p2p one leaf n={n} {prec}")
    x, y, z, m = W.uniform(n, 71)
    ref = O.direct(x, y, z, m)
    out = host(H().solve(*to_dev(x, y, z, m), p=4, method="fmm", precision=prec, leaf_max=n))
    if n == 1:
        assert all(float(o[0]) == 0.0 for o in out)
        return
    assert_close(out, ref, tol, f"one leaf {prec}")


@pytest.mark.parametrize("eps2", [0.0, 1e-4])
@pytest.mark.parametrize("leaf", [3, 20, 64, 100])
def test_p2p_depth_one_tree(leaf, eps2):
    n = 8 * leaf - 3 * (leaf > 3)  # one split, 8 leaves of about `leaf` particles
    x, y, z, m = W.uniform(n, 72)
    T = O.Tree(x, y, z, leaf)
    say(f"p2p n={n} leaf={leaf} eps2={eps2}: depth {T.depth}")
    ref = T.fmm(m, 6, eps2=eps2)
    out = host(H().solve(*to_dev(x, y, z, m), p=6, method="fmm", precision="fp64",
                         leaf_max=leaf, eps2=eps2))
    assert_close(out, ref, 1e-12, "vs oracle fmm")


# ---------------------------------------------------------------- W and X lists
# Leaves of up to 100 particles beside a layer of fine cells: chunks of every
# fill in P2L, W lists short and long against leaves on either side of 64
# targets, at the orders where the terms' split over the lanes changes.  FP64
# as in the other comparisons; FP32 on sets without close pairs.
@pytest.mark.parametrize("kind,leaf,p,prec", [("layer", 2, 1, "fp64"), ("layer", 7, 2, "fp64"),
                                              ("layer", 40, 5, "fp64"), ("layer", 100, 8, "fp64"),
                                              ("layer", 40, 11, "fp64"), ("layer", 20, 16, "fp64"),
                                              ("plummer", 3, 4, "fp32"), ("plummer", 20, 9, "fp32"),
                                              ("plummer", 100, 16, "fp32")])
def test_fmm_w_and_x_lists(kind, leaf, p, prec):
    if kind == "layer":
        x, y, z = (np.ascontiguousarray(a) for a in _points(kind).T)
        m = np.random.default_rng(8).uniform(0.5, 1.5, len(x)) / len(x)
    else:
        x, y, z, m = W.make(kind, 6000, 45)
    T = O.Tree(x, y, z, leaf)
    longest = [int(np.diff(T.list(w)[0]).max()) for w in (2, 3)]
    say(f"fmm {prec} {kind} n={len(x)} leaf={leaf} p={p}: longest W, X {longest}")
    assert min(longest) > 0
    out = host(H().solve(*to_dev(x, y, z, m), p=p, method="fmm", precision=prec, leaf_max=leaf))
    assert_close(out, T.fmm(m, p), 1e-12 if prec == "fp64" else 1e-5, "vs oracle fmm")


# ---------------------------------------------------------------- treecode
# Barnes-Hut lists and the p = 3 far field on leaves of every size up to and
# beyond the lanes of a wave, and down to the last levels of the key.
@pytest.mark.parametrize("kind,n,leaf", [("plummer", 3000, 1), ("plummer", 4001, 3),
                                         ("uniform", 20000, 70), ("uniform", 9000, 150),
                                         ("corner", 0, 1)])
def test_treecode_far_leaf_sizes(kind, n, leaf):
    if kind == "corner":
        x, y, z = (np.ascontiguousarray(a) for a in _points(kind).T)
        m = np.full(len(x), 1.0 / len(x))
    else:
        x, y, z, m = W.make(kind, n, 81)
    say(f"treecode p=3 {kind} n={len(x)} leaf={leaf}")
    T = O.Tree(x, y, z, leaf)
    for theta in (0.5, 0.8):
        ref = O.treecode(x, y, z, m, 3, theta, leaf)
        t = H().Tree(*to_dev(x, y, z), leaf_max=leaf)
        t.upward(to_dev(m)[0], 3, H().TREECODE, H().FP64)
        out = host(t.evaluate(theta=theta))
        for w in range(2):
            off, it = T.bh_lists(m, theta, w)
            goff, git = (a.cpu().numpy() for a in t.bh_list(w))
            for b in range(T.ncells):
                assert np.array_equal(np.sort(git[goff[b]:goff[b + 1]]),
                                      np.sort(it[off[b]:off[b + 1]])), (w, b)
        assert_close(out, ref, 1e-12, f"theta {theta} fp64")
        if kind != "corner":  # (there the closest pairs are beyond FP32)
            out = host(H().solve(*to_dev(x, y, z, m), p=3, method="treecode", theta=theta,
                                 precision="fp32", leaf_max=leaf))
            assert_close(out, ref, 2e-5, f"theta {theta} fp32")


# The FP32 range of the treecodes' far field at p = 3: sums over moments and
# distances in fixed units must not leave it where the field itself does not.
# Scaling masses and lengths by powers of two scales every FP32 operation
# exactly (separations here are above 1e-3, far from the 1e-12 at which P2P
# starts to round differently), so the scaled results are those of the unscaled
# set but for the FP64 box geometry's last bits: 1e-6 of the largest value.
# 20000 stars of 2^108 at 2^55 (a total of 7e36 within 4e16); masses of 1e-34.
@pytest.mark.parametrize("method", ["treecode", "treecode_fmmlist"])
@pytest.mark.parametrize("me,le", [(108, 55), (-113, 0), (-20, 20)])
def test_treecode_fp32_range(method, me, le):
    x, y, z, _ = W.make("plummer", 20000, 83)
    m = np.random.default_rng(84).uniform(0.5, 1.5, len(x))
    say(f"{method} masses 2^{me} lengths 2^{le}")

    def field(a, b):
        c = 2.0 ** b
        o = host(H().solve(*to_dev(x * c, y * c, z * c, m * 2.0 ** a), p=3, method=method,
                           precision="fp32", leaf_max=16))
        return [o[0] * 2.0 ** (b - a)] + [v * 2.0 ** (2 * b - a) for v in o[1:]]

    assert_close(field(me, le), field(0, 0), 1e-6, "scaled vs unscaled")


# Targets far outside a tiny set: only the far field's scale counts (1/S^2 is
# beyond FP32, the field is not).
@pytest.mark.parametrize("method", ["treecode", "treecode_fmmlist"])
def test_treecode_fp32_range_small_lengths(method):
    x, y, z, m = W.make("plummer", 3000, 85)
    rng = np.random.default_rng(86)
    tx, ty, tz = (np.ascontiguousarray(a) for a in rng.uniform(400.0, 900.0, (3, 50)))
    ref = O.direct_points(x, y, z, m, tx, ty, tz)
    say(f"{method} lengths 2^-70")
    c, k = 2.0 ** -70, 2.0 ** -40
    o = host(H().solve(*to_dev(x * c, y * c, z * c, m * k), p=3, method=method, precision="fp32",
                       leaf_max=16, targets=to_dev(tx * c, ty * c, tz * c)))
    # the octupole that p = 3 leaves out: below (20 / 700)^3 of the field
    assert_close([o[0] * (c / k)] + [v * (c * c / k) for v in o[1:]], ref, 1e-4, "vs direct")


# ---------------------------------------------------------------- list sizes
# With theta = 0 every box meets every leaf: 50000 leaves of one particle make
# 2.5e9 P2P items, more than the int32 offsets hold.  Refused from the counts,
# before anything is written, and the tree goes on with the next evaluation; the
# same boxes at theta = 0.9 (below the limit, summed in 64 bits too) against the
# oracle, FP64 as in the other comparisons.
@pytest.mark.parametrize("nt", [0, 150000])
def test_bh_lists_beyond_int32_refused(nt):
    n = 50000
    x, y, z, m = W.uniform(n, 91)
    dev = to_dev(x, y, z, m)
    tp = W.uniform(nt, 92)[:3] if nt else None
    tg = to_dev(*tp) if nt else None
    say(f"bh list items beyond int32 nt={nt}")
    t = H().Tree(*dev[:3], leaf_max=1, max_targets=nt)
    t.upward(dev[3], 3, H().TREECODE, H().FP64)
    first = host(t.evaluate(theta=0.9, targets=tg))
    st = t.stats()
    assert (st["n_target_boxes"] if nt else n) * n > 2 ** 31
    with pytest.raises(H().HfmmError) as e:
        t.evaluate(theta=0.0, targets=tg)
    assert e.value.code == H().E_UNSUPPORTED
    out = host(t.evaluate(theta=0.9, targets=tg))
    assert all(np.array_equal(a, b) for a, b in zip(out, first))
    ids = W.sample_targets(nt or n, 64, 93)
    T = O.Tree(x, y, z, 1)
    ref = (T.treecode_points(m, 3, 0.9, *[c[ids] for c in tp]) if nt
           else T.treecode(m, 3, 0.9, targets=ids))
    assert_close([o[ids] for o in out], ref, 1e-12, "theta 0.9 vs oracle")


# 4e6 boxes with about 190 V cells on each of some seven levels: 3e9 M2P items.
def test_box_lists_beyond_int32_refused():
    n, nt = 1 << 21, 1 << 23
    rng = np.random.default_rng(94)
    src = to_dev(*rng.random((3, n)))
    tg = to_dev(*rng.random((3, nt)))
    say(f"box list items beyond int32 n={n} nt={nt}")
    t = H().Tree(*src, leaf_max=1, max_targets=nt, arena_bytes_hint=48 << 30)
    t.upward(torch.ones(n, dtype=torch.float64, device="cuda"), 1, H().TREECODE_FMMLIST,
             H().FP32)
    with pytest.raises(H().HfmmError) as e:
        t.evaluate(targets=tg)
    assert e.value.code == H().E_UNSUPPORTED


# 1.9e7 cells, whose V entries number beyond int32 (they are not packed, so the
# count is all that could wrap): a cell of the interior has 189.
def test_v_list_total_beyond_int32():
    say("V entries beyond int32")
    # a lattice of 256^3 sites, one particle each, in one cell each of level 8
    g = (torch.arange(256, dtype=torch.float64, device="cuda") + 0.5) / 256
    x, y, z = (a.reshape(-1).contiguous() for a in torch.meshgrid(g, g, g, indexing="ij"))
    # (the root's faces, so that the cells are the lattice's)
    ends = torch.tensor([0.0, 1.0], dtype=torch.float64, device="cuda")
    x, y, z = (torch.cat([a, ends]) for a in (x, y, z))
    t = H().Tree(x, y, z, leaf_max=2, arena_bytes_hint=64 << 30)
    t.upward(torch.ones_like(x), 1, H().FMM, H().FP32)
    st = t.stats()
    # sources within +-3 of a cell per axis that are children of the parents'
    # neighbours, less the adjacent ones, summed over the cells of a level
    want = 0
    for lv in range(2, 9):
        k = 2 ** lv
        near = sum(min(k - 1, c + 1) - max(0, c - 1) + 1 for c in range(k))
        par = sum(min(k, 2 * (c // 2) + 4) - max(0, 2 * (c // 2) - 2) for c in range(k))
        want += par ** 3 - near ** 3
    assert st["n_cells"] == sum(8 ** lv for lv in range(9))
    assert st["list_v"] == want and want > 2 ** 31


# Lengths whose squares overflow or lose bits: the lists are still those of the
# acceptance itself, here at 2^-525 and 2^511 times a Plummer sphere.
@pytest.mark.parametrize("le", [-525, 0, 511])
def test_bh_lists_at_extreme_lengths(le):
    x, y, z, m = W.make("plummer", 3000, 87)
    x, y, z = (a * 2.0 ** le for a in (x, y, z))
    say(f"bh lists, lengths 2^{le}")
    T = O.Tree(x, y, z, 1)
    t = H().Tree(*to_dev(x, y, z), leaf_max=1)
    t.upward(to_dev(m)[0], 3, H().TREECODE, H().FP64)
    t.evaluate(theta=0.7)
    for w in range(2):
        off, it = T.bh_lists(m, 0.7, w)
        goff, git = (a.cpu().numpy() for a in t.bh_list(w))
        assert np.array_equal(goff, off)
        for b in range(T.ncells):
            assert np.array_equal(np.sort(git[goff[b]:goff[b + 1]]),
                                  np.sort(it[off[b]:off[b + 1]])), (w, b)
