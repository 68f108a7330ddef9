"""The repulsive walk at point counts around the bounds where several waves share
a group of 64 points, around whole groups and blocks, and where the waves' lists
overflow, against the fp64 oracle: the bars of the other parity tests (fp32
gradients within rel-L2 1e-3, Z within 1e-5, interactions within 0.1%; fp64 1e-9,
1e-12, 1e-6)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2212_11506_amd as bh
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# two points have P = Q, so that at exaggeration 1 their gradient is exactly 0 and has no relative error
ALPHA = 12.0


def _p(n):
    return synth.ring_p(n, 3, 2) if n >= 10 else synth.random_p(n, 1)


def _check(g, Z, inter, ref, bars):
    go, Zo, io = ref[:3]
    assert np.linalg.norm(g - go) <= bars[0] * np.linalg.norm(go)
    assert abs(Z - Zo) <= bars[1] * Zo
    assert abs(inter - io) <= bars[2] * io


# groups of 64: up to 480 take 8 waves, up to 6400 blocks of 256 threads; theta 0.05 fills the waves' lists
@pytest.mark.parametrize("n, theta", [(2, 0.5), (63, 0.8), (65, 0.5), (1025, 0.8), (6000, 0.05), (3001, 0.0), (480 * 64, 0.5),
                                      (480 * 64, 0.8), (480 * 64 + 1, 0.5), (480 * 64 + 1, 0.8), (6400 * 64, 0.5),
                                      (6400 * 64 + 1, 0.8)])
def test_walk_2d(n, theta):
    Y = synth.random_y(n, n, dups=n // 10)
    p = _p(n)
    P = bh.Csr.from_numpy(*p, device=DEV)
    ws = torch.empty(bh.workspace_size(n, P.nnz), dtype=torch.uint8, device=DEV)
    g, Z = bh.gradient(torch.from_numpy(Y).to(DEV), P, theta, ALPHA, workspace=ws)
    _check(g.cpu().numpy(), Z, bh.get_stats(ws)["interactions"], oracle.gradient(Y, *p, theta, ALPHA), (1e-3, 1e-5, 1e-3))


# up to 256 groups take 16 waves, 512 8, 1024 4, 8192 2
@pytest.mark.parametrize("n", [3, 66, 256 * 64 + 1, 512 * 64 + 63, 1024 * 64 + 1, 8192 * 64 + 1])
def test_walk_f64(n):
    Y = synth.random_y(n, n, dups=n // 10).astype(np.float64)
    p = _p(n)
    P = bh.CsrF64.from_numpy(*p, device=DEV)
    ws = torch.empty(bh.workspace_size_f64(n, P.nnz), dtype=torch.uint8, device=DEV)
    g, Z = bh.gradient_f64(torch.from_numpy(Y).to(DEV), P, 0.5, ALPHA, workspace=ws)
    _check(g.cpu().numpy(), Z, bh.get_stats(ws)["interactions"], oracle.gradient(Y, *p, 0.5, ALPHA), (1e-9, 1e-12, 1e-6))


# up to 128 groups take 16 waves, then blocks of 256 threads
@pytest.mark.parametrize("n, theta", [(2, 0.5), (65, 0.8), (2049, 0.5), (2000, 0.0), (128 * 64, 0.8), (128 * 64, 0.2),
                                      (128 * 64 + 1, 0.5), (40_000, 0.8)])
def test_walk_3d(n, theta):
    Y = synth.random_y3(n, n, dups=n // 10)
    p = _p(n)
    P = bh.Csr.from_numpy(*p, device=DEV)
    ws = torch.empty(bh.workspace_size_3d(n, P.nnz), dtype=torch.uint8, device=DEV)
    g, Z = bh.gradient_3d(torch.from_numpy(Y).to(DEV), P, theta, ALPHA, workspace=ws)
    _check(g.cpu().numpy(), Z, bh.get_stats(ws)["interactions"], oracle.gradient3(Y, *p, theta, ALPHA), (1e-3, 1e-5, 1e-3))


# one bucket: the walk visits every record, an odd or even number of them, up to the one that ends it
@pytest.mark.parametrize("n", [480 * 64 + 1, 480 * 64 + 2])
@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("theta", [0.5, 0.8])
def test_walk_one_bucket(n, d, theta):
    Y = torch.full((n, d), 1.5, device=DEV)
    P = bh.Csr.from_numpy(*_p(n), device=DEV)
    g, Z = (bh.gradient if d == 2 else bh.gradient_3d)(Y, P, theta, ALPHA)
    assert not g.any()
    # each pair weighs exactly 1, and a point's sum of them is below 2^24
    assert abs(Z - n * (n - 1)) <= 2.0 ** -24 * n * (n - 1)


# Trees of 2n nodes, the most there are: the root has one child, which holds every
# point.  In fp32 only two equal points make one; in fp64 also a box a few ulps wide,
# whose centre rounds to its lower end.
@pytest.mark.parametrize("theta", [0.0, 0.5, 0.8])
@pytest.mark.parametrize("form", ["f32", "layout", "f64", "3d"])
def test_two_equal_points(form, theta):
    Y = torch.full((2, 3 if form == "3d" else 2), 1.5, dtype=torch.float64 if form == "f64" else torch.float32, device=DEV)
    size, grad = {"f64": (bh.workspace_size_f64, bh.gradient_f64), "3d": (bh.workspace_size_3d, bh.gradient_3d)}.get(
        form, (bh.workspace_size, bh.gradient))
    P = (bh.CsrF64 if form == "f64" else bh.Csr).from_numpy(*_p(2), device=DEV)
    ws = torch.empty(size(2, P.nnz), dtype=torch.uint8, device=DEV)
    if form == "layout":
        P = bh.Layout(P, Y, workspace=ws)
    g, Z = grad(Y, P, theta, ALPHA, workspace=ws)
    stats = bh.get_stats(ws)
    assert stats["nodes"] == 4 and stats["interactions"] == 2
    assert Z == 2.0 and not g.any()


@pytest.mark.parametrize("ulps", [[0, 0, 1], [0, 0, 1, 1], [1, 0, 0, 1]])
def test_full_tree_f64(ulps):
    n = len(ulps)
    Y = np.stack([1.0 + np.array(ulps) * 2.0 ** -52, np.full(n, 2.0)], 1)
    p = _p(n)
    P = bh.CsrF64.from_numpy(*p, device=DEV)
    ws = torch.empty(bh.workspace_size_f64(n, P.nnz), dtype=torch.uint8, device=DEV)
    g, Z = bh.gradient_f64(torch.from_numpy(Y).to(DEV), P, 0.5, ALPHA, workspace=ws)
    assert bh.get_stats(ws)["nodes"] == 2 * n
    assert Z == n * (n - 1)  # every weight rounds to 1
    go = oracle.gradient(Y, *p, 0.5, ALPHA)[0]
    assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-9 * np.linalg.norm(go)


# At an angle this wide the outer points take the root, while the two at its centre
# take every point one by one: for an outer point one of those lies at a distance
# beyond the largest float, and must leave its sums alone.
@pytest.mark.parametrize("d", [2, 3])
def test_box_wider_than_the_largest_float(d):
    Y = torch.zeros((4, d), device=DEV)  # (four, each child of the root holds one place: its centre is 0 exactly)
    Y[0, 0], Y[0, 1], Y[1, 0], Y[1, 1] = -2e38, 1e38, 2e38, -1e38
    P = bh.Csr.from_numpy(np.zeros(5, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32), device=DEV)
    g, Z = (bh.gradient if d == 2 else bh.gradient_3d)(Y, P, 1e30, 1.0)
    assert Z == 2.0 and not g.any()  # two equal points; everything else weighs 0


def _late(n, d, seed):
    """clusters of very different width, some points repeated"""
    rng = np.random.default_rng(seed)
    c = rng.integers(0, 9, n)
    Y = rng.uniform(-50.0, 50.0, (9, d))[c] + (10.0 ** rng.uniform(-4, 1, 9))[c, None] * rng.normal(size=(n, d))
    Y[rng.integers(0, n, n // 10)] = Y[0]
    return Y.astype(np.float32)


def _buckets(n, d, seed):
    """nine points in ten in three places"""
    rng = np.random.default_rng(seed)
    Y = rng.normal(size=(n, d))
    m = rng.random(n) < 0.9
    Y[m] = Y[rng.integers(0, 3, n)][m]
    return Y.astype(np.float32)


def _same_in_every_form(Y, theta):
    n, d = Y.shape
    f, Z, inter = bh.debug_walk(Y, theta)
    assert torch.isfinite(f).all()
    if theta == 0.0:
        assert inter == n * (n - 1)
    for form in (0, 1) if d == 2 else (1,):
        f1, Z1, inter1 = bh.debug_walk(Y, theta, form)
        assert torch.equal(f, f1) and inter == inter1
        assert abs(Z - Z1) <= 1e-12 * Z


# Every form of the walk visits the same records for a point and adds them up in the
# same order: the forces agree bit for bit and the interactions exactly (a wave's list
# holds 256 entries: theta 0.05 and 0 fill it, and what is left of its part is walked).
# Z is summed over other groupings of the points, in fp64.
@pytest.mark.parametrize("late", [False, True])
@pytest.mark.parametrize("d, n, theta", [(2, 2, 0.5), (2, 63, 0.8), (2, 65, 0.0), (2, 1025, 0.5), (2, 3001, 0.0),
                                         (2, 6000, 0.05), (2, 9973, 0.8), (2, 480 * 64, 0.5), (2, 480 * 64 + 1, 0.3),
                                         (2, 6400 * 64 + 1, 0.5), (3, 3, 0.5), (3, 65, 0.0), (3, 2000, 0.0),
                                         (3, 2049, 0.8), (3, 128 * 64, 0.2), (3, 128 * 64, 0.5), (3, 128 * 64 + 1, 0.5)])
def test_walk_forms_agree(d, n, theta, late):
    Y = _late(n, d, n) if late else (synth.random_y if d == 2 else synth.random_y3)(n, n, dups=n // 10)
    Y = torch.from_numpy(Y).to(DEV)
    _same_in_every_form(Y, theta)


# A list filled in the middle of a bucket, whose points are records one behind another:
# parts with an odd and an even number of them left, and several such parts in a group.
@pytest.mark.parametrize("theta", [0.1, 0.5, 0.8])
@pytest.mark.parametrize("d, n", [(2, 700), (2, 701), (2, 5003), (2, 480 * 64), (3, 700), (3, 701), (3, 128 * 64)])
def test_walk_forms_agree_in_buckets(d, n, theta):
    _same_in_every_form(torch.from_numpy(_buckets(n, d, n)).to(DEV), theta)


@pytest.mark.parametrize("d, n", [(2, 257), (2, 4001), (2, 4002), (3, 4001), (3, 4002)])
def test_walk_forms_agree_in_one_place(d, n):
    _same_in_every_form(torch.full((n, d), 1.5, device=DEV), 0.5)
