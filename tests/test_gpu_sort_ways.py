"""The order of the codes at the sizes where the sort changes its way (all against
all, samples and buckets, radix passes) and at the edges of its 64-key groups:
codes, order and permutation are those of a stable sort, for distinct points, for
many equal codes, for codes with equal low words and where the sampled points all
lie before the others, so that one bucket holds nearly everything.  Then the calls
that sort points of another type or a layout's keys."""
import numpy as np
import pytest
import torch

import oracle
import paper_2212_11506_amd as bh
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _sampled(n):
    """the positions that the sample sort looks at"""
    j = np.arange((n + 63) // 64, dtype=np.uint64)
    return np.minimum(j * 64 + (((j * 2654435761) & 0xFFFFFFFF) >> 26), n - 1).astype(np.int64)


def _points(kind, n, d):
    rng = np.random.default_rng(n + d)
    if kind == "random":
        return rng.normal(0, 10, (n, d)).astype(np.float32)
    if kind == "duplicates":
        y = rng.normal(0, 10, (n, d)).astype(np.float32)
        return np.where(rng.uniform(size=(n, 1)) < 0.6, y[:1], y[rng.integers(0, n, n)])
    if kind == "grid":  # few codes, equal low words
        return rng.integers(0, 9, (n, d)).astype(np.float32)
    assert kind == "one_bucket"
    y = rng.uniform(1, 2, (n, d)).astype(np.float32)
    y[_sampled(n)] = rng.uniform(0, 0.1, (_sampled(n).size, d)).astype(np.float32)
    return y


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("kind", ["random", "duplicates", "grid", "one_bucket"])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1000, 8191, 8192, 8193, 8256, 12_345, 20_000, 2**19 - 1, 2**19, 2**19 + 1])
def test_order(n, kind, d):
    y = torch.from_numpy(_points(kind, n, d)).to(DEV)
    codes, scodes, perm, _ = (bh.debug_sort if d == 2 else bh.debug_sort_3d)(y)
    codes = codes.cpu().numpy().view(np.uint64)
    order = np.argsort(codes, kind="stable")
    np.testing.assert_array_equal(perm.cpu().numpy().view(np.uint32), order.astype(np.uint32))
    np.testing.assert_array_equal(scodes.cpu().numpy().view(np.uint64), codes[order])


@pytest.mark.parametrize("n", [8192, 8193])
def test_fp64_and_layouts(n):
    Y, p = synth.random_y(n, 7), synth.random_p(n, 8)
    y = torch.from_numpy(Y).to(DEV)
    P = bh.Csr.from_numpy(*p, device=DEV)
    go, Zo = oracle.gradient(Y, *p, 0.5, 12.0)[:2]
    for form in (P, bh.Layout(P), bh.Layout(P, y)):
        g, Z = bh.gradient(y, form, 0.5, 12.0)
        assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-3 * np.linalg.norm(go)
        assert abs(Z - Zo) <= 1e-5 * Zo
    P64 = bh.CsrF64.from_numpy(p[0], p[1], p[2].astype(np.float64), device=DEV)
    go, Zo = oracle.gradient(Y.astype(np.float64), p[0], p[1], p[2].astype(np.float64), 0.5, 12.0)[:2]
    for form in (P64, bh.LayoutF64(P64, y.double())):
        g, Z = bh.gradient_f64(y.double(), form, 0.5, 12.0)
        # the bars of the fp64 parity tests
        assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-9 * np.linalg.norm(go)
        assert abs(Z - Zo) <= 1e-12 * Zo


@pytest.mark.parametrize("n", [1024, 1025, 2**18, 2**18 + 1])
def test_cell_sums(n):
    """Up to 256 tiles of 1024 points the tiles' totals are scanned by every block: the
    centre of each cell is its points' mean, within fp32 rounding of it and (cells of
    more than 32 points) of a difference of two fp64 prefix sums of y - centre"""
    y = _points("random", n, 2)
    t = bh.debug_tree(torch.from_numpy(y).to(DEV))
    _, _, perm, params = bh.debug_sort(torch.from_numpy(y).to(DEV))
    ys = y[perm.cpu().numpy().view(np.uint32)].astype(np.longdouble)
    b, e = (t[k].cpu().numpy().view(np.uint32).astype(np.int64) for k in ("begin", "end"))
    assert b[0] == 0 and e[0] == n and b.size == t["nodes"]
    sums = np.concatenate([np.zeros((1, 2), np.longdouble), np.cumsum(ys, 0)])
    cnt = (e - b)[:, None]
    com = ((sums[e] - sums[b]) / cnt).astype(np.float64)
    smax = np.abs(y.astype(np.float64) - np.array(params[4:6])).sum(0)
    # (1e-12: the rounding of this reference, prefix sums of 80-bit floats up to 3e6)
    tol = 7e-8 * np.abs(com) + np.where(cnt > 32, 8 * 2.0 ** -52 * smax / cnt, 0.0) + 1e-12 / cnt
    summ = t["summary"].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(summ[:, :2] - com) <= tol)
    assert np.array_equal(summ[:, 2], cnt[:, 0])
