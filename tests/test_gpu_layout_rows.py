"""Relabelled rows of a layout at the lengths where their sort changes form (one,
two, four and eight registers a lane, then LDS, then in their own order), with
columns out of range and graphs whose components only the later entries of a row
join: the gradient through the layout against the oracle (rel-L2 1e-3, Z 1e-5) on
valid rows, and against the plain call (1e-5) where columns are out of range.  At the
point count from which eight registers do not serve, the rows themselves."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
import paper_2212_11506_amd as bh
import synth
from layout_tables import layout_arrays

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _csr(n, lengths, seed, far=False):
    """rows of the given lengths (cycled), distinct columns; symmetric is not needed for the forces"""
    rng = np.random.default_rng(seed)
    col, ptr = [], [0]
    for i in range(n):
        k = min(lengths[i % len(lengths)], n - 1)
        c = rng.choice(n - 1, size=k, replace=False)
        c = np.sort(c + (c >= i))
        col.append(c[::-1] if far else c)
        ptr.append(ptr[-1] + k)
    col = np.concatenate(col).astype(np.int32)
    return np.array(ptr, np.int64), col, (rng.uniform(0.5, 1.5, col.size) / col.size).astype(np.float32)


@pytest.mark.parametrize("lengths", [[0, 1, 2, 3], [63, 64, 65], [127, 128, 129, 1], [255, 256, 257], [511, 512, 513, 5],
                                     [2000, 1, 0, 700]])
@pytest.mark.parametrize("form", ["f32", "f64", "3d"])
def test_row_lengths(lengths, form):
    n = 2600
    p = _csr(n, lengths, sum(lengths))
    if form == "3d":
        Y = synth.random_y3(n, 3)
        lay = bh.Layout3(bh.Csr.from_numpy(*p, device=DEV), torch.from_numpy(Y).to(DEV))
        g, Z = bh.gradient_3d(torch.from_numpy(Y).to(DEV), lay, 0.5, 12.0)
        go, Zo = oracle.gradient3(Y, *p, 0.5, 12.0)[:2]
    elif form == "f64":
        Y = synth.random_y(n, 3).astype(np.float64)
        lay = bh.LayoutF64(bh.CsrF64.from_numpy(*p, device=DEV), torch.from_numpy(Y).to(DEV))
        g, Z = bh.gradient_f64(torch.from_numpy(Y).to(DEV), lay, 0.5, 12.0)
        go, Zo = oracle.gradient(Y, *p, 0.5, 12.0)[:2]
    else:
        Y = synth.random_y(n, 3)
        lay = bh.Layout(bh.Csr.from_numpy(*p, device=DEV), torch.from_numpy(Y).to(DEV))
        g, Z = bh.gradient(torch.from_numpy(Y).to(DEV), lay, 0.5, 12.0)
        go, Zo = oracle.gradient(Y, *p, 0.5, 12.0)[:2]
    assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-3 * np.linalg.norm(go)
    assert abs(Z - Zo) <= 1e-5 * Zo


def test_columns_out_of_range_are_kept_out():
    n = 2600
    ptr, col, val = _csr(n, [60, 200, 300, 600], 5)
    Y = torch.from_numpy(synth.random_y(n, 3)).to(DEV)
    keep = np.arange(col.size) % 7 != 0
    bad = col.copy()
    bad[~keep] = np.where(np.arange((~keep).sum()) % 2 == 0, -1, n + 5)
    g, _ = bh.gradient(Y, bh.Layout(bh.Csr.from_numpy(ptr, bad, val, device=DEV), Y), 0.5, 12.0)
    rows = np.repeat(np.arange(n), np.diff(ptr))[keep]
    ptr2 = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    g2, _ = bh.gradient(Y, bh.Csr.from_numpy(ptr2, col[keep], val[keep], device=DEV), 0.5, 12.0)
    assert float((g - g2).norm()) <= 1e-5 * float(g2.norm())


def test_components_joined_by_later_entries():
    """Four even parts of the index range are rings of near neighbours; single far entries, not among a
    row's first four, join the first two and the last two."""
    n, k = 40_000, 6
    q = n // 4
    i = np.arange(n)
    part = i // q
    near = np.stack([part * q + (i - part * q + o) % q for o in (-3, -2, -1, 1, 2, 3)], 1)
    rows, cols = np.repeat(i, k), near.reshape(-1)
    a = np.array([q - 1, 3 * q - 1])
    b = np.array([2 * q - 1, 4 * q - 1])
    rows = np.concatenate([rows, a, b])
    cols = np.concatenate([cols, b, a])
    o = np.lexsort((cols, rows))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    col = cols[o].astype(np.int32)
    P = bh.Csr.from_numpy(ptr, col, np.full(col.size, 1.0 / col.size, np.float32), device=DEV)
    Y = synth.random_y(n, 1)
    lay = bh.Layout(P, torch.from_numpy(Y).to(DEV))
    perm = lay.mem[:4 * n].view(torch.int32).cpu().numpy()
    comp = perm // (2 * q)  # position -> the half its point lies in
    assert np.array_equal(comp, np.sort(comp)), "a component's points are not together"


@pytest.mark.parametrize("form, longest", [("f32", 8192), ("f64", 4096)])
@pytest.mark.parametrize("over", [0, 1])
def test_rows_at_the_end_of_the_lds_sort(form, longest, over):
    """The longest rows that the sort in LDS takes, and with one entry more."""
    n = 9000
    p = _csr(n, [3] * 1000 + [longest + over, longest - 1], 9)
    Y = synth.random_y(n, 3)
    if form == "f64":
        Y = Y.astype(np.float64)
        lay = bh.LayoutF64(bh.CsrF64.from_numpy(*p, device=DEV), torch.from_numpy(Y).to(DEV))
        g, Z = bh.gradient_f64(torch.from_numpy(Y).to(DEV), lay, 0.5, 12.0)
    else:
        lay = bh.Layout(bh.Csr.from_numpy(*p, device=DEV), torch.from_numpy(Y).to(DEV))
        g, Z = bh.gradient(torch.from_numpy(Y).to(DEV), lay, 0.5, 12.0)
    assert lay.tiles == 0  # a slice with so long a row is mostly padding, or the row is not sorted
    go, Zo = oracle.gradient(Y, *p, 0.5, 12.0)[:2]
    assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-3 * np.linalg.norm(go)
    assert abs(Z - Zo) <= 1e-5 * Zo


@pytest.mark.parametrize("n", [(1 << 23) - 1, 1 << 23])
def test_rows_where_the_place_takes_nine_bits(n):
    """Below 2^23 points rows of up to 512 entries are sorted in registers, from there on up to 256.  The
    rows and columns in use are the last ones, so that the renumbered columns are the largest there are."""
    rng = np.random.default_rng(n)
    lengths = [255, 256, 257, 511, 512, 513] * 7
    rows = np.sort(rng.choice(30_000, len(lengths), replace=False)) + n - 30_000
    rows[-1] = n - 1
    ptr = np.zeros(n + 1, np.int64)
    ptr[rows + 1] = lengths
    ptr = np.cumsum(ptr)
    col = np.concatenate([rng.permutation(30_000)[:k] for k in lengths]).astype(np.int32) + np.int32(n - 30_000)
    val = rng.permutation(col.size).astype(np.float32) + 1.0
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    Y = torch.randn((n, 2), generator=gen, device=DEV)
    lay = bh.Layout(bh.Csr.from_numpy(ptr, col, val, device=DEV), Y)
    end = 2 * 4 * n + 8 * (n + 1) + 2 * 4 * (lay.nnz + 3 * n + 4) + 5 * 256  # of the arrays read below
    perm, rank, rp, c, v = layout_arrays(SimpleNamespace(n=n, nnz=lay.nnz, mem=lay.mem[:end]))
    assert int(rank[col].max()) > n - 30_000
    for r, k in zip(rows, lengths):
        at = rp[rank[r]]
        assert perm[rank[r]] == r and rp[rank[r] + 1] - at == (k + 3) // 4 * 4
        new = rank[col[ptr[r]:ptr[r] + k]].astype(np.int64)
        o = np.argsort(new)
        assert np.array_equal(c[at:at + k], new[o]) and np.array_equal(v[at:at + k], val[ptr[r]:ptr[r] + k][o])
        assert not v[at + k:rp[rank[r] + 1]].any()
