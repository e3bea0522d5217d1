"""The node split's sweeps on the Gram matrix at the sizes where they can go
wrong: columns off and on the block pairs (32), the smallest that take them,
rows on both sides of the preconditioning's limit, spectra that are graded,
degenerate, of low rank or zero, scales near the ends of FP64's range.

Gates: the columns count as orthogonal at |x_i . x_j| <= 8 sqrt(rows) eps |x_i|
|x_j|, twice that for the vectors; values and the product to 1e-13 of the
largest value (a thousand roundings of the up to 600 terms a value sums)."""
import threading

import numpy as np
import pytest
import torch

import paper_1905_01330_amd as tn
from test_gpu_split import decompose_sweeps

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
EPS = np.finfo(np.float64).eps


def check(a):
    u, s, vt, _ = tn.split_node_full_svd(torch.tensor(a, device=DEV), [0], [1])
    torch.cuda.synchronize()
    u, s, vt = (x.cpu().numpy() for x in (u, s, vt))
    s = np.diag(s) if s.ndim == 2 else s
    ref = np.linalg.svd(a, compute_uv=False)
    top = max(ref[0], np.finfo(np.float64).tiny)
    assert np.abs(s - ref).max() <= 1e-13 * top
    assert np.abs((u * s) @ vt - a).max() <= 1e-13 * top
    # rank-deficient nodes: vectors of values at rounding level are not compared
    big = s > 1e-12 * top
    gate = 16 * np.sqrt(max(a.shape)) * EPS
    for q in (u[:, big].T, vt[big]):
        assert np.abs(q @ q.T - np.eye(int(big.sum()))).max(initial=0) <= gate


def spectrum(m, n, s, seed):
    rng = np.random.default_rng(seed)
    u = np.linalg.qr(rng.standard_normal((m, len(s))))[0]
    v = np.linalg.qr(rng.standard_normal((n, len(s))))[0]
    return (u * s) @ v.T


@pytest.mark.parametrize("n", [31, 32, 33, 63, 64, 65, 96, 97, 130, 257])
@pytest.mark.parametrize("extra", [0, 1, 70])
def test_shapes(n, extra):
    check(np.random.default_rng(n + extra).standard_normal((n, n + extra)))


@pytest.mark.parametrize("shape", [(2049, 32), (2100, 70), (40, 2500), (512, 300), (513, 300), (1025, 64), (1500, 50)])
def test_long_sides(shape):
    check(np.random.default_rng(shape[0]).standard_normal(shape))


@pytest.mark.parametrize("rows", [90, 2060])
@pytest.mark.parametrize("kind", ["graded", "degenerate", "rank 5", "zero columns", "orthogonal", "zero", "equal columns"])
def test_spectra(kind, rows):
    n = 66
    if kind == "graded":
        a = spectrum(rows, n, np.exp(-0.5 * np.arange(n)), 1)
    elif kind == "degenerate":
        a = spectrum(rows, n, np.r_[np.ones(33), np.full(33, 0.5)], 2)
    elif kind == "rank 5":
        a = spectrum(rows, n, np.arange(5, 0, -1.0), 3)
    elif kind == "orthogonal":
        a = np.eye(rows, n)[:, ::-1] * np.arange(1.0, n + 1)
    else:
        a = np.random.default_rng(4).standard_normal((rows, n))
        if kind == "zero":
            a[:] = 0
        elif kind == "zero columns":
            a[:, 7::9] = 0
        else:
            a[:, 40:] = a[:, 3:4]
    check(a)


@pytest.mark.parametrize("scale", [1e-120, 1e-60, 1e60])
def test_scales(scale):
    check(scale * np.random.default_rng(5).standard_normal((50, 48)))


def test_small_values_next_to_large_ones():
    """Columns of very different size: each value keeps its own digits (the
    spread columns are orthogonal to 1e-8, so their norms are the values' to 1e-15)."""
    rng = np.random.default_rng(6)
    q = np.linalg.qr(rng.standard_normal((80, 40)))[0]
    norms = 10.0 ** (-rng.permutation(40) / 3.0)
    u, s, vt, _ = tn.split_node_full_svd(torch.tensor(q * norms, device=DEV), [0], [1])
    s = s.cpu().numpy()
    s = np.diag(s) if s.ndim == 2 else s
    np.testing.assert_allclose(s, np.sort(norms)[::-1], rtol=1e-13)


def blocks(rows, sizes, scales, seed):
    """A node of column blocks of independent normal entries, each far below the
    one before it, and its values: a block's are those of what it leaves beside
    the earlier blocks, to the square of the blocks' ratio."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((rows, sum(sizes)))
    r = np.linalg.qr(a)[1]
    ends = np.cumsum(sizes)
    s = [np.linalg.svd(r[e - n:e, e - n:e], compute_uv=False) * f for n, e, f in zip(sizes, ends, scales)]
    return a * np.repeat(scales, sizes), np.concatenate(s)


# block pairs are at most ten in condition: a value's error is ten times the
# gate of the columns' orthogonality (sqrt(rows) 2e-15 there), 1e-12 in all
@pytest.mark.parametrize("rows", [90, 2060])
@pytest.mark.parametrize("scales", [[1, 1e-20, 1e-40, 1e-60], [1, 1e-50, 1e-75, 1e-100], [1e60, 1, 1e-30, 1e-60]])
def test_spread_columns_that_are_not_orthogonal(scales, rows):
    """Columns up to 1e-120 of the largest, not orthogonal to each other nor to
    it: their angles are below single precision's range and the squares of
    their products below double's, and the sweeps on the Gram matrix end all
    the same."""
    a, want = blocks(rows, [16, 20, 10, 4], scales, rows)
    ga = torch.tensor(a, device=DEV)
    k, sweeps = decompose_sweeps(ga, 1)
    assert k == 50 and sweeps <= 20
    s = np.diag(tn.split_node_full_svd(ga, [0], [1])[1].cpu().numpy())
    np.testing.assert_allclose(s, want, rtol=1e-12)


@pytest.mark.parametrize("rows", [90, 2060])
@pytest.mark.parametrize("n", [50, 64])
def test_columns_sweeps_take_over(n, rows):
    """Squares of the small columns vanish in a Gram matrix scaled by the large
    one: its sweeps do not end, and those on the columns finish the node."""
    a, want = blocks(rows, [1, n - 1], [1e89, 1e-72], n)
    ga = torch.tensor(a, device=DEV)
    k, sweeps = decompose_sweeps(ga, 1)
    assert k == n and sweeps > 30
    u, s, vt, _ = (x.cpu().numpy() for x in tn.split_node_full_svd(ga, [0], [1]))
    np.testing.assert_allclose(np.diag(s), want, rtol=1e-12)
    # the small columns' part of the node from the small values alone
    np.testing.assert_allclose(u[:, 1:] @ s[1:, 1:] @ vt[1:, 1:], (a - np.outer(u[:, 0], u[:, 0] @ a))[:, 1:],
                               rtol=0, atol=1e-12 * want[1])


@pytest.mark.parametrize("shape", [(33, 40), (97, 97), (130, 300), (2060, 70)])
def test_workspace_holding_nan(shape):
    """What the workspace held before plays no part: its memory is full of NaN."""
    a = np.random.default_rng(shape[1]).standard_normal(shape)
    poison = torch.full((16 << 20,), float("nan"), dtype=torch.float64, device=DEV)
    del poison
    check(a)


def test_beside_a_capture_on_other_streams():
    """A split leaves a capture that another thread has under way alone, on
    whichever streams either works: its reads share no stream with it."""
    rng = np.random.default_rng(8)
    a = rng.standard_normal((70, 40))
    ga = torch.tensor(a, device=DEV)
    dims = [1, 2, 4, 8, 16, 32, 33, 32, 16, 8, 4, 2, 1]
    raw = [rng.standard_normal((dims[k], 2, dims[k + 1])) for k in range(len(dims) - 1)]
    sites = [torch.tensor(x, device=DEV) for x in raw]
    wantnorm = float(tn.mps_left_canonicalize(sites))
    want = [x.cpu().numpy() for x in sites]
    for x, r in zip(sites, raw):
        x.copy_(torch.tensor(r, device=DEV))
    streams = [torch.cuda.Stream() for _ in range(5)]
    torch.cuda.synchronize()
    got, failed = [], []

    def splits():
        try:
            for st in streams:
                with torch.cuda.stream(st):
                    got.append(tn.split_node_full_svd(ga, [0], [1])[1].cpu().numpy())
        except Exception as e:   # noqa: BLE001 (re-raised on the main thread)
            failed.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        lognorm = tn.mps_left_canonicalize(sites)
        worker = threading.Thread(target=splits)
        worker.start()
        worker.join(60)
    assert not failed, failed
    s0 = np.linalg.svd(a)[1]
    assert len(got) == len(streams)
    for s in got:
        np.testing.assert_allclose(np.diag(s) if s.ndim == 2 else s, s0, rtol=0, atol=1e-13 * s0[0])
    graph.replay()
    torch.cuda.synchronize()
    assert float(lognorm) == wantnorm and all(np.array_equal(x.cpu().numpy(), w) for x, w in zip(sites, want))


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("shape", [(20, 12), (40, 33), (130, 97), (2060, 70)])
def test_a_node_that_is_not_finite(shape, bad):
    """One bad entry: the call ends, keeps every value and shows the entry;
    columns of norm NaN still have a rank each."""
    a = np.random.default_rng(shape[0]).standard_normal(shape)
    a[3, 5] = bad
    u, s, vt, _ = tn.split_node_full_svd(torch.tensor(a, device=DEV), [0], [1])
    torch.cuda.synchronize()
    assert u.shape == (shape[0], shape[1]) and vt.shape == (shape[1], shape[1])
    assert not torch.isfinite(s).all()
