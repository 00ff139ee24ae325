"""Dense matrices, whose blocks take exactly the widths asked for, at the
edges of the kernels' tiles: forward and gradient against a library inverse.

A dense matrix of order n with supernodes capped at `cap` is a chain of
blocks of `cap` columns and a remainder, each with all later columns below
it.  The matrices are diagonally dominant (condition number below 4), so
with errors of about n * 2^-53 per product the bars of 1e-12 leave two
orders of magnitude.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _dense(n, seed):
    from paper_1404_0447_amd import workloads as W
    rng = np.random.default_rng(seed)
    a = rng.uniform(-1.0, 1.0, (n, n)) / n
    a = 0.5 * (a + a.T) + np.eye(n)
    cols, rows = np.triu_indices(n)  # row-major upper = lower triangle by columns
    colptr = np.concatenate([[0], np.cumsum(np.arange(n, 0, -1))]).astype(np.int64)
    return a, W.Matrix(n, colptr, rows.astype(np.int32), a[rows, cols].copy())


def _plan(m, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1404_0447_amd import selinv as S
    return S.Plan.from_matrix(m, **kw).bind()


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("n,cap", [(1, 128), (15, 128), (16, 128), (17, 128), (33, 128), (65, 128), (127, 128),
                                   (128, 128), (129, 128), (200, 37), (330, 100), (600, 128), (777, 100)])
def test_dense_gradient(n, cap, det):
    import torch
    a, m = _dense(n, n)
    p = _plan(m, max_super=cap, deterministic=det)
    p.factor(torch.as_tensor(m.vals, device="cuda"))
    p.invert()
    p.sync_status()
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(n), np.diff(cp))
    w = np.random.default_rng(n + 1).standard_normal(len(ri))
    g = p.backward(torch.as_tensor(w, device="cuda")).cpu().numpy()
    i, j = perm[ri], perm[cols]
    gm = np.zeros((n, n))
    np.add.at(gm, (i, j), w)
    np.add.at(gm, (j, i), w)
    x = np.linalg.inv(a)
    d = -(x @ gm @ x)
    acols, arows = np.triu_indices(n)
    ref = np.where(arows == acols, 0.5, 1.0) * d[arows, acols]
    assert np.abs(g - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("run", ["levels", "persistent"])
@pytest.mark.parametrize("n,cap", [(1, 128), (2, 128), (15, 128), (16, 128), (17, 128), (31, 128), (32, 128),
                                   (33, 128), (48, 128), (63, 128), (64, 128), (65, 128), (112, 128), (113, 128),
                                   (127, 128), (128, 128), (129, 128), (90, 17), (135, 64), (250, 49), (385, 128), (777, 128), (1153, 96)])
def test_dense_forward(n, cap, run):
    """Selected inverse and factor of chains of blocks of `cap` columns."""
    import torch
    a, m = _dense(n, n)
    p = _plan(m, max_super=cap, exec_cap=min(cap, 128))
    v = torch.as_tensor(m.vals, device="cuda")
    if run == "levels":
        p.factor(v)
        sel = p.invert()
    else:
        p.set_schedule(mb_tiles=0, small_s=0)
        sel = p.run(v)
    p.sync_status()
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(n), np.diff(cp))
    ap = a[np.ix_(perm, perm)]
    assert np.abs(sel.cpu().numpy() - np.linalg.inv(ap)[ri, cols]).max() <= 1e-12
    lv = p.factor_values().cpu().numpy()
    ld = np.zeros((n, n))
    ld[ri, cols] = lv
    d = np.diag(ld).copy()
    np.fill_diagonal(ld, 1.0)
    assert np.abs(ld @ np.diag(d) @ ld.T - ap).max() <= 1e-12


@pytest.mark.parametrize("run", ["levels", "persistent"])
@pytest.mark.parametrize("n,cap", [(9, 2), (14, 3), (21, 4), (30, 5), (34, 7), (49, 8), (50, 9), (61, 12), (47, 15),
                                   (64, 16), (65, 16), (272, 16), (271, 13)])
def test_small_blocks(n, cap, run):
    """Blocks of at most 16 columns, each whole on one wave; the rows below
    them run through every count from 0 to n - cap that the chain has."""
    import torch
    a, m = _dense(n, n)
    p = _plan(m, max_super=cap, exec_cap=cap)
    v = torch.as_tensor(m.vals, device="cuda")
    if run == "levels":
        p.factor(v)
        sel = p.invert()
    else:
        p.set_schedule(small_s=16)
        sel = p.run(v)
    p.sync_status()
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(n), np.diff(cp))
    ap = a[np.ix_(perm, perm)]
    assert np.abs(sel.cpu().numpy() - np.linalg.inv(ap)[ri, cols]).max() <= 1e-12
    ld = np.zeros((n, n))
    ld[ri, cols] = p.factor_values().cpu().numpy()
    d = np.diag(ld).copy()
    np.fill_diagonal(ld, 1.0)
    assert np.abs(ld @ np.diag(d) @ ld.T - ap).max() <= 1e-12


@pytest.mark.parametrize("n,cap", [(1, 64), (2, 64), (15, 64), (16, 64), (17, 64), (31, 64), (33, 64), (63, 64), (64, 64),
                                   (65, 64), (90, 17), (129, 32), (250, 49), (333, 64), (777, 64)])
def test_dense_complex(n, cap):
    """Selected inverse of complex symmetric chains: diagonal 1 + i / 2."""
    import torch
    a, m = _dense(n, n)
    b, mb = _dense(n, n + 1)
    z = a + 0.5j * b
    p = _plan(m, max_super=cap, exec_cap=cap, complex_values=True)
    p.factor_complex(torch.as_tensor(m.vals + 0.5j * mb.vals, device="cuda"))
    sel = p.invert_complex()
    p.sync_status()
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(n), np.diff(cp))
    x = np.linalg.inv(z[np.ix_(perm, perm)])
    assert np.abs(sel.cpu().numpy() - x[ri, cols]).max() <= 1e-12
