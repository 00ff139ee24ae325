"""Batches of one dense pattern: levels of so many tiles that the kernels of
whole 64-wide tiles run, at widths and row counts that are no multiples of
their tiles, against a library inverse.  The matrices are those of the tile
edge tests (condition number below 4), with the bars that follow from it."""
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


def _most_tiles(p):
    """Largest number of 64-wide panel tiles and of Schur tiles of a level."""
    b = p.blocks()
    s, c, level = (np.asarray(b[k]) for k in ("s", "c", "level"))
    r = -(-c // 64)
    return [int(np.bincount(level, weights=w).max()) for w in (r * -(-s // 64), r * (r + 1) // 2)]


def _compare(p, sel, matrices, bar):
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(p.n), np.diff(cp))
    n = len(matrices[0])
    for k, a in enumerate(matrices):
        e = slice(cp[k * n], cp[(k + 1) * n])
        q = perm[k * n:(k + 1) * n] - k * n
        x = np.linalg.inv(a[np.ix_(q, q)])
        assert np.abs(sel[e] - x[ri[e] - k * n, cols[e] - k * n]).max() <= bar, k


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("n,cap,count", [(147, 17, 130), (200, 37, 100), (301, 49, 80), (330, 100, 100), (385, 128, 60)])
def test_batch(n, cap, count, det):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1404_0447_amd import selinv as S
    ms = [_dense(n, 1000 * n + k) for k in range(count)]
    p = S.Plan.batch([m for _, m in ms], max_super=cap, exec_cap=cap, deterministic=det).bind()
    assert min(_most_tiles(p)) > 256  # both tiled kernels run
    p.factor(torch.as_tensor(np.concatenate([m.vals for _, m in ms]), device="cuda"))
    sel = p.invert()
    p.sync_status()
    _compare(p, sel.cpu().numpy(), [a for a, _ in ms], 1e-12)


@pytest.mark.parametrize("n,cap,count", [(147, 17, 130), (200, 37, 100), (250, 49, 80), (301, 64, 60)])
def test_poles(n, cap, count):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1404_0447_amd import selinv as S
    a, m = _dense(n, n)
    b, mb = _dense(n, n + 1)
    w = np.linspace(0.3, 0.6, count)
    p = S.Plan.poles(m, count, max_super=cap, exec_cap=cap).bind()
    panel, schur = _most_tiles(p)
    assert panel > 160 and schur > 384  # both tiled kernels run
    p.factor_complex(torch.as_tensor(np.concatenate([m.vals + 1j * x * mb.vals for x in w]), device="cuda"))
    sel = p.invert_complex()
    p.sync_status()
    _compare(p, sel.cpu().numpy(), [a + 1j * x * b for x in w], 1e-12)
