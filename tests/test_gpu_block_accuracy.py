"""Diagonal blocks that are ill-conditioned inside: one dense matrix, one
block, so that the selected inverse is the kernel's T and the exported factor
its L and D.

The bars are those of elimination in the order of the pivots, whatever way a
kernel arranges it:
  inverse   2^-52 kappa times the growth of the elimination (1 for positive
            definite matrices), relative to the largest entry;
  factor    |L D L^T - A| <= (s + 2) 2^-53 sum_k |l_ik d_k l_jk|, which for a
            positive definite matrix is at most (s + 2) 2^-53 max |A|.
References are refined in extended precision.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _matrix(a):
    from paper_1404_0447_amd import workloads as W
    n = len(a)
    cols, rows = np.triu_indices(n)  # row-major upper = lower triangle by columns
    colptr = np.concatenate([[0], np.cumsum(np.arange(n, 0, -1))]).astype(np.int64)
    return W.Matrix(n, colptr, rows.astype(np.int32), a[rows, cols].copy())


def _inverse(a):
    """Refined by Newton steps in extended precision."""
    wide = np.clongdouble if np.iscomplexobj(a) else np.longdouble
    x, al = np.linalg.inv(a).astype(wide), a.astype(wide)
    for _ in range(4):
        x = x @ (2 * np.eye(len(a)) - al @ x)
    return x


def _growth(a):
    """Largest entry of any Schur complement over the largest of A."""
    m, top = a.astype(np.clongdouble if np.iscomplexobj(a) else np.longdouble), np.abs(a).max()
    for j in range(len(a) - 1):
        m = m[1:, 1:] - np.outer(m[1:, 0], m[0, 1:]) / m[0, 0]
        top = max(top, np.abs(m).max())
    return float(top / np.abs(a).max())


def spd(s, kappa, seed):
    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.standard_normal((s, s)))
    w = np.logspace(0, -np.log10(kappa), s)
    rng.shuffle(w)
    a = (q * w) @ q.T
    return 0.5 * (a + a.T)


def gaussian_kernel(s):
    """Smooth: the leading block holds nearly all of the condition number."""
    x = np.linspace(0, 1, s)
    return np.exp(-0.5 * ((x[:, None] - x) / 0.2) ** 2) + 1e-6 * np.eye(s)


def indefinite(s, kappa, seed):
    """A random symmetric matrix whose leading 16 x 16 block has an eigenvalue
    1 / kappa of its largest."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((s, s))
    a = a + a.T
    w, q = np.linalg.eigh(a[:16, :16])
    w[np.argmin(np.abs(w))] = np.abs(w).max() / kappa
    b = (q * w) @ q.T
    a[:16, :16] = 0.5 * (b + b.T)
    return a


def _check(a, run, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1404_0447_amd import selinv as S
    s = len(a)
    m = _matrix(a)
    p = S.Plan.from_matrix(m, **kw).bind()
    v = torch.as_tensor(m.vals, device="cuda")
    if run == "levels":
        p.factor(v)
        sel = p.invert()
    else:
        p.set_schedule(mb_tiles=0)
        sel = p.run(v)
    p.sync_status()  # raises where a pivot is refused
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(s), np.diff(cp))
    ap = a[np.ix_(perm, perm)]
    x = _inverse(ap)
    bar = 2 * U * np.linalg.cond(ap) * _growth(ap)
    assert np.abs(sel.cpu().numpy() - x[ri, cols]).max() <= bar * np.abs(x).max()
    ld = np.zeros((s, s))
    ld[ri, cols] = p.factor_values().cpu().numpy()
    d = np.diag(ld).copy()
    np.fill_diagonal(ld, 1.0)
    wl, wd = ld.astype(np.longdouble), d.astype(np.longdouble)
    terms = np.abs(wl) @ np.diag(np.abs(wd)) @ np.abs(wl).T
    assert (np.abs((wl * wd) @ wl.T - ap) <= (s + 2) * U * terms).all()
    return p, x, ri, cols, perm


RUNS = ["levels", "persistent"]


@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("kappa", [1e2, 1e6, 1e10])
@pytest.mark.parametrize("s", [4, 8, 16, 17, 24, 32, 33, 48, 64, 100, 128])
def test_spd_block(s, kappa, run):
    _check(spd(s, kappa, s), run)


@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("s", [16, 17, 24, 32, 64, 128])
def test_gaussian_kernel_block(s, run):
    _check(gaussian_kernel(s), run)


@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("kappa", [1e2, 1e4, 1e6])
@pytest.mark.parametrize("s", [17, 32, 64, 128])
def test_nearly_singular_leading_block(s, kappa, run):
    _check(indefinite(s, kappa, s), run, require_spd=False)


@pytest.mark.parametrize("s", [24, 128])
def test_gradient(s):
    """d f / d a = -(X S X), X accurate to the inverse's bar on either side."""
    import torch
    a = gaussian_kernel(s)
    p, x, ri, cols, perm = _check(a, "levels")
    w = np.random.default_rng(s).standard_normal(len(ri))
    g = p.backward(torch.as_tensor(w, device="cuda")).cpu().numpy()
    gm = np.zeros((s, s), np.longdouble)
    np.add.at(gm, (ri, cols), w)
    np.add.at(gm, (cols, ri), w)
    back = np.argsort(perm)
    d = -(x @ gm @ x)[np.ix_(back, back)]
    acols, arows = np.triu_indices(s)
    ref = np.where(arows == acols, 0.5, 1.0) * d[arows, acols]
    assert np.abs(g - ref).max() <= 4 * 2 * U * np.linalg.cond(a) * np.abs(ref).max()


def nearly_singular_complex(s, kappa, seed):
    """Complex symmetric, shifted so close to an eigenvalue of its leading
    16 x 16 block that 1 / kappa of it is left."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((s, s)) + 1j * rng.standard_normal((s, s))
    a = 0.5 * (a + a.T)
    lam = np.linalg.eigvals(a[:16, :16])
    return a - lam[np.argmax(np.abs(lam))] * (1.0 - 1.0 / kappa) * np.eye(s)


def _check_complex(a):
    """Complex products carry an error of up to 2 sqrt(2) times a real one's."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1404_0447_amd import selinv as S
    s = len(a)
    m = _matrix(a)
    p = S.Plan.from_matrix(m, complex_values=True).bind()
    p.factor_complex(torch.as_tensor(m.vals, device="cuda"))
    sel = p.invert_complex()
    p.sync_status()
    cp, ri, perm = p.pattern()
    cols = np.repeat(np.arange(s), np.diff(cp))
    ap = a[np.ix_(perm, perm)]
    x = _inverse(ap)
    bar = 2 * np.sqrt(2) * 2 * U * np.linalg.cond(ap) * _growth(ap)
    assert np.abs(sel.cpu().numpy() - x[ri, cols]).max() <= bar * np.abs(x).max()


@pytest.mark.parametrize("kappa", [1e2, 1e4, 1e6])
@pytest.mark.parametrize("s", [16, 17, 32, 33, 48, 64])
def test_complex_nearly_singular_leading_block(s, kappa):
    _check_complex(nearly_singular_complex(s, kappa, s))


@pytest.mark.parametrize("eta", [1.0, 0.1, 0.01])
@pytest.mark.parametrize("s", [17, 33, 64])
def test_complex_near_the_real_axis(s, eta):
    """H + i eta, the matrices of poles next to the spectrum."""
    _check_complex(indefinite(s, 1e2, s) + 1j * eta * np.eye(s))


@pytest.mark.parametrize("s", [8, 16, 32, 48, 64])
def test_complex_roundings_per_pivot(s):
    """Each pivot's update rounds an entry once, at the entry's size.

    Diagonally dominant blocks H + i eta: every pivot changes the diagonal,
    which makes up the norm, by a small part of itself, so a rounding is
    uniform and independent of the others: 2 U / sqrt(12) of the binade's
    floor, over mantissas drawn log-uniformly sqrt(0.75 / (2 ln 2)) of that,
    0.425 U in all.  s pivots add up to 0.425 U sqrt(s); with two roundings a
    pivot it is 0.60 U sqrt(s).  The bar lies midway."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1404_0447_amd import selinv as S
    rng, errors = np.random.default_rng(s), []
    for _ in range(24):
        h = rng.standard_normal((s, s))
        a = 0.5 * (h + h.T) + 1j * 4 * np.sqrt(s) * 2.0 ** rng.uniform() * np.eye(s)
        m = _matrix(a)
        p = S.Plan.from_matrix(m, complex_values=True).bind()
        p.factor_complex(torch.as_tensor(m.vals, device="cuda"))
        sel = p.invert_complex().cpu().numpy()
        p.sync_status()
        _, ri, perm = p.pattern()
        assert len(ri) == s * (s + 1) // 2
        x = np.zeros((s, s), np.clongdouble)
        cols = np.repeat(np.arange(s), np.arange(s, 0, -1))
        x[ri, cols] = x[cols, ri] = sel
        ref = _inverse(a[np.ix_(perm, perm)])
        errors.append(np.sqrt((np.abs(x - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))
    assert np.mean(errors) <= 0.51 * U * np.sqrt(s)
