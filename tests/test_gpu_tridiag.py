"""The lowest eigenpair of a tridiagonal matrix, as the solves find it.

A particle on a chain with hops t and levels e is a tridiagonal matrix in the one-particle strings, and
Lanczos from the first site gives back that matrix exactly: alpha = e, beta = |t|, and the Ritz vector is
the eigenvector.  The eigenvalue is held against LAPACK's and the pair against its residual.

Bounds, over the norm: the multisection ends within 4.4e-16 of the eigenvalue and its minors' rounding
is a change of the entries by a few units; 16 units for the value and 64 for the residual of the pair,
whose twisted factorization has two rounded operations per entry.
"""
import numpy as np
import pytest
from scipy.linalg import eigh_tridiagonal

import workloads as wl

from _util import say

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def _matrix(kind, m):
    rng = np.random.default_rng(m)
    i = np.arange(m)
    if kind == "random":
        return rng.standard_normal(m), 0.1 + rng.random(m - 1)
    if kind == "laplacian":
        return np.full(m, 2.0), np.full(m - 1, 1.0)
    if kind == "graded":  # twelve orders of magnitude, the small end first
        return 10.0 ** (12.0 * i / max(1, m - 1) - 12.0), 0.1 * 10.0 ** (12.0 * i[1:] / max(1, m - 1) - 12.0)
    if kind == "graded down":
        e, t = _matrix("graded", m)
        return e[::-1].copy(), t[::-1].copy()
    if kind == "clustered":  # equal levels, hops of 1e-8 of them
        return np.full(m, -3.0), np.full(m - 1, 3e-8)
    if kind == "split":  # nearly two matrices
        e, t = rng.standard_normal(m), 0.1 + rng.random(m - 1)
        t[(m - 1) // 2] = 1e-11 * 4.0
        return e, t
    if kind == "wilkinson":  # pairs of eigenvalues that agree to many digits, the lowest among them
        return -np.abs(i - (m - 1) / 2.0), np.full(m - 1, 1.0)
    raise ValueError(kind)


def _chain(e, t):
    m = len(e)
    n = max(2, m)
    terms = [(float(x), [(q, wl.P1)]) for q, x in enumerate(e)]
    for q, x in enumerate(t):
        terms += [(float(x), [(q, wl.RAISE), (q + 1, wl.LOWER)]), (float(x), [(q, wl.LOWER), (q + 1, wl.RAISE)])]
    keys = wl.ints_to_keys([1 << q for q in range(m)], n)
    sub = qsd.Subspace(keys, n)
    return qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(wl.TermList.from_terms(n, terms)))


def _check(e, t, m, value, s):
    lo = eigh_tridiagonal(e[:m], t[: m - 1], select="i", select_range=(0, 0))[0][0]
    r = np.abs(np.concatenate([t[: m - 1], [0.0]])) + np.abs(np.concatenate([[0.0], t[: m - 1]]))
    norm = float(np.max(np.abs(e[:m]) + r))
    assert abs(value - lo) <= 16 * EPS * norm, (value, lo)
    assert abs(np.linalg.norm(s) - 1.0) <= 64 * EPS
    assert not np.any(s[m:])
    res = e[:m] * s[:m] - value * s[:m]
    res[1:] += t[: m - 1] * s[: m - 1]
    res[:-1] += t[: m - 1] * s[1:m]
    assert np.linalg.norm(res) <= 64 * EPS * norm
    return np.linalg.norm(res) / norm


@pytest.mark.parametrize("kind", ["random", "laplacian", "graded", "graded down", "clustered", "split", "wilkinson"])
@pytest.mark.parametrize("m", [2, 3, 9, 64, 65, 257, 1000])
def test_chain(kind, m):
    """The whole matrix, and a leading part of it."""
    e, t = _matrix(kind, m)
    H = _chain(e, t)
    v0 = torch.zeros(m, dtype=torch.float64, device="cuda")
    v0[0] = 1.0
    for k in sorted({m, (m + 1) // 2}):
        value, s, info = H.lanczos(max_iter=k, tol=1e-300, v0="user", v0_vector=v0, check_every=97, want_vector=True,
                                   raise_on_nonconv=False)
        # (a solve ends before k where the estimate underflows)
        res = _check(e, t, info["iterations"], value, s.cpu().numpy())
        say("chain", kind, m, k, info["iterations"], value, res)
        if info["iterations"] < m and not info["converged"]:
            j = info["iterations"]
            last = abs(t[j - 1] * s[j - 1].item())
            assert abs(info["ritz_residual"] - last) <= 4 * EPS * max(last, 1e-300)


def test_single_row():
    H = _chain(np.array([-1.5]), np.array([]))
    value, s, info = H.lanczos(want_vector=True)
    assert value == -1.5 and abs(s[0].item()) == 1.0 and info["converged"]
