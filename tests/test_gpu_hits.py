"""GPU parity of the element lists of sparse operators.

With a slot-order schedule (and inside a Lanczos solve) an operator with at most N off-diagonal
elements runs from a list of its elements, whose terms are evaluated by each SpMV; an operator
with more runs through the row engine.  Either way a row's sum is formed from the same terms in the
same order, so the results are bitwise those of the table path (QSD_SCHED_HASH_LOOKUP).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import rowwise as orw
from oracle import subspace as osub

from _util import c2_keys, dyadic_vector, heavy_hex_small, say

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu

SLOT = qsd.SCHED_ALL


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def _chain_keys(n, pairs):
    """``n`` strings of 40 qubits, ``pairs`` of which have a neighbour under one XXZ bond."""
    rng = np.random.default_rng(n)
    a = np.unique(rng.integers(0, 1 << 40, size=n, dtype=np.uint64) & ~np.uint64(3) | np.uint64(1))
    b = (a[:pairs] & ~np.uint64(3)) | np.uint64(2)
    return np.concatenate([a[: max(1, n - pairs)], b]).reshape(-1, 1)


def _star_keys(n, others):
    """A string, its ``n`` single flips, and ``others`` far from them and from each other."""
    rng = np.random.default_rng(n)
    ref = int(rng.integers(1, 1 << 50))
    vals = [ref] + [ref ^ (1 << q) for q in range(n)]
    # a parity that single flips change keeps these apart: even weight, none within one flip
    while len(vals) < n + 1 + others:
        v = int(rng.integers(0, 1 << 62)) | (int(rng.integers(0, 1 << 36)) << 62 if n > 62 else 0)
        v &= (1 << n) - 1
        if bin(v ^ ref).count("1") % 2 == 0:
            vals.append(v)
    return wl.ints_to_keys(sorted(set(vals)), n)


# no element at all, one row in few, at most N elements, and more (the row engine): sizes around
# the tile of 256 rows and past the 512 tiles from which a sample is counted first
CASES = {
    "none": (lambda: (c2_keys(3_000), wl.xxz_grid_6x6())),
    "few": (lambda: (_chain_keys(511, 40), wl.xxz_terms(40, [(0, 1), (7, 31)], 1.0, 0.5))),
    "edge": (lambda: (_chain_keys(257, 120), wl.xxz_terms(40, [(0, 1)], 1.0, 0.5))),
    "sampled": (lambda: (_chain_keys(140_000, 30_000), wl.xxz_terms(40, [(0, 1)], 1.0, 0.5))),
    # rows of up to 60 and 100 elements among rows of one (a wave of their own beyond eight)
    "long_rows": (lambda: (_star_keys(60, 3_000), wl.tfim_chain(60))),
    "longer_rows": (lambda: (_star_keys(100, 9_000), wl.tfim_chain(100))),
    "wide": (lambda: heavy_hex_small(4_000)[::-1]),
    "dense": (lambda: (wl.full_space(9), wl.xxz_terms(9, [(q, q + 1) for q in range(8)], 1.0, 0.5))),
    "one_row": (lambda: (c2_keys(1), wl.xxz_grid_6x6())),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("nvec,dtype", [(1, torch.float64), (3, torch.float64), (8, torch.float32), (16, torch.float64)])
def test_list_bitwise(name, nvec, dtype):
    keys, tl = CASES[name]()
    sub = qsd.Subspace(keys, tl.n_qubits)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
    rng = np.random.default_rng(nvec)
    x = torch.from_numpy(rng.standard_normal((sub.N, nvec) if nvec > 1 else sub.N)).to(dtype).cuda()
    say("element list", name, sub.N, nvec, dtype)
    H.schedule = qsd.SCHED_FILTER_FIRST | qsd.SCHED_HASH_LOOKUP
    want = H.matvec(x)
    H.schedule = SLOT
    for _ in range(2):
        y = torch.full_like(x, float("nan"))
        H.matvec(x, out=y)
        assert torch.equal(y, want)
        sub.rehash(0.25)  # the list does not depend on the table
    # a leading dimension beyond the vectors, written beside them
    big = torch.from_numpy(rng.standard_normal((sub.N, nvec + 3))).to(dtype).cuda()
    outs = []
    for s in (SLOT, qsd.SCHED_FILTER_FIRST | qsd.SCHED_HASH_LOOKUP):
        H.schedule = s
        y = torch.full((sub.N, nvec + 2), 7.0, dtype=dtype, device="cuda")
        e = y.element_size()
        H.matvec_raw(nvec, big.data_ptr() + e, nvec + 3, y.data_ptr() + e, nvec + 2, H._dtype_code(big))
        outs.append(y)
    assert torch.equal(*outs) and bool((outs[0][:, 0] == 7.0).all())


@pytest.mark.parametrize("nvec,dtype", [(1, torch.complex128), (3, torch.complex64), (6, torch.complex128)])
def test_list_complex(nvec, dtype):
    """A sparse complex operator (a phase on the hops, a Y word) against the table path, and the
    oracle for dyadic data."""
    keys = _chain_keys(700, 200)
    tl = wl.TermList.from_terms(40, [(0.5 + 0.25j, [(0, 6), (1, 5)]), (0.5 - 0.25j, [(0, 5), (1, 6)]),
                                     (0.75, [(2, 4), (3, 3), (9, 0)]), (1.5, [(4, 0)])])
    sub = qsd.Subspace(keys, 40)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
    rng = np.random.default_rng(3)
    X = dyadic_vector(rng, sub.N, nvec=nvec) + 1j * dyadic_vector(rng, sub.N, nvec=nvec)
    x = torch.from_numpy(X).to(dtype).cuda()
    H.schedule = qsd.SCHED_FILTER_FIRST | qsd.SCHED_HASH_LOOKUP
    want = H.matvec(x)
    H.schedule = SLOT
    assert torch.equal(H.matvec(x), want)
    if dtype == torch.complex128:
        y_o = orw.matvec_c(osub.canonical_keys(keys), tl, X.reshape(sub.N, -1))
        np.testing.assert_array_equal(want.cpu().numpy().reshape(sub.N, -1), y_o)


@pytest.mark.parametrize("graph", [False, True])
def test_solve_bitwise(graph):
    """A solve that makes its own list gives bitwise the energy of one through the table."""
    hh, keys = heavy_hex_small(4_000)
    for k, tl in ((keys, hh), CASES["sampled"]()):
        H = qsd.SubspaceHamiltonian(qsd.Subspace(k, tl.n_qubits), qsd.operator_from_termlist(tl))
        out = []
        for s in (0, qsd.SCHED_HASH_LOOKUP):
            H.schedule = qsd.SCHED_FILTER_FIRST | s
            torch.cuda.synchronize()
            st = torch.cuda.Stream()  # a graph is not captured on the default stream
            e, v, info = H.lanczos(tol=1e-9, max_iter=80, want_vector=True, use_graph=graph, raise_on_nonconv=False,
                                   stream=st)
            st.synchronize()
            out.append((e, info["iterations"], v))
        say("solve", H.N, out[0][:2])
        assert out[0][:2] == out[1][:2] and torch.equal(out[0][2], out[1][2])


# an operator whose schedule was never set takes its rows in slot order where at most one column per
# sampled row is present (fewer rows than the sample, a tile's edge, several tiles), and in canonical
# order otherwise; a set schedule is what it says
@pytest.mark.parametrize("nvec,dtype", [(1, torch.float64), (3, torch.float32), (16, torch.float64)])
@pytest.mark.parametrize("name,n", [("few", 2), ("few", 64), ("few", 257), ("few", 20_001), ("dense", 300),
                                    ("dense", 6000), ("complex", 700)])
def test_unset_schedule_bitwise(name, n, nvec, dtype):
    if name == "dense":
        keys, ops = np.arange(n, dtype=np.uint64).reshape(-1, 1), wl.tfim_chain(40)
    else:
        keys, ops = _chain_keys(n, n // 8), wl.xxz_terms(40, [(0, 1), (7, 31)], 1.0, 0.5)
        if name == "complex":
            ops = wl.TermList.from_terms(40, list(ops.terms()) + [(0.5j, [(3, wl.RAISE), (9, wl.LOWER)]),
                                                                  (-0.5j, [(3, wl.LOWER), (9, wl.RAISE)])], False)
            dtype = {torch.float64: torch.complex128, torch.float32: torch.complex64}[dtype]
    sub = qsd.Subspace(keys, 40)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    assert H.is_complex == (name == "complex")
    default = qsd.SCHED_XCD_REMAP | qsd.SCHED_FILTER_FIRST
    x = torch.randn((sub.N, nvec) if nvec > 1 else sub.N, dtype=dtype, device="cuda")
    say("unset schedule", name, n, nvec, dtype)
    assert H.schedule == default
    y = H.matvec(x, out=torch.full_like(x, float("nan")))
    b = qsd.matvec_batched([H, H], [x, x])
    H.schedule = default
    z = H.matvec(x, out=torch.full_like(x, float("nan")))
    assert torch.equal(y, z) and torch.equal(b[0], z) and torch.equal(b[1], z)
