"""Stored-CSR SpMM: every vector's result is bitwise that of its own SpMV, whatever the number of
vectors (rows of 1, 4, 16 and 32 entry slots, all widths of the vector chunks, full and partial)."""
import pytest

import workloads as wl

from _util import c2_keys, c3_parts, say

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def _molecular(na, nb):
    ops, keys = c3_parts(na, nb)
    return keys, ops


def _phases(n):
    """A ring of hops with phases and a field: complex, some four entries per row per site pair."""
    terms = [(0.25 + 0.1 * q, [(q, 0)]) for q in range(n)]
    for q in range(n):
        p = (q + 1) % n
        terms += [(0.5 + 0.25j, [(q, 6), (p, 5)]), (0.5 - 0.25j, [(q, 5), (p, 6)])]
    return wl.full_space(n), wl.TermList.from_terms(n, terms)


CASES = {  # mean entries per row and with them the slots
    "1 slot": (lambda: (c2_keys(20_001), wl.xxz_grid_6x6()), 0, 6),
    "4 slots": (lambda: (wl.full_space(13), wl.tfim_chain(13)), 6, 24),
    "16 slots": (lambda: _molecular(200, 180), 24, 96),
    "32 slots": (lambda: _molecular(401, 380), 96, 1000),
    "complex, 4 slots": (lambda: _phases(13), 6, 24),
    "complex, 1 slot": (lambda: _phases(5), 0, 6),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("double,index", [(True, qsd.INDEX_I32), (False, qsd.INDEX_I64)])
def test_columns_bitwise(name, double, index):
    make, lo, hi = CASES[name]
    keys, tl = make()
    H = qsd.SubspaceHamiltonian(qsd.Subspace(keys, tl.n_qubits), qsd.operator_from_termlist(tl))
    dtype = ((torch.complex128 if double else torch.complex64) if H.is_complex else
             (torch.float64 if double else torch.float32))
    m = qsd.CsrMatrix(H, index, dtype)
    assert lo <= m.nnz / m.N < hi
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    X = torch.randn((m.N, 16), dtype=dtype, device="cuda", generator=gen)
    want = torch.stack([m.matvec(X[:, v].contiguous()) for v in range(16)], dim=1)
    say("columns", name, dtype, m.N, m.nnz)
    for nvec in (2, 3, 4, 5, 8, 9, 16):
        x = X[:, :nvec].contiguous()
        y = m.matvec(x, out=torch.full_like(x, float("nan")))
        assert torch.equal(y, want[:, :nvec]), nvec
