"""Sizes at which a launch, a table or an allocation meets its limit: what was accepted there stays
accepted, and gives the results of the ordinary sizes."""
import numpy as np
import pytest

import workloads as wl

from _util import c2_keys, say
from test_gpu_hits import CASES

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu

DEFAULT = qsd.SCHED_XCD_REMAP | qsd.SCHED_FILTER_FIRST


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def test_table_of_2_to_32_slots():
    """The largest table that is accepted (34 GB): built and rehashed to, every string is found and
    the SpMV is bitwise that of the ordinary table."""
    keys, tl = c2_keys(4_200), wl.xxz_grid_6x6()
    op = qsd.operator_from_termlist(tl)
    small = qsd.Subspace(keys, tl.n_qubits)
    x = torch.randn(small.N, dtype=torch.float64, device="cuda")
    want = qsd.SubspaceHamiltonian(small, op).matvec(x)
    for sub in (qsd.Subspace(keys, tl.n_qubits, max_load=1e-6), small):
        if sub is small:
            sub.rehash(1e-6)
        say("slots", sub.capacity)
        assert sub.capacity == 1 << 32
        assert torch.equal(sub.lookup(sub.keys()), torch.arange(sub.N, device="cuda"))
        H = qsd.SubspaceHamiltonian(sub, op)
        for sched in (DEFAULT, qsd.SCHED_ALL, qsd.SCHED_SLOT_ORDER | qsd.SCHED_HASH_LOOKUP):
            H.schedule = sched
            assert torch.equal(H.matvec(x), want)
        del H, sub
        torch.cuda.empty_cache()


def _flips(nlo, nhi, split, qubits):
    """Rows (a, b), a < nlo and b < nhi, of strings of 2 * split qubits, ascending, on the GPU, and the
    sum of X on ``qubits`` with a field."""
    b = torch.arange(nhi, dtype=torch.int64, device="cuda") << split
    keys = (b[:, None] + torch.arange(nlo, dtype=torch.int64, device="cuda")[None, :]).reshape(-1, 1)
    terms = [(0.25 + 0.125 * k, [(q, wl.X)]) for k, q in enumerate(qubits)]
    terms += [(0.5 + 0.0625 * q, [(q, wl.Z)]) for q in range(2 * split)]
    return keys, wl.TermList.from_terms(2 * split, terms)


def test_csr_spmm_of_2_to_26_rows():
    """Rows times lanes of a row reach 2^32: 16 vectors on a matrix of nine entries per row."""
    keys, tl = _flips(4096, 16384, 14, (0, 1, 5, 11, 14, 15, 20, 27))
    sub = qsd.Subspace(keys, 28, assume_sorted_unique=True)
    del keys
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
    m = qsd.CsrMatrix(H, dtype=torch.float32)
    assert m.N == 1 << 26 and m.nnz == 9 * m.N
    say("csr", m.N, m.nnz)
    X = torch.randn((m.N, 16), dtype=torch.float32, device="cuda")
    Y = m.matvec(X, out=torch.full_like(X, float("nan")))
    for v in (0, 7, 15):
        assert torch.equal(m.matvec(X[:, v].contiguous()), Y[:, v])
    del X, Y, m, H, sub
    torch.cuda.empty_cache()


class _Peak:
    """Allocator over PyTorch's that follows the bytes in use and refuses blocks for which
    ``refuse(nbytes)`` holds."""

    def __init__(self, refuse=None):
        self.live, self.now, self.peak, self.sizes = {}, 0, 0, []

        def alloc(ctx, nbytes, stream):
            if refuse and refuse(int(nbytes)):
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))
            self.live[int(p)] = int(nbytes)
            self.sizes.append(int(nbytes))
            self.now += int(nbytes)
            self.peak = max(self.peak, self.now)
            return p

        def free(ctx, ptr, stream):
            self.now -= self.live.pop(int(ptr))
            torch.cuda.caching_allocator_delete(int(ptr))

        self.struct = qsd.Allocator(None, qsd.ALLOC_FN(alloc), qsd.FREE_FN(free))


def _long_tails(words):
    """Three low parts, every high part of 16 qubits; every high qubit's flip has a term that wants a
    low qubit and ``words`` more on the high qubits, which a plan lists per high part."""
    terms = []
    for q in range(16, 32):
        terms += [(0.5 + 0.01 * q, [(q, wl.X)]), (0.25, [(0, wl.P1), (q, wl.X)])]
        others = [r for r in range(16, 32) if r != q]
        pairs = [(a, b, c) for a in others for b in others if a < b for c in others if b < c][:words]
        terms += [(0.125 + 0.001 * k, [(r, wl.Z) for r in w] + [(q, wl.X)]) for k, w in enumerate(pairs)]
    keys = (np.arange(1 << 16, dtype=np.uint64)[:, None] << np.uint64(16)) + np.array([1, 2, 5], dtype=np.uint64)
    return keys.reshape(-1, 1), wl.TermList.from_terms(32, terms)


@pytest.mark.parametrize("words,path", [(8, qsd.PATH_FACTORED), (200, qsd.PATH_PRODUCT_MAP)])
def test_plan_is_bounded(words, path):
    """Lists of 2.5 GB for a subspace of 196 608 strings are not made, and not asked for."""
    keys, tl = _long_tails(words)
    sub = qsd.Subspace(keys, 32)
    a = _Peak()
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl), allocator=a.struct)
    say("lists", words, H.spmv_path, max(a.sizes))
    assert H.spmv_path == path and a.peak < 1 << 30
    x = torch.randn(sub.N, dtype=torch.float64, device="cuda")
    y = H.matvec(x)
    H.schedule = DEFAULT | qsd.SCHED_HASH_LOOKUP
    assert torch.equal(H.matvec(x), y)
    del H


def test_plan_that_does_not_fit():
    """Every block of a plan that is larger than the operator's tables can be refused: the operator is
    bound all the same and runs from the product map."""
    w = wl.c3_molecular(1500, 60)
    sub = qsd.Subspace(w.keys, 32)
    op = qsd.operator_from_termlist(w.ops)
    a = _Peak()
    H = qsd.SubspaceHamiltonian(sub, op, allocator=a.struct)
    assert H.spmv_path == qsd.PATH_FACTORED
    x = torch.randn(sub.N, dtype=torch.float64, device="cuda")
    want = H.matvec(x)
    lists = max(a.sizes)
    say("blocks", a.sizes)
    b = _Peak(refuse=lambda n: n == lists)
    G = qsd.SubspaceHamiltonian(sub, op, allocator=b.struct)
    assert G.spmv_path == qsd.PATH_PRODUCT_MAP and max(b.sizes) < lists
    assert torch.equal(G.matvec(x), want)
    del G, H
    assert not a.live and not b.live


def test_element_list_that_does_not_fit():
    """The element list's memory is refused, the counts that come before it or the list itself: the
    slot-order schedules go by row bits, and a solve by the table."""
    keys, tl = CASES["sampled"]()
    sub = qsd.Subspace(keys, tl.n_qubits)
    op = qsd.operator_from_termlist(tl)
    H = qsd.SubspaceHamiltonian(sub, op)
    x = torch.randn(sub.N, dtype=torch.float64, device="cuda")
    want = H.matvec(x)
    solve = dict(tol=1e-9, max_iter=60, want_vector=True, raise_on_nonconv=False)
    energy = H.lanczos(**solve)
    log = _Peak()
    G = qsd.SubspaceHamiltonian(sub, op, allocator=log.struct)
    bound = len(log.sizes)
    G.schedule = qsd.SCHED_ALL
    assert G.spmv_path == qsd.PATH_ELEMENTS
    *_, counts, bits, sums, records = log.sizes[bound:]  # (sums: the scan's scratch)
    assert counts >= 8 * sub.N and bits >= sub.N / 8
    for size in (counts, sums, records):
        off = [False]
        a = _Peak(refuse=lambda n: n == size and off[0])
        G = qsd.SubspaceHamiltonian(sub, op, allocator=a.struct)
        off[0] = True
        e = G.lanczos(**solve)
        assert e[0] == energy[0] and torch.equal(e[1], energy[1])
        G.schedule = qsd.SCHED_ALL
        assert G.spmv_path == qsd.PATH_SLOTS_SPLIT
        assert torch.equal(G.matvec(x, out=torch.full_like(x, float("nan"))), want)
        del G
        assert not a.live


def test_element_list_of_2_to_28_rows():
    """An element in each of 2^28 rows and 16 vectors: rows times vectors are 2^32 lanes."""
    n = 1 << 28
    keys = torch.arange(n, dtype=torch.int64, device="cuda").reshape(-1, 1)
    sub = qsd.Subspace(keys, 40, max_load=0.5, assume_sorted_unique=True)
    del keys
    tl = wl.TermList.from_terms(40, [(0.75, [(0, wl.X)]), (0.5, [(3, wl.Z)])])
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
    H.schedule = qsd.SCHED_ALL
    assert H.spmv_path == qsd.PATH_ELEMENTS
    X = torch.randn((n, 16), dtype=torch.float32, device="cuda")
    Y = H.matvec(X, out=torch.full_like(X, float("nan")))
    for v in (0, 9, 15):
        assert torch.equal(H.matvec(X[:, v].contiguous()), Y[:, v])
    del X, Y, H, sub
    torch.cuda.empty_cache()


@pytest.mark.parametrize("entry", ["matvec_batched", "matvec_batched_noalloc"])
def test_batched_factored_workgroups(entry):
    """Requests of two low and 65 536 high parts beside one of 512 low parts, whose workgroups are the
    launch's: 2^23 workgroups of 512 threads and more."""
    terms = [(0.5, [(q, wl.X)]) for q in (0, 16, 24, 31)] + [(0.25 + 0.01 * q, [(q, wl.Z)]) for q in range(32)]
    tl = wl.TermList.from_terms(32, terms)
    op = qsd.operator_from_termlist(tl)
    hams = []
    for nlo, nhi in ((2, 1 << 16), (512, 2)):
        keys = (np.arange(nhi, dtype=np.uint64)[:, None] << np.uint64(16)) + np.arange(nlo, dtype=np.uint64)
        hams.append(qsd.SubspaceHamiltonian(qsd.Subspace(keys.reshape(-1, 1), 32), op))
        assert hams[-1].spmv_path == qsd.PATH_FACTORED
    hams = [hams[0]] * 32 + [hams[1]]
    xs = [torch.randn((h.N, 16), dtype=torch.float64, device="cuda") for h in hams]
    say("batched", entry)
    ys = getattr(qsd, entry)(hams, xs, [torch.full_like(x, float("nan")) for x in xs])
    for h, x, y in zip(hams, xs, ys):
        assert torch.equal(y, h.matvec(x))


@pytest.mark.parametrize("qubits,words", [(36, 1), (100, 2), (200, 4)])
def test_subspace_build_memory(qubits, words):
    """What a build holds at its peak: two buffers for the sort, and the subspace itself with the counts
    of its slot order."""
    n = 200_003
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    bits = torch.randint(0, 1 << 62, (n, words), dtype=torch.int64, device="cuda", generator=g)
    bits[:, -1] &= (1 << (qubits - 64 * (words - 1))) - 1
    bits[n // 2:] = bits[: n - n // 2].clone()  # duplicates
    a = _Peak()
    sub = qsd.Subspace(bits, qubits, allocator=a.struct)
    say("peak", sub.N, a.peak)
    assert sub.N <= n // 2 + 1
    own = sub.N * (8 * words + 8 + 4 + 8 * words + 8) + sub.capacity * 8 + sub.capacity // 8
    assert a.peak <= 2 * 8 * words * n + own + sub.capacity // 32 * 8 + (1 << 18)
    assert torch.equal(sub.lookup(sub.keys()), torch.arange(sub.N, device="cuda"))
    assert bool((sub.lookup(bits) >= 0).all())
    del sub
    assert not a.live


@pytest.mark.parametrize("build", ["to_csr", "lower_mirror"])
def test_csr_build_of_more_than_2_to_24_rows(build):
    """A workgroup per row sorts its entries: 2^24 rows of 256 threads are 2^32."""
    n = (1 << 24) + 300
    keys = torch.arange(n, dtype=torch.int64, device="cuda").reshape(-1, 1) * 2
    sub = qsd.Subspace(keys, 40, assume_sorted_unique=True)
    tl = wl.TermList.from_terms(40, [(0.75, [(1, wl.X)]), (0.25, [(2, wl.X)]), (0.5, [(3, wl.Z)])])
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
    if build == "to_csr":
        indptr, indices, data = H.to_csr()
    else:
        indptr, indices, data = qsd.CsrMatrix(H, qsd.INDEX_I64, lower_mirror=True).export()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), indptr[1:] - indptr[:-1])
    bits = (keys[indices, 0] ^ keys[rows, 0])
    assert torch.equal(torch.unique(bits), torch.tensor([0, 2, 4], device="cuda"))
    want = torch.where(bits == 2, 0.75, torch.where(bits == 4, 0.25, 0.5 - (keys[rows, 0] >> 3 & 1).double()))
    assert torch.equal(data, want)
    later = rows[1:] == rows[:-1]
    assert bool((indices[1:][later] > indices[:-1][later]).all())
    torch.cuda.empty_cache()


def test_refused_block_leaves_no_error():
    """An allocator that asks the runtime, and leaves the runtime's error behind: what is done without
    the block does not report it."""
    import ctypes

    runtime = ctypes.CDLL(qsd.LIB_PATH)  # (its hipMalloc is the one the library is bound to)
    w = wl.c3_molecular(1500, 60)
    sub = qsd.Subspace(w.keys, 32)
    op = qsd.operator_from_termlist(w.ops)
    a = _Peak()
    H = qsd.SubspaceHamiltonian(sub, op, allocator=a.struct)
    lists = max(a.sizes)

    def refuse(n):
        if n != lists:
            return False
        p = ctypes.c_void_p()
        assert runtime.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 55)) != 0
        return True

    b = _Peak(refuse=refuse)
    G = qsd.SubspaceHamiltonian(sub, op, allocator=b.struct)
    assert G.spmv_path == qsd.PATH_PRODUCT_MAP
    x = torch.randn(sub.N, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    G.matvec(x, out=y)
    assert torch.equal(H.matvec(x), y)
    del G, H
