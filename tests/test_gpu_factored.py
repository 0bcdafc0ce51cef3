"""GPU parity of the factored SpMV on alpha x beta product subspaces.

An operator whose groups keep their classes apart (low part only, both, high part only) runs from
lists worked out once per part; any other runs from the product map.  Every element is the same
sum of the same terms and every row takes its elements in the same order, so the results are
bitwise those of the hash-table path (QSD_SCHED_HASH_LOOKUP) for any coefficients, and the
oracle's for dyadic ones: no tolerance.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import rowwise as orw
from oracle import subspace as osub

from _util import c3_parts, dyadic, dyadic_vector, say

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu

DEFAULT = qsd.SCHED_XCD_REMAP | qsd.SCHED_FILTER_FIRST


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def _same_as_table(H, x):
    """The default path against the table path, bitwise; rows that no lane writes stay NaN."""
    y = torch.full_like(x, float("nan"))
    H.schedule = DEFAULT
    H.matvec(x, out=y)
    z = torch.full_like(x, float("nan"))
    H.schedule = DEFAULT | qsd.SCHED_HASH_LOOKUP
    H.matvec(x, out=z)
    H.schedule = DEFAULT
    assert not torch.isnan(z).any()
    assert torch.equal(y, z)
    return y


def _vec(N, nvec, dtype, seed=0):
    x = np.random.default_rng(seed).standard_normal((N, nvec) if nvec > 1 else N)
    return torch.from_numpy(x).to(dtype).cuda()


# tiles of 256 low parts: one short of, at and past the edge; single parts; every width of the
# vector chunks (1, 2, 4) with full and partial last chunks; sizes whose LDS row forces the
# narrower chunks (1500 and 2500 strings)
@pytest.mark.parametrize("na,nb,nvec,dtype", [
    (255, 5, 1, torch.float64), (256, 5, 2, torch.float64), (257, 5, 3, torch.float64), (257, 5, 16, torch.float32),
    (1, 70, 5, torch.float64), (70, 1, 4, torch.float32), (2, 2, 1, torch.float64), (64, 64, 8, torch.float64),
    (1500, 3, 4, torch.float64), (2500, 3, 2, torch.float64), (4368, 2, 1, torch.float64), (2500, 3, 4, torch.float32)])
def test_molecular_bitwise(na, nb, nvec, dtype):
    if na > 1 and nb > 1:
        ops, keys = c3_parts(na, nb)
    else:
        w = wl.c3_molecular(na, nb)
        ops, keys = w.ops, w.keys
    sub = qsd.Subspace(keys, ops.n_qubits)
    assert sub.hash_info()[2]
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    say("factored", na, nb, nvec, dtype)
    _same_as_table(H, _vec(sub.N, nvec, dtype))


# tiles of up to 512 low parts of one size: one short of, at and past the edges, a last tile that is
# nearly empty and one that ends inside a wave
@pytest.mark.parametrize("na,nb,nvec,dtype", [
    (63, 3, 1, torch.float64), (65, 3, 1, torch.float32), (511, 3, 1, torch.float64), (512, 2, 1, torch.float64),
    (513, 3, 1, torch.float64), (513, 3, 7, torch.float32), (1025, 2, 1, torch.float64), (1537, 2, 2, torch.float64)])
def test_tiles_bitwise(na, nb, nvec, dtype):
    ops, keys = c3_parts(na, nb)
    sub = qsd.Subspace(keys, ops.n_qubits)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    say("factored tiles", na, nb, nvec, dtype)
    _same_as_table(H, _vec(sub.N, nvec, dtype))


# whole groups of vectors are read at once where x, y and their row stride are aligned: aligned, one
# element off in x, in y or in both, a stride that is no multiple of 16 bytes, and a short last group
@pytest.mark.parametrize("nvec,dtype", [(2, torch.float64), (4, torch.float64), (6, torch.float64), (8, torch.float64),
                                        (2, torch.float32), (4, torch.float32), (6, torch.float32)])
def test_alignment_bitwise(nvec, dtype):
    ops, keys = c3_parts(130, 9)
    sub = qsd.Subspace(keys, ops.n_qubits)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    x = _vec(sub.N, nvec, dtype)
    say("factored alignment", nvec, dtype)
    want = _same_as_table(H, x)
    n = x.numel()
    for ox, oy in ((1, 0), (0, 1), (1, 1), (2, 2)):
        xs = torch.zeros(n + 4, dtype=dtype, device="cuda")[ox:ox + n].view_as(x).copy_(x)
        ys = torch.full((n + 4,), float("nan"), dtype=dtype, device="cuda")
        y = ys[oy:oy + n].view_as(x)
        H.matvec(xs, out=y)
        assert torch.equal(y, want)
        assert int(torch.isnan(ys).sum()) == 4  # nothing beside y


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_stays_in_its_rows(value):
    """The entries that fill up the lists add 0 * 0: a value of x that is not finite reaches the rows
    that have an element there and no other."""
    ops, keys = c3_parts(130, 9)
    sub = qsd.Subspace(keys, ops.n_qubits)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    x = _vec(sub.N, 1, torch.float64)
    x[130 * 4 + 7] = value
    y = H.matvec(x)
    H.schedule = DEFAULT | qsd.SCHED_HASH_LOOKUP
    z = H.matvec(x)
    bad = ~torch.isfinite(z)
    assert 0 < int(bad.sum()) < sub.N
    assert torch.equal(bad, ~torch.isfinite(y)) and torch.equal(y[~bad], z[~bad])


def _edited(ops, keep=None, extra=()):
    terms = [t for k, t in enumerate(ops.terms()) if keep is None or keep(k, t)]
    return wl.TermList.from_terms(ops.n_qubits, terms + list(extra), ops.fermionic)


C, A = wl.F_CRE, wl.F_ANN


@pytest.mark.parametrize("name", ["absent_pairs", "no_one_body", "one_body", "zero_coefficient", "three_body"])
def test_molecular_variants(name):
    """Operators at the edges of the rule: pairs of single excitations without a term, single
    excitations without their spectator-free term, no two-body part, a term whose coefficient
    cancels, a term with two spectators."""
    ops, keys = c3_parts(37, 29)
    rng = np.random.default_rng(5)
    drop = rng.random(ops.n_terms) < 0.3
    if name == "absent_pairs":
        tl = _edited(ops, lambda k, t: len(t[1]) == 2 or not drop[k])
    elif name == "no_one_body":
        tl = _edited(ops, lambda k, t: len(t[1]) == 4)
    elif name == "one_body":
        tl = _edited(ops, lambda k, t: len(t[1]) == 2)
    elif name == "zero_coefficient":
        # the same alpha x beta double excitation written in another order, cancelling
        tl = _edited(wl.TermList.from_terms(32, [], True), None, [
            (0.5, [(1, C), (20, C), (22, A), (3, A)]), (-0.5, [(20, C), (1, C), (3, A), (22, A)]),
            (0.25, [(2, C), (20, C), (22, A), (3, A)]), (0.75, [(0, C), (3, A)]), (0.5, [(17, C), (22, A)])])
    else:
        tl = _edited(ops, None, [(0.3, [(0, C), (3, A), (17, C), (17, A), (18, C), (18, A)]),
                                 (0.3, [(3, C), (0, A), (17, C), (17, A), (18, C), (18, A)])])
    tl = dyadic(tl) if name != "zero_coefficient" else tl
    sub = qsd.Subspace(keys, 32)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
    X = dyadic_vector(rng, sub.N, nvec=3)
    say("variant", name, tl.n_terms)
    y = _same_as_table(H, torch.from_numpy(X).cuda())
    np.testing.assert_array_equal(y.cpu().numpy(), orw.matvec_c(osub.canonical_keys(keys), tl, X).real)


@pytest.mark.parametrize("n,order", [(12, {}), (12, {"order_by_parts": True}), (7, {"order_by_parts": True}),
                                     (7, {"ladder_ints": False, "order_by_parts": True})])
def test_qubit_words_bitwise(n, order):
    """Random words over the whole real alphabet on a full space (a product of its halves, of
    unequal widths for 7 qubits): whatever path the rule picks equals the table's."""
    rng = np.random.default_rng(n)
    letters = (0, 1, 2, 3, 5, 6)
    for trial in range(4):
        terms = [(1.0, [(q, 3)]) for q in range(n)] if trial == 0 else []
        for _ in range(40):
            qs = rng.choice(n, size=int(rng.integers(1, 5)), replace=False)
            terms.append((float(rng.standard_normal()), [(int(q), int(rng.choice(letters))) for q in qs]))
        keys = wl.full_space(n)
        sub = qsd.Subspace(keys, n)
        H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(wl.TermList.from_terms(n, terms), **order))
        say("words", n, order, trial)
        _same_as_table(H, _vec(sub.N, 1, torch.float64, trial))
    tl = wl.tfim_chain(n)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl, **order))
    _same_as_table(H, _vec(sub.N, 2, torch.float32))


def test_non_finite_and_strided_vectors():
    """Infinities and NaN reach only the rows that have an element there, and a leading dimension
    beyond the vector count (with an unaligned first column) is read as the table path reads it."""
    ops, keys = c3_parts(70, 40)
    rng = np.random.default_rng(8)
    drop = rng.random(ops.n_terms) < 0.3
    for tl in (ops, _edited(ops, lambda k, t: len(t[1]) == 2 or not drop[k])):
        sub = qsd.Subspace(keys, 32)
        H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
        x = _vec(sub.N, 1, torch.float64, 3)
        x[17], x[1200] = float("inf"), float("nan")
        outs = []
        for s in (DEFAULT, DEFAULT | qsd.SCHED_HASH_LOOKUP):
            H.schedule = s
            outs.append(H.matvec(x))
        assert torch.equal(outs[0].isnan(), outs[1].isnan())
        ok = ~outs[0].isnan()
        assert torch.equal(outs[0][ok], outs[1][ok]) and int(ok.sum()) < sub.N
        big = _vec(sub.N, 7, torch.float64, 4)
        got = []
        for s in (DEFAULT, DEFAULT | qsd.SCHED_HASH_LOOKUP):
            H.schedule = s
            y = torch.full((sub.N, 9), 5.0, dtype=torch.float64, device="cuda")
            H.matvec_raw(3, big.data_ptr() + 8, 7, y.data_ptr() + 16, 9, qsd.F64)
            got.append(y)
        assert torch.equal(*got) and bool((got[0][:, :2] == 5.0).all()) and bool((got[0][:, 5:] == 5.0).all())


def test_rehash_keeps_the_results():
    """The plan follows the split it was built for: another split or none runs without it, the
    same split at another load runs with it, and an operator bound while there was none too."""
    ops, keys = c3_parts(60, 45)
    sub = qsd.Subspace(keys, 32)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    x = _vec(sub.N, 1, torch.float64)
    want = H.matvec(x)
    for load, split in ((0.25, 0), (0.5, 5), (0.03125, 16)):
        sub.rehash(load, split)
        assert torch.equal(H.matvec(x), want)
        G = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
        assert torch.equal(G.matvec(x), want)
    sub.rehash(0.125, 0)
    G = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(ops))
    sub.rehash(0.125, 16)
    assert torch.equal(G.matvec(x), want)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_batched_mix(dtype):
    """Factored requests beside product-map (group order by weight), table and non-product ones
    in one batched call and in one Lanczos batch: bitwise the single calls' results."""
    hams = []
    for na, nb, kw in ((257, 3, {}), (40, 40, {}), (40, 40, {"order_by_parts": False}), (1, 30, {}), (1200, 2, {})):
        ops, keys = c3_parts(na, nb) if na > 1 else (lambda w: (w.ops, w.keys))(wl.c3_molecular(na, nb))
        hams.append(qsd.SubspaceHamiltonian(qsd.Subspace(keys, 32), qsd.operator_from_termlist(ops, **kw)))
    hams.append(qsd.SubspaceHamiltonian(hams[1].subspace, hams[1].op))
    hams[-1].schedule |= qsd.SCHED_HASH_LOOKUP
    hams.append(qsd.SubspaceHamiltonian(qsd.Subspace(wl.full_space(9), 9), qsd.operator_from_termlist(wl.tfim_chain(9))))
    nvecs = [1, 5, 2, 16, 3, 1, 1]
    xs = [_vec(h.N, nv, dtype, k) for k, (h, nv) in enumerate(zip(hams, nvecs))]
    say("batched mix", dtype)
    for entry in (qsd.matvec_batched, qsd.matvec_batched_noalloc):
        ys = entry(hams, xs, [torch.full_like(x, float("nan")) for x in xs])
        for h, x, y in zip(hams, xs, ys):
            assert torch.equal(y, h.matvec(x))
    b = qsd.LanczosBatch(8, max_iter=60, spmv_dtype="f64" if dtype == torch.float64 else "f32")
    one = qsd.LanczosBatch(8, max_iter=60, spmv_dtype="f64" if dtype == torch.float64 else "f32")
    slots = [b.add(h, v0="random", seed=k) for k, h in enumerate(hams)]
    b.step(12)
    st, e, it, rr = b.poll()
    for k, h in enumerate(hams):
        s = one.add(h, v0="random", seed=k)
        one.step(12)
        _, e1, it1, rr1 = one.poll()
        assert (e1[s], it1[s], rr1[s]) == (e[slots[k]], it[slots[k]], rr[slots[k]])
        one.remove(s)
    assert e[slots[1]] == e[slots[1]] and st[slots[1]] != 0


@pytest.mark.parametrize("na,nb", [(257, 7), (40, 40), (1, 60), (60, 1), (513, 3)])
@pytest.mark.parametrize("index,dtype", [(qsd.INDEX_I32, torch.float64), (qsd.INDEX_I64, torch.float32)])
def test_csr_bitwise(na, nb, index, dtype):
    """The CSR build from the lists against the row engine's (structure and values bitwise), with
    every pair of keys present and with pairs missing, and on a spin chain."""
    if na > 1 and nb > 1:
        ops, keys = c3_parts(na, nb)
    else:
        w = wl.c3_molecular(na, nb)
        ops, keys = w.ops, w.keys
    drop = np.random.default_rng(6).random(ops.n_terms) < 0.3
    cases = [(ops, keys), (_edited(ops, lambda k, t: len(t[1]) == 2 or not drop[k]), keys)]
    if na == nb:
        cases.append((wl.tfim_chain(11), wl.full_space(11)))
    for tl, ks in cases:
        sub = qsd.Subspace(ks, tl.n_qubits)
        assert sub.hash_info()[2]
        H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(tl))
        say("factored CSR", na, nb, tl.n_terms, index, dtype)
        H.schedule = DEFAULT | qsd.SCHED_HASH_LOOKUP
        want = H.to_csr(index, dtype)
        H.schedule = DEFAULT
        got = H.to_csr(index, dtype)
        for g, w_ in zip(got, want):
            assert torch.equal(g, w_)
        A = qsd.CsrMatrix(H, index, dtype)
        for g, w_ in zip(A.export(), want):
            assert torch.equal(g, w_)
