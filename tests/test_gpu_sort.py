"""GPU parity of what a new subspace and operator are set up with: sorted, deduplicated keys and the
diagonal, exactly.

The keys are sorted by digits or by merging sorted tiles (4096 words of keys), whichever takes fewer
passes; the order of distinct keys is unique, so numpy's is the oracle.
"""
import numpy as np
import pytest

import workloads as wl

from _util import say

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def _check(bits, n_qubits):
    want = np.unique(bits[:, ::-1], axis=0)[:, ::-1]
    sub = qsd.Subspace(torch.from_numpy(bits.view(np.int64)).cuda(), n_qubits)
    got = sub.keys().cpu().numpy().view(np.uint64).reshape(-1, bits.shape[1])
    assert sub.N == want.shape[0]
    assert np.array_equal(got, want)


def _bits(n, n_qubits, seed=0):
    W = (n_qubits + 63) // 64
    b = np.random.default_rng(seed).integers(0, 1 << 64, (n, W), dtype=np.uint64)
    if n_qubits % 64:
        b[:, -1] &= np.uint64((1 << n_qubits % 64) - 1)
    return b


# one short of, at and past a tile, two tiles, and an odd number of runs at every level; keys of 1,
# 2, 3 (padded to 4), 5 and 16 words; few digits with many keys take the digit passes
@pytest.mark.parametrize("n_qubits,n", [
    (64, 1), (64, 2), (64, 257), (64, 4095), (64, 4096), (64, 4097), (64, 20481), (40, 300000), (20, 70000),
    (128, 2047), (128, 2049), (100, 10241), (192, 1025), (150, 5121), (200, 3 * 1024), (320, 513), (500, 2561),
    (1024, 255), (1000, 257), (1000, 1281)])
def test_sorted_unique(n_qubits, n):
    say("sort", n_qubits, n)
    _check(_bits(n, n_qubits), n_qubits)


@pytest.mark.parametrize("order", ["sorted", "reversed", "few", "equal", "low_word", "high_word"])
def test_sort_patterns(order):
    n_qubits, n = 200, 7000
    b = _bits(n, n_qubits, 1)
    if order in ("sorted", "reversed"):
        b = np.unique(b[:, ::-1], axis=0)[:, ::-1]
        if order == "reversed":
            b = b[::-1]
    elif order == "few":
        b = b[np.random.default_rng(2).integers(0, 9, n)]
    elif order == "equal":
        b[:] = b[0]
    elif order == "low_word":
        b[:, 1:] = b[0, 1:]
    else:
        b[:, :-1] = b[0, :-1]
    say("sort", order)
    _check(np.ascontiguousarray(b), n_qubits)


# the diagonal's runs: masks in one or two 32-bit words of the key, in the same words for any number of
# terms, in more words, with projectors, and of a complex operator
@pytest.mark.parametrize("n_qubits,kinds,seed", [
    (12, "zz", 0), (40, "zz", 1), (40, "n", 2), (64, "zzzz", 3), (100, "zz n zzzz identity", 4), (200, "zz", 5),
    (200, "zz n zzzz", 6), (500, "zz n", 7), (100, "zz n complex", 8)])
def test_diagonal_exact(n_qubits, kinds, seed):
    rng = np.random.default_rng(seed)
    terms = []
    for k in kinds.split():
        for j in range(37):
            c = float(rng.integers(-64, 65)) / 16 or 0.25
            if k == "zz":  # neighbours: many terms in the same words
                q = int(rng.integers(0, n_qubits - 1))
                terms.append((c, [(q, wl.Z), (q + 1, wl.Z)][: 1 + j % 2]))
            elif k == "zzzz":
                terms.append((c, [(int(q), wl.Z) for q in sorted(rng.choice(n_qubits, 4, replace=False))]))
            elif k == "n":
                qs = sorted(rng.choice(n_qubits, 1 + j % 3, replace=False))
                terms.append((c, [(int(q), (wl.P1, wl.P0, wl.Z)[(i + j) % 3]) for i, q in enumerate(qs)]))
            elif k == "identity":
                terms.append((c, []))
                break
            else:
                terms.append((1j * c, [(j, wl.RAISE), (j + 1, wl.LOWER)]))
    ops = wl.TermList.from_terms(n_qubits, terms, False)
    b = np.unique(_bits(3000, n_qubits, seed)[:, ::-1], axis=0)[:, ::-1]
    H = qsd.SubspaceHamiltonian(qsd.Subspace(torch.from_numpy(b.copy().view(np.int64)).cuda(), n_qubits),
                                qsd.operator_from_termlist(ops))
    got = H.diagonal().cpu().numpy()
    want = np.zeros(len(b))
    for c, word in terms:
        if isinstance(c, complex):
            continue
        v = np.full(len(b), c)
        for q, code in word:
            bit = (b[:, q // 64] >> np.uint64(q % 64)) & np.uint64(1)
            v *= {wl.Z: 1 - 2 * bit.astype(np.int64), wl.P1: bit.astype(np.int64),
                  wl.P0: 1 - bit.astype(np.int64)}[code]
        want += v
    say("diagonal", n_qubits, kinds)
    assert np.array_equal(got, want)
