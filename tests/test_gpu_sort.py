"""GPU parity of the canonical order of a subspace: sorted, deduplicated keys, exactly.

The keys are sorted by digits or by merging sorted tiles (4096 words of keys), whichever takes fewer
passes; the order of distinct keys is unique, so numpy's is the oracle.
"""
import numpy as np
import pytest

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
