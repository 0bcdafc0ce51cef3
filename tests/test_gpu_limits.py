"""Sizes at which a launch, a table or an allocation meets its limit: what was accepted there stays
accepted, and gives the results of the ordinary sizes."""
import numpy as np
import pytest

import workloads as wl

from _util import c2_keys, say

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
