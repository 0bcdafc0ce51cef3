"""A batched SpMV in a captured graph: every replay is the eager call on what x holds then, also after the
call that was captured has long returned and its host memory has been used for something else."""
import numpy as np
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


def _ham(keys, tl, **kw):
    return qsd.SubspaceHamiltonian(qsd.Subspace(keys, tl.n_qubits), qsd.operator_from_termlist(tl, **kw))


# a table of one piece and of many (tiles of some 200 000 rows), factored and other requests
@pytest.mark.parametrize("rows", [700, 200_000])
def test_noalloc_replays(rows):
    ops, keys = c3_parts(40, 30)
    hams = [_ham(keys, ops), _ham(c2_keys(rows), wl.xxz_grid_6x6()), _ham(keys, ops, order_by_parts=False),
            _ham(wl.full_space(9), wl.tfim_chain(9))]
    xs = [torch.randn((h.N, 3), dtype=torch.float64, device="cuda") for h in hams]
    ys = [torch.empty_like(x) for x in xs]
    qsd.matvec_batched_noalloc(hams, xs, ys)  # (resolves the library's scratch)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        qsd.matvec_batched_noalloc(hams, xs, ys)
    junk = [np.full(n, 255, dtype=np.uint8) for n in (4096, 65536, 1 << 20, 1 << 22)]
    for k in range(4):
        for x, y in zip(xs, ys):
            x.copy_(torch.randn_like(x))
            y.fill_(float("nan"))
        want = [h.matvec(x) for h, x in zip(hams, xs)]
        other = qsd.matvec_batched_noalloc(hams[::-1], xs[::-1], [torch.empty_like(x) for x in xs[::-1]])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        say("replay", rows, k, len(junk))
        for y, w, o in zip(ys, want, other[::-1]):
            assert torch.equal(y, w) and torch.equal(o, w)
