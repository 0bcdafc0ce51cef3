"""GPU parity of the Lanczos iteration whose first update and second projection share one pass over
the basis, against the same iteration (two classical Gram-Schmidt passes) in torch FP64.

Both run the same number of steps from the same vector; the Ritz value then differs by rounding in
the steps, eps * |H| * steps (|H| < 4 per qubit, 260 steps: 1e-12 relative), so 1e-11 bounds it.
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


def _ritz(H, v, steps):
    V, alpha, beta = [v / v.norm()], [], []
    for _ in range(steps):
        w = H.matvec(V[-1])
        B = torch.stack(V)
        h = B @ w
        w -= h @ B
        g = B @ w
        w -= g @ B
        alpha.append(float(h[-1] + g[-1]))
        beta.append(float(w.norm()))
        V.append(w / beta[-1])
    return np.linalg.eigvalsh(np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1))[0]


# the fused form starts at 2M / rows vectors and at least 17, and takes up to 256: not reached, reached
# on the way and left again, from 17 on; rows that end a tile of 64, and that leave one row in the last
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n_qubits,rows,steps", [
    (12, 4096, 40), (14, 16384, 262), (14, 8193, 250), (17, 100001, 50), (17, 131072, 33)])
def test_ritz_value(n_qubits, rows, steps, graph):
    ops = wl.TermList.from_terms(
        n_qubits, [(-1.0, [(q, wl.Z), ((q + 1) % n_qubits, wl.Z)]) for q in range(n_qubits)]
        + [(-0.7 - 0.05 * q, [(q, wl.X)]) for q in range(n_qubits)], False)
    keys = np.arange(rows, dtype=np.uint64).reshape(-1, 1)
    H = qsd.SubspaceHamiltonian(qsd.Subspace(keys, n_qubits), qsd.operator_from_termlist(ops))
    x = torch.from_numpy(np.random.default_rng(rows).standard_normal(rows)).cuda()
    say("fused basis", n_qubits, rows, steps, graph)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):  # (the default stream cannot be captured)
        e = [H.lanczos(max_iter=steps, tol=1e-300, v0="user", v0_vector=x, use_graph=g, stream=stream,
                       raise_on_nonconv=False)[0] for g in {False, graph}]
    want = _ritz(H, x, steps)
    assert len(set(e)) == 1  # a captured iteration is the same to the bit
    assert abs(e[0] - want) <= 1e-11 * abs(want)
