"""Which kernels an operator's SpMV takes.

The factored lists, the element list, the product map and the row engine give bitwise the same
results, so a comparison of results does not show that the one that was meant ran; these tests do.
"""
import itertools

import numpy as np
import pytest

import workloads as wl

from _util import c2_keys, c3_parts, heavy_hex_small, say
from test_gpu_factored import _edited
from test_gpu_hits import CASES, _chain_keys

torch = pytest.importorskip("torch")
qsd = pytest.importorskip("paper_2603_18731_amd")

pytestmark = pytest.mark.gpu

DEFAULT = qsd.SCHED_XCD_REMAP | qsd.SCHED_FILTER_FIRST
C, A = wl.F_CRE, wl.F_ANN


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qsd.lib()


def _ham(keys, tl, **kw):
    return qsd.SubspaceHamiltonian(qsd.Subspace(keys, tl.n_qubits), qsd.operator_from_termlist(tl, **kw))


@pytest.mark.parametrize("na,nb", [(1, 70), (70, 1), (2, 2), (64, 64), (257, 5), (513, 3), (1500, 3), (4368, 2)])
def test_molecular_is_factored(na, nb):
    w = wl.c3_molecular(na, nb)
    H = _ham(w.keys, w.ops)
    assert H.spmv_path == qsd.PATH_FACTORED
    H.schedule = DEFAULT | qsd.SCHED_HASH_LOOKUP
    assert H.spmv_path == qsd.PATH_ROWS
    assert _ham(w.keys, w.ops, order_by_parts=False).spmv_path == qsd.PATH_PRODUCT_MAP


def _variants():
    ops, _ = c3_parts(37, 29)
    drop = np.random.default_rng(5).random(ops.n_terms) < 0.3
    three = [(0.3, [(0, C), (3, A), (17, C), (17, A), (18, C), (18, A)]),
             (0.3, [(3, C), (0, A), (17, C), (17, A), (18, C), (18, A)])]
    return {
        "absent_pairs": (_edited(ops, lambda k, t: len(t[1]) == 2 or not drop[k]), qsd.PATH_FACTORED),
        "one_body": (_edited(ops, lambda k, t: len(t[1]) == 2), qsd.PATH_FACTORED),
        # a term that wants two qubits of the other part
        "three_body": (_edited(ops, None, three), qsd.PATH_PRODUCT_MAP),
        # an element whose coefficient is complex
        "complex": (_edited(wl.TermList.from_terms(32, [], True), None,
                            [(0.5j, [(0, C), (3, A)]), (-0.5j, [(3, C), (0, A)])]), qsd.PATH_PRODUCT_MAP),
    }


@pytest.mark.parametrize("name", ["absent_pairs", "one_body", "three_body", "complex"])
def test_molecular_variants(name):
    tl, path = _variants()[name]
    assert _ham(c3_parts(37, 29)[1], tl).spmv_path == path


def test_spin_chains():
    assert _ham(wl.full_space(12), wl.tfim_chain(12)).spmv_path == qsd.PATH_FACTORED
    # a sector of fixed magnetization is no product, and has several elements per row
    keys = np.array([sum(1 << q for q in c) for c in itertools.combinations(range(12), 6)], dtype=np.uint64)
    H = _ham(keys.reshape(-1, 1), wl.xxz_terms(12, [(q, q + 1) for q in range(11)], 1.0, 0.5))
    assert H.spmv_path == qsd.PATH_ROWS
    H.schedule = qsd.SCHED_ALL
    assert H.spmv_path == qsd.PATH_SLOTS_SPLIT


def test_rehash_moves_the_path():
    ops, keys = c3_parts(60, 45)
    sub = qsd.Subspace(keys, 32)
    op = qsd.operator_from_termlist(ops)
    H = qsd.SubspaceHamiltonian(sub, op)
    for load, split, path in ((0.25, 0, qsd.PATH_ROWS), (0.5, 20, qsd.PATH_ROWS), (0.03125, 16, qsd.PATH_FACTORED)):
        sub.rehash(load, split)
        assert H.spmv_path == path, split
    sub.rehash(0.125, 0)
    G = qsd.SubspaceHamiltonian(sub, op)  # bound while there is no product map: no lists
    sub.rehash(0.125, 16)
    assert G.spmv_path == qsd.PATH_PRODUCT_MAP and H.spmv_path == qsd.PATH_FACTORED


@pytest.mark.parametrize("name", ["none", "few", "edge", "sampled", "long_rows", "wide", "one_row"])
def test_sparse_operators_take_the_list(name):
    keys, tl = CASES[name]()
    H = _ham(keys, tl)
    say("path", name, H.N, H.spmv_path)
    H.schedule = DEFAULT
    assert H.spmv_path == qsd.PATH_ROWS
    H.schedule = qsd.SCHED_SLOT_ORDER
    assert H.spmv_path == qsd.PATH_ELEMENTS
    H.autotune(reps=1, load=False)
    assert H.spmv_path == (qsd.PATH_ELEMENTS if H.schedule & qsd.SCHED_SLOT_ORDER else qsd.PATH_ROWS)


def test_unset_schedule_samples():
    H = _ham(_chain_keys(20_001, 2_500), wl.xxz_terms(40, [(0, 1), (7, 31)], 1.0, 0.5))
    assert H.spmv_path == qsd.PATH_SLOTS and H.schedule == DEFAULT
    H.schedule = DEFAULT
    assert H.spmv_path == qsd.PATH_ROWS
    H = _ham(np.arange(6000, dtype=np.uint64).reshape(-1, 1), wl.tfim_chain(40))
    assert H.spmv_path == qsd.PATH_ROWS


@pytest.mark.parametrize("name", ["few", "sampled", "wide"])
def test_slot_order_through_the_table_is_split(name):
    """A sparse operator under SLOT_ORDER | HASH_LOOKUP, which the element list does not serve: the
    rows without elements are still written apart (the list holds the bits that say which)."""
    keys, tl = CASES[name]()
    H = _ham(keys, tl)
    x = torch.randn((H.N, 3), dtype=torch.float64, device="cuda")
    H.schedule = DEFAULT | qsd.SCHED_HASH_LOOKUP
    want = H.matvec(x)
    for extra in (0, qsd.SCHED_XCD_REMAP, qsd.SCHED_LOCKSTEP, qsd.SCHED_FILTER_FIRST):
        H.schedule = qsd.SCHED_SLOT_ORDER | qsd.SCHED_HASH_LOOKUP | extra
        assert H.spmv_path == qsd.PATH_SLOTS_SPLIT
        assert torch.equal(H.matvec(x, out=torch.full_like(x, float("nan"))), want)


def test_dense_solve_makes_no_count():
    """A solve asks a sample whether a list pays before it counts the elements of all rows, which takes
    as long as an SpMV: a dense operator of many groups takes no more memory than its basis."""
    ops, keys = c3_parts(60, 60)
    sizes = []

    def alloc(ctx, nbytes, stream):
        sizes.append(int(nbytes))
        return torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))

    a = qsd.Allocator(None, qsd.ALLOC_FN(alloc), qsd.FREE_FN(lambda c, p, s: torch.cuda.caching_allocator_delete(int(p))))
    H = qsd.SubspaceHamiltonian(qsd.Subspace(keys, 32), qsd.operator_from_termlist(ops, order_by_parts=False),
                                allocator=a)
    assert H.spmv_path == qsd.PATH_PRODUCT_MAP
    del sizes[:]
    H.lanczos(tol=1e-9, max_iter=60, raise_on_nonconv=False)
    say("solve", H.N, sizes)
    assert max(sizes) >= 60 * 8 * H.N and all(n < 8 * H.N for n in sizes if n != max(sizes))
    del H


@pytest.mark.parametrize("schedule", [True, False])
def test_autotune_keeps_the_table_of_a_list(schedule):
    """An SpMV from the element list reads no table, so the autotuner does not choose one by chance."""
    keys, tl = CASES["sampled"]()
    H = _ham(keys, tl)
    H.schedule = qsd.SCHED_ALL
    before = H.subspace.capacity
    r = H.autotune(reps=1, schedule=schedule, load=True, split=True)
    say("tuned", r)
    assert H.spmv_path == qsd.PATH_ELEMENTS and np.isfinite(r["ms"]) and r["ms"] > 0
    assert H.subspace.capacity == before == r["capacity"] and r["split"] == 0 and r["max_load"] == 0.125
