"""Performance cases of the subspace-Hamiltonian library: what a program that uses it waits for.

The entry points are the binding's: ``SubspaceHamiltonian.matvec`` (matrix-free SpMV / SpMM, the
hot path), ``CsrMatrix.matvec`` and ``to_csr`` (the stored alternative), ``lanczos`` (a whole
ground-state solve), ``matvec_batched`` (serving) and the set-up of a new sample
(``Subspace`` + ``SubspaceHamiltonian``).  Models are the repository's workloads: TFIM-12, XXZ on
the 6x6 grid, the 200-qubit heavy-hex model and the 16-orbital molecular Hamiltonian on
alpha x beta product subspaces.

A case is a dict: ``op`` (the entry point), ``model``, its size (``n`` distinct samples, or ``na`` x ``nb``
alpha and beta strings), ``nvec``, ``dtype`` and ``tuned`` (hash load and schedule set to what the
autotuner keeps on the sparse models, as a program that tuned once does; otherwise the defaults).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_18731_amd as qsd
import workloads as wl

NORB, NEL = 16, 5                          # molecular model: orbitals, electrons per spin
N_STRINGS = math.comb(NORB, NEL)           # 4368 strings of one spin
DTYPES = {"f64": torch.float64, "f32": torch.float32}


# ------------------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: one SpMV on a few thousand states, all latency
        dict(name="tfim_matvec", op="matvec", model="tfim", n=4096, nvec=1, dtype="f64", tuned=False),
        # the smallest solve: every launch and host round trip of an iteration counts
        dict(name="tfim_solve", op="lanczos", model="tfim", n=4096, nvec=1, dtype="f64", tuned=False),
        # spin model on samples of a symmetry sector, tuned once and applied many times
        dict(name="xxz_matvec", op="matvec", model="xxz", n=1 << 20, nvec=1, dtype="f64", tuned=True),
        # wide strings (four key words), eight vectors at once (block eigensolvers)
        dict(name="hex_spmm8", op="matvec", model="hex", n=3_000_000, nvec=8, dtype="f64", tuned=True),
        # chemistry: the largest product subspace a benchmark of the repository uses
        dict(name="fermi_matvec_1500", op="matvec", model="fermi", na=1500, nb=1500, nvec=1, dtype="f64", tuned=False),
        # an ordinary, ragged product subspace in single precision
        dict(name="fermi_matvec_337x411_f32", op="matvec", model="fermi", na=337, nb=411, nvec=1, dtype="f32",
             tuned=False),
        # block solves on a product subspace: eight vectors
        dict(name="fermi_spmm8_300", op="matvec", model="fermi", na=300, nb=300, nvec=8, dtype="f64", tuned=False),
        # the stored matrix, applied many times by an eigensolver
        dict(name="fermi_csr_matvec_600", op="csr_matvec", model="fermi", na=600, nb=600, nvec=1, dtype="f64",
             tuned=False),
        # building that matrix once for a sample
        dict(name="fermi_csr_build_301", op="csr_build", model="fermi", na=301, nb=301, nvec=1, dtype="f64",
             tuned=False),
        # a whole ground-state solve with its vector, orthogonalization against a long basis
        dict(name="hex_solve", op="lanczos", model="hex", n=700_000, nvec=1, dtype="f64", tuned=False),
        # serving: two dozen independent operators in one call
        dict(name="batched_24", op="batched", model="mixed", n=24, nvec=1, dtype="f64", tuned=False),
        # a new sample: sort, deduplicate, hash, bind the operator, diagonal
        dict(name="hex_setup", op="setup", model="hex", n=1_000_000, nvec=1, dtype="f64", tuned=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["matvec"] * 5 + ["csr_matvec", "csr_build", "lanczos", "batched", "setup"])
    if op == "matvec":
        model = rng.choice(["xxz", "hex", "fermi", "fermi"])
        nvec = rng.choice([1, 1, 2, 3, 4, 8, 16])
        dtype = rng.choice(["f64", "f64", "f32"])
        if model == "fermi":
            most = 1500 if nvec == 1 else 420
            return dict(op=op, model=model, na=_log_int(rng, 24, most), nb=_log_int(rng, 24, most), nvec=nvec,
                        dtype=dtype, tuned=False)
        return dict(op=op, model=model, n=_log_int(rng, 3_000, 1_000_000), nvec=nvec, dtype=dtype,
                    tuned=rng.random() < 0.5)
    if op == "csr_matvec":
        return dict(op=op, model="fermi", na=_log_int(rng, 40, 600), nb=_log_int(rng, 40, 600), nvec=rng.choice([1, 1, 4]),
                    dtype=rng.choice(["f64", "f32"]), tuned=False)
    if op == "csr_build":
        return dict(op=op, model="fermi", na=_log_int(rng, 40, 301), nb=_log_int(rng, 40, 301), nvec=1,
                    dtype=rng.choice(["f64", "f32"]), tuned=False)
    if op == "lanczos":
        return dict(op=op, model=rng.choice(["xxz", "hex"]), n=_log_int(rng, 5_000, 400_000), nvec=1, dtype="f64",
                    tuned=False)
    if op == "batched":
        return dict(op=op, model="mixed", n=rng.randint(4, 24), nvec=1, dtype=rng.choice(["f64", "f32"]), tuned=False)
    return dict(op=op, model=rng.choice(["xxz", "hex"]), n=_log_int(rng, 10_000, 1_000_000), nvec=1, dtype="f64",
                tuned=False)


# ---------------------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _bit(q):
    """The int64 whose bit ``q`` is set (bit 63 is the sign)."""
    return (1 << q) if q < 63 else -(1 << 63)


def _pick(rows, n, g):
    """``n`` distinct rows of ``rows`` [m][W] in random order (equal rows have equal images)."""
    odd = (0x9E3779B97F4A7C15, 0xC2B2AE3D27D4EB4F, 0x165667B19E3779F9, 0x27D4EB2F165667C5)
    image = torch.zeros(rows.shape[0], dtype=torch.int64, device="cuda")
    for w in range(rows.shape[1]):
        image = (image ^ (rows[:, w] * (odd[w] - (1 << 64) if odd[w] >> 63 else odd[w]))) * 31
    srt, perm = torch.sort(image)
    first = torch.ones_like(srt, dtype=torch.bool)
    first[1:] = srt[1:] != srt[:-1]
    once = perm[first]
    assert once.numel() >= n
    return rows[once[torch.randperm(once.numel(), generator=g, device="cuda")[:n]]]


def _xxz_bits(n, g):
    """``n`` distinct weight-18 strings of 36 bits."""
    out, m = [], n + n // 64 + 64
    for a in range(0, m, 1 << 18):
        sel = torch.rand((min(1 << 18, m - a), 36), generator=g, device="cuda").argsort(1)[:, :18]
        out.append((torch.ones_like(sel) << sel).sum(1))
    return _pick(torch.cat(out).reshape(-1, 1), n, g)


def _hex_bits(n, g):
    """``n`` distinct strings: the two-colouring with up to six flips, [n][4] words."""
    nq, edges = wl.heavy_hex_200()
    ref = np.zeros(4, dtype=np.uint64)
    for q in np.nonzero(wl.two_colouring(nq, edges) == 1)[0]:
        ref[q // 64] |= np.uint64(1) << np.uint64(q % 64)
    m = 2 * n + 1024
    keys = torch.from_numpy(ref.view(np.int64)).cuda().repeat(m, 1)
    k = torch.randint(1, 7, (m,), generator=g, device="cuda")
    pos = torch.randint(0, nq, (m, 6), generator=g, device="cuda")
    for j in range(6):
        on = k > j
        for i in range(j):
            on = on & (pos[:, i] != pos[:, j])
        bit = torch.ones_like(pos[:, j]) << (pos[:, j] % 64)
        for w in range(4):
            keys[:, w] ^= torch.where(on & (pos[:, j] // 64 == w), bit, torch.zeros_like(bit))
    return _pick(keys, n, g)


def _fermi_strings(case, seed):
    """Sampled alpha and beta strings.  A matrix that is returned keeps its sample from seed to
    seed (the integrals change), so that it has one size."""
    na, nb = case["na"], case["nb"]
    rng = np.random.default_rng(seed if case["op"] != "csr_build" else na * 10_000 + nb)
    s = wl.weight_strings(NORB, NEL)
    a = np.sort(s[rng.choice(s.size, size=na, replace=False)]).astype(np.int64)
    b = np.sort(s[rng.choice(s.size, size=nb, replace=False)]).astype(np.int64)
    return a, b


def _fermi_terms(h, eri):
    """The term list of ``workloads.molecular_terms``, written with array operations."""
    n = NORB
    p, q = (v.ravel() for v in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    p2, q2, r2, s2 = (v.ravel() for v in np.meshgrid(*[np.arange(n)] * 4, indexing="ij"))
    idx, code, coef, length = [], [], [], []
    for s in (0, n):
        idx.append(np.stack([p + s, q + s], 1).ravel())
        code.append(np.tile([wl.F_CRE, wl.F_ANN], p.size))
        coef.append(h.ravel())
        length.append(np.full(p.size, 2))
    for s in (0, n):
        for t in (0, n):
            idx.append(np.stack([p2 + s, r2 + t, s2 + t, q2 + s], 1).ravel())
            code.append(np.tile([wl.F_CRE, wl.F_CRE, wl.F_ANN, wl.F_ANN], p2.size))
            coef.append(0.5 * eri.ravel())
            length.append(np.full(p2.size, 4))
    ptr = np.concatenate([[0], np.cumsum(np.concatenate(length))]).astype(np.int64)
    return wl.TermList(2 * n, ptr, np.concatenate(idx).astype(np.int32), np.concatenate(code).astype(np.uint8),
                       np.concatenate(coef).astype(np.complex128), True)


def _requests(case, seed):
    """The batched case's requests: sizes log-uniform over 1e3 .. 6e4 rows, families in turn."""
    rng = np.random.default_rng(case["n"])
    out = []
    for k in range(case["n"]):
        size = int(math.exp(rng.uniform(math.log(1e3), math.log(6e4))))
        model = ("tfim", "xxz", "fermi")[k % 3]
        c = dict(op="matvec", model=model, nvec=1, dtype=case["dtype"], tuned=False)
        if model == "fermi":
            side = max(24, int(math.sqrt(size)))
            c.update(na=side, nb=side + 1)
        else:
            c.update(n=min(size, 4096) if model == "tfim" else size)
        out.append((c, seed * 1000 + k))
    return out


def _inputs(case, seed):
    """Bit-strings (device, [n][W]), qubits and term list of one operator."""
    model = case["model"]
    if model == "tfim":
        # a sample (the full space when n = 4096) of the 12-qubit chain at a field near criticality
        field = 1.0 + 0.2 * (np.random.default_rng(seed).random() - 0.5)
        bits = torch.randperm(4096, generator=_gen(seed), device="cuda")[: case["n"]].reshape(-1, 1)
        return bits, 12, wl.tfim_chain(12, 1.0, field)
    if model == "xxz":
        return _xxz_bits(case["n"], _gen(seed)), 36, wl.xxz_grid_6x6()
    if model == "hex":
        return _hex_bits(case["n"], _gen(seed)), 200, wl.heavy_hex_xy_field()
    a, b = _fermi_strings(case, seed)
    keys = ((b[:, None] << NORB) | a[None, :]).reshape(-1, 1)
    return torch.from_numpy(keys).cuda(), 2 * NORB, _fermi_terms(*wl.molecular_integrals(NORB, seed))


def _vectors(N, case, seed):
    g = _gen(seed + 1)
    shape = (N,) if case["nvec"] == 1 else (N, case["nvec"])
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float64) / math.sqrt(N)).to(DTYPES[case["dtype"]])


def _operator(case, seed):
    bits, nq, terms = _inputs(case, seed)
    sub = qsd.Subspace(bits, nq)
    H = qsd.SubspaceHamiltonian(sub, qsd.operator_from_termlist(terms))
    if case["tuned"]:
        sub.rehash(1.0 / 32.0)
        H.schedule = qsd.SCHED_ALL if case["nvec"] == 1 else \
            qsd.SCHED_XCD_REMAP | qsd.SCHED_SLOT_ORDER | qsd.SCHED_FILTER_FIRST
    return H


def prepare(case, seed):
    op = case["op"]
    if op == "batched":
        hams = [_operator(c, s) for c, s in _requests(case, seed)]
        xs = [_vectors(H.N, c, s) for H, (c, s) in zip(hams, _requests(case, seed))]
        return dict(op=op, hams=hams, xs=xs, ys=[torch.empty_like(x) for x in xs])
    if op == "setup":
        # a raw sample: one string in eight was measured twice
        bits, nq, terms = _inputs(case, seed)
        bits = torch.cat([bits, bits[: case["n"] // 8]])
        return dict(op=op, bits=bits, nq=nq, operator=qsd.operator_from_termlist(terms))
    H = _operator(case, seed)
    if op == "lanczos":
        return dict(op=op, H=H, seed=seed)
    if op == "csr_build":
        return dict(op=op, H=H, dtype=DTYPES[case["dtype"]])
    if op == "csr_matvec":
        H = qsd.CsrMatrix(H, qsd.INDEX_I32, DTYPES[case["dtype"]])
    x = _vectors(H.N, case, seed)
    return dict(op=op, H=H, x=x, y=torch.empty_like(x))


def run(state):
    op = state["op"]
    if op in ("matvec", "csr_matvec"):
        return state["H"].matvec(state["x"], out=state["y"])
    if op == "batched":
        return qsd.matvec_batched(state["hams"], state["xs"], state["ys"])
    if op == "csr_build":
        return state["H"].to_csr(qsd.INDEX_I32, state["dtype"])
    if op == "lanczos":
        e, v, _ = state["H"].lanczos(v0="uniform", want_vector=True, max_iter=300, raise_on_nonconv=False)
        return e, v
    sub = qsd.Subspace(state["bits"], state["nq"])
    H = qsd.SubspaceHamiltonian(sub, state["operator"])
    return sub.keys(), H.diagonal()


# ------------------------------------------------------------------------------------ work

def _rows(case):
    return case["na"] * case["nb"] if case["model"] == "fermi" else case["n"]


def _nnz(case):
    """Stored elements (expected over the samples), the diagonal included."""
    N = _rows(case)
    if case["model"] == "fermi":
        one, two = NEL * (NORB - NEL), math.comb(NEL, 2) * math.comb(NORB - NEL, 2)
        fa, fb = ((case[k] - 1) / (N_STRINGS - 1) for k in ("na", "nb"))
        return N * (1 + (one + two) * (fa + fb) + one * one * fa * fb)
    if case["model"] == "tfim":
        return N * (1 + 12 * N / 4096)
    if case["model"] == "xxz":
        return N * (1 + 31 * N / math.comb(36, 18))
    return N * 1.1


def work(case):
    op = case["op"]
    if op == "batched":
        parts = [work(c) for c, _ in _requests(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    N, nnz, v = _rows(case), _nnz(case), case["nvec"]
    s = 8 if case["dtype"] == "f64" else 4
    W = 4 if case["model"] == "hex" else 1
    keys = N * 8 * W
    if op == "setup":
        return {"bytes": 9 * keys // 8 + keys + 8 * N, "flops": N * 200.0 if W == 4 else N * 60.0}
    if op == "csr_build":
        return {"bytes": keys + nnz * (4 + s) + 8 * (N + 1), "flops": nnz}
    if op == "csr_matvec":
        return {"bytes": nnz * (4 + s) + 8 * N + 2 * s * v * N, "flops": 2 * nnz * v}
    one = {"bytes": keys + 8 * N + 2 * s * v * N, "flops": 2 * nnz * v}
    if op == "matvec":
        return one
    # a solve: its iterations' SpMVs, and the basis read twice per classical Gram-Schmidt pass
    m = {"tfim": 30, "xxz": 45, "hex": 100}[case["model"]]
    basis = 4 * 8 * N * m * (m + 1) / 2
    return {"bytes": m * one["bytes"] + basis, "flops": m * one["flops"] + basis / 4}


# ----------------------------------------------------------------------------------- exact

def _order(bits):
    """The distinct rows ``bits`` [n][W] in ascending unsigned order."""
    out = bits
    for w in range(bits.shape[1]):  # least significant word first: a stable sort per word
        out = out[torch.argsort(out[:, w] ^ _bit(63), stable=True)]
    return out


def _lookup(keys):
    """A function of a word-wise flip mask: for every row, the index of row ^ mask or -1."""
    W = keys.shape[1]
    if W == 1:
        col = keys[:, 0].contiguous()

        def find(mask):
            want = col ^ mask[0]
            at = torch.searchsorted(col, want).clamp_(max=col.numel() - 1)
            return torch.where(col[at] == want, at, -1)

        return find
    # wide rows: sorted 64-bit images (one pseudo-random word per bit), matches compared in full
    words = torch.from_numpy(np.random.default_rng(12345).integers(-2**62, 2**62, size=64 * W)).cuda()
    image = torch.zeros(keys.shape[0], dtype=torch.int64, device="cuda")
    for q in range(64 * W):
        image ^= torch.where(((keys[:, q // 64] >> (q % 64)) & 1) == 1, words[q], 0)
    srt, perm = torch.sort(image)

    def find(mask):
        flip = 0
        for q in range(64 * W):
            if (mask[q // 64] >> (q % 64)) & 1:
                flip ^= int(words[q])
        want = image ^ flip
        at = torch.searchsorted(srt, want).clamp_(max=srt.numel() - 1)
        j = perm[at]
        same = srt[at] == want
        for w in range(W):
            same &= keys[j, w] == (keys[:, w] ^ mask[w])
        return torch.where(same, j, -1)

    return find


def _spin_model(case, seed):
    """(keys, diagonal, hops): hops = (qubits flipped, coefficient, both bits must differ)."""
    bits, nq, terms = _inputs(case, seed)
    keys = _order(bits)

    def z(q):
        return 1.0 - 2.0 * ((keys[:, q // 64] >> (q % 64)) & 1).double()

    diag = torch.zeros(keys.shape[0], dtype=torch.float64, device="cuda")
    hops = {}
    for c, word in terms.terms():
        if all(k == wl.Z for _, k in word):
            t = torch.full_like(diag, c.real)
            for q, _ in word:
                t = t * z(q)
            diag += t
        else:
            hops[tuple(q for q, _ in word)] = (c.real, len(word) == 2)
    return keys, diag, [(q, c, d) for q, (c, d) in hops.items()]


def _spin_matvec(case, seed, x):
    keys, diag, hops = _spin_model(case, seed)
    find = _lookup(keys)
    X = x.reshape(keys.shape[0], -1).double()
    Y = diag[:, None] * X
    for qs, c, differ in hops:
        mask = [0] * keys.shape[1]
        for q in qs:
            mask[q // 64] ^= _bit(q % 64)
        j = find(mask)
        if differ:
            a, b = qs
            j = torch.where((((keys[:, a // 64] >> (a % 64)) ^ (keys[:, b // 64] >> (b % 64))) & 1) == 1, j, -1)
        rows = torch.nonzero(j >= 0)[:, 0]
        Y[rows] += c * X[j[rows]]
    return Y.reshape(x.shape)


def _excitations(strings):
    """For every pair (p, q) the row action of a+_p a_q on every 16-bit string: partner and sign
    (0 where it vanishes), [256][65536 strings] gathered at ``strings``."""
    s = strings
    part, sign = [], []
    for p in range(NORB):
        for q in range(NORB):
            if p == q:
                part.append(s)
                sign.append(((s >> p) & 1).double())
                continue
            ok = (((s >> p) & 1) == 1) & (((s >> q) & 1) == 0)
            lo, hi = min(p, q), max(p, q)
            cnt = torch.zeros_like(s)
            for r in range(lo + 1, hi):
                cnt += (s >> r) & 1
            part.append(s ^ ((1 << p) | (1 << q)))
            sign.append(torch.where(ok, 1.0 - 2.0 * (cnt & 1).double(), 0.0))
    return torch.stack(part), torch.stack(sign)


class _Molecule:
    def __init__(self, case, seed):
        a, b = _fermi_strings(case, seed)
        h, eri = wl.molecular_integrals(NORB, seed)
        self.h = torch.from_numpy(h).cuda().reshape(-1)
        self.eri = torch.from_numpy(eri).cuda().reshape(NORB * NORB, NORB * NORB)
        self.S = [torch.from_numpy(v).cuda() for v in (a, b)]
        self.pos, self.E, self.one_spin = [], [], []
        for s in self.S:
            pos = torch.full((1 << NORB,), -1, dtype=torch.int64, device="cuda")
            pos[s] = torch.arange(s.numel(), device="cuda")
            self.pos.append(pos)
            self.E.append(_excitations(s))
            self.one_spin.append(self._same_spin(s, pos, *self.E[-1]))

    def _same_spin(self, s, pos, part, sign):
        """sum h_pq E_pq + 1/2 sum (pq|rs) (E_pq E_rs - delta_qr E_ps) on the sampled strings."""
        n = s.numel()
        M = torch.zeros((n, n), dtype=torch.float64, device="cuda")
        rows = torch.arange(n, device="cuda")
        every = torch.arange(1 << NORB, device="cuda")
        ap, asg = _excitations(every)

        def put(i, col, val):
            j = pos[col]
            ok = (j >= 0) & (val != 0)
            M.index_put_((i[ok], j[ok]), val[ok], accumulate=True)

        contracted = torch.einsum("pqqs->ps", self.eri.reshape([NORB] * 4)).reshape(-1)
        for pq in range(NORB * NORB):
            put(rows, part[pq], sign[pq] * (self.h[pq] - 0.5 * contracted[pq]))
            on = torch.nonzero(sign[pq])[:, 0]
            mid = part[pq, on]
            val = 0.5 * sign[pq, on][None, :] * asg[:, mid] * self.eri[pq][:, None]
            put(on[None, :].expand(val.shape), ap[:, mid], val)
        return M

    def matvec(self, x):
        """y[b][a] = sum over both spins' matrices and (pq|rs) E_pq (alpha) E_rs (beta)."""
        na, nb = (s.numel() for s in self.S)
        X = x.reshape(nb, na, -1).double().permute(2, 0, 1).contiguous()  # [v][b][a]
        Y = torch.stack([self.one_spin[1] @ v + v @ self.one_spin[0].T for v in X])
        (pa, sa), (pb, sb) = self.E
        ja, jb = self.pos[0][pa], self.pos[1][pb]
        ra = torch.arange(na, device="cuda").expand(ja.shape)
        ok = (ja >= 0) & (sa != 0)
        for rs in range(NORB * NORB):
            on = torch.nonzero((sb[rs] != 0) & (jb[rs] >= 0))[:, 0]
            if on.numel() == 0:
                continue
            G = torch.zeros((na, na), dtype=torch.float64, device="cuda")
            G.index_put_((ra[ok], ja[ok]), (sa * self.eri[:, rs][:, None])[ok], accumulate=True)
            for v in range(X.shape[0]):
                Y[v, on] += sb[rs, on][:, None] * (X[v, jb[rs, on]] @ G.T)
        return Y.permute(1, 2, 0).reshape(x.shape)

    def csr_values(self):
        """Values of all stored elements, rows then columns ascending."""
        (na, nb), pairs = (s.numel() for s in self.S), []
        for k in (0, 1):
            s, d = self.S[k], None
            d = s[:, None] ^ s[None, :]
            dist = sum(((d >> q) & 1) for q in range(NORB))
            one = torch.nonzero(dist == 2)
            two = torch.nonzero(dist == 4)
            i, j = one[:, 0], one[:, 1]
            p = ((s[i] & ~s[j]).double().log2()).long()
            q = ((s[j] & ~s[i]).double().log2()).long()
            pairs.append((i, j, p * NORB + q, self.E[k][1][p * NORB + q, i], two[:, 0], two[:, 1]))
        occ = [torch.stack([(s >> q) & 1 for q in range(NORB)], 1).double() for s in self.S]
        dd = torch.arange(NORB, device="cuda") * (NORB + 1)
        coul = self.eri[dd][:, dd]
        A, B = torch.arange(na, device="cuda"), torch.arange(nb, device="cuda")
        R, C, V = [], [], []

        def add(bi, bj, ai, aj, v):
            r, c, v = torch.broadcast_tensors(bi * na + ai, bj * na + aj, v)
            R.append(r.reshape(-1)), C.append(c.reshape(-1)), V.append(v.reshape(-1))

        Ha, Hb = self.one_spin
        (ia, ja, ea, ga, ua, va), (ib, jb, eb, gb, ub, vb) = pairs
        add(B[:, None], B[:, None], A[None, :], A[None, :],
            Hb.diagonal()[:, None] + Ha.diagonal()[None, :] + occ[1] @ coul @ occ[0].T)
        add(B[:, None], B[:, None], ia[None, :], ja[None, :], Ha[ia, ja][None, :] + occ[1] @ (self.eri[dd][:, ea] * ga))
        add(B[:, None], B[:, None], ua[None, :], va[None, :], Ha[ua, va][None, :])
        add(ib[:, None], jb[:, None], A[None, :], A[None, :], Hb[ib, jb][:, None] + (self.eri[eb][:, dd] * gb[:, None]) @ occ[0].T)
        add(ub[:, None], vb[:, None], A[None, :], A[None, :], Hb[ub, vb][:, None])
        add(ib[:, None], jb[:, None], ia[None, :], ja[None, :], self.eri[eb][:, ea] * gb[:, None] * ga[None, :])
        r, c, v = torch.cat(R), torch.cat(C), torch.cat(V)
        return v[torch.argsort(r * (na * nb) + c)]


def _exact_matvec(case, seed):
    if case["model"] == "fermi":
        return _Molecule(case, seed).matvec(_vectors(case["na"] * case["nb"], case, seed))
    return _spin_matvec(case, seed, _vectors(_rows(case), case, seed))


def exact(case, seed):
    op = case["op"]
    if op in ("matvec", "csr_matvec"):
        return _exact_matvec(case, seed)
    if op == "batched":
        return [_exact_matvec(c, s) for c, s in _requests(case, seed)]
    if op == "csr_build":
        return None, None, _Molecule(case, seed).csr_values()
    if op == "setup":
        keys, diag, _ = _spin_model(case, seed)
        return None, diag
    if case["model"] == "tfim" and case["n"] == 4096:
        # free-fermion energy of the periodic chain, antiperiodic momenta
        f = 1.0 + 0.2 * (np.random.default_rng(seed).random() - 0.5)
        k = math.pi * (2 * np.arange(12) + 1) / 12
        return float(-np.sum(np.sqrt(1.0 + f * f - 2.0 * f * np.cos(k)))), None
    return None
