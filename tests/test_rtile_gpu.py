"""Register tile passes (csrc/rtile.hpp) against the oracle at every tile width
they take: each kind of matrix with its target on register, lane, wavefront
and outer bits in turn, controls of both values in every position, blocks of
diagonal gates short and long, angles from the device, and tiles that no gate
touches.  Tolerances are the library's: 1e-12 (complex128) and 1e-5
(complex64) of the largest amplitude."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 1e-5}
# tiles of 64, 128, 256 and 512 lanes (16 complex128 or 32 complex64 per lane)
WIDTHS = [("c128", m) for m in (10, 11, 12, 13)] + [("c64", m) for m in (11, 12, 13, 14)]


def _matrix(rng, shape):
    a, b, c = rng.uniform(0, 2 * np.pi, 3)
    if shape == "general":
        return W.haar_unitary_2x2(int(rng.integers(1 << 30)))
    if shape == "cross":     # real diagonal, imaginary off-diagonal
        return (np.cos(a), 0.0, 0.0, -np.sin(a), 0.0, -np.sin(a), np.cos(a), 0.0)
    if shape == "diagonal":  # not of unit modulus
        return (0.9 * np.cos(a), 0.9 * np.sin(a), 0.0, 0.0, 0.0, 0.0, 1.1 * np.cos(b), 1.1 * np.sin(b))
    return (np.cos(a), 0.0, -np.sin(a), 0.0, np.sin(a), 0.0, np.cos(a), 0.0)


def _random_circuit(n, count, seed, params=0):
    rng = np.random.default_rng(seed)
    kinds = ["X", "Y", "Z", "H", "RX", "RY", "RZ", "P", "U", "~RX", "~RZ", "~P", "~U"]
    gates = []
    for _ in range(count):
        kind = kinds[int(rng.integers(len(kinds)))]
        t = int(rng.integers(n))
        nc = int(rng.integers(0, 4))
        ctrls = tuple(int(q) for q in rng.choice([q for q in range(n) if q != t], size=nc, replace=False))
        vals = tuple(int(v) for v in rng.integers(0, 2, size=nc))
        mat = _matrix(rng, ("general", "cross", "diagonal", "real")[int(rng.integers(4))]) if kind[-1] == "U" else None
        p = int(rng.integers(params)) if params and kind in ("RX", "RY", "RZ", "P") and rng.random() < 0.7 else -1
        gates.append(W.Gate(kind, t, ctrls, vals, float(rng.uniform(0, 6.28)) if p < 0 else 0.0, p, mat))
    return W.Circuit(n, gates, rng.uniform(0, 6.28, params) if params else None)


def _diagonal_circuit(n, count, seed):
    """Blocks of diagonal gates between two layers of H: up to `count` phases
    in a row, many sharing a condition."""
    rng = np.random.default_rng(seed)
    gates = [W.Gate("H", q) for q in range(n)]
    for _ in range(count):
        t = int(rng.integers(n))
        nc = int(rng.integers(0, 4))
        ctrls = tuple(int(q) for q in rng.choice([q for q in range(n) if q != t], size=nc, replace=False))
        gates.append(W.Gate(("P", "RZ", "Z")[int(rng.integers(3))], t, ctrls,
                            tuple(int(v) for v in rng.integers(0, 2, size=nc)), float(rng.uniform(0, 6.28))))
    return W.Circuit(n, gates + [W.Gate("H", q) for q in range(n)])


def _check(gpu, circ, dtype, params=None, seed=3, slack=0.0):
    psi0 = W.random_state(circ.n, seed)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    psi = torch.tensor(psi0, device="cuda").to(tdt)
    plan = gpu.Circuit(circ.n, circ, dtype=gpu.SV_C128 if dtype == "c128" else gpu.SV_C64, nparams=circ.nparams)
    for p in ([None] if params is None else params):
        start = psi.cpu().numpy().astype(np.complex128)
        plan.run(psi, None if p is None else torch.tensor(p, device="cuda"))
        ref = oracle.run_circuit(circ, params=p, psi0=start)
        got = psi.cpu().numpy().astype(np.complex128)
        assert np.abs(got - ref).max() <= (TOL[dtype] + slack) * np.abs(ref).max()


@pytest.mark.parametrize("dtype,m", WIDTHS)
@pytest.mark.parametrize("extra", [0, 2, 9])
def test_all_kinds(gpu, dtype, m, extra):
    """One tile, a few, and more than there are CUs (up to 256 tiles a lane
    holds half as many amplitudes)."""
    if extra == 9 and m > 12:
        pytest.skip("tiles of 512 lanes hold the same amplitudes per lane at every count")
    gpu.sv_tune_set("tile_log2_" + dtype, m)
    _check(gpu, _random_circuit(m + extra, 160 if extra < 9 else 60, 100 * m + extra), dtype)


@pytest.mark.parametrize("dtype,m", WIDTHS)
def test_narrow_low_block_and_angles(gpu, dtype, m):
    gpu.sv_tune_set("tile_log2_" + dtype, m)
    gpu.sv_tune_set("tile_low_bits_" + dtype, 1 + m // 13 * 3)
    c = _random_circuit(m + 2, 120, 7 * m, params=24)
    rng = np.random.default_rng(m)
    _check(gpu, c, dtype, params=[c.params, rng.uniform(0, 6.28, 24)])


@pytest.mark.parametrize("dtype,m", [("c128", 10), ("c128", 12), ("c64", 11), ("c64", 14)])
@pytest.mark.parametrize("count,extra", [(5, 1), (60, 1), (3000, 1), (40, 9)])
def test_diagonal_blocks(gpu, dtype, m, count, extra):
    """A block adds phases: up to `count` additions, each rounding a sum of
    at most 2 pi count to 53 bits (beside the library's tolerance)."""
    gpu.sv_tune_set("tile_log2_" + dtype, m)
    _check(gpu, _diagonal_circuit(m + extra, count, count + m), dtype, slack=2 * np.pi * count ** 2 * 2.0 ** -53)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_untouched_tiles_keep_their_bytes(gpu, dtype):
    """Every gate needs one of two outer controls: tiles with both clear stay
    as they are, bit for bit (and the rest follow the oracle)."""
    n = 15
    rng = np.random.default_rng(5)
    gates = [W.Gate("RY", int(rng.integers(0, 8)), (13 if i % 2 else 14,), (1,), float(rng.uniform(0, 6)))
             for i in range(24)]
    c = W.Circuit(n, gates)
    gpu.sv_tune_set("tile_log2_" + dtype, 11)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    psi = torch.tensor(W.random_state(n, 8), device="cuda").to(tdt)
    before = psi.clone()
    gpu.Circuit(n, c, dtype=gpu.SV_C128 if dtype == "c128" else gpu.SV_C64).run(psi)
    k = 1 << 13
    assert torch.equal(psi[:k], before[:k])
    ref = oracle.run_circuit(c, psi0=before.cpu().numpy().astype(np.complex128))
    assert np.abs(psi.cpu().numpy() - ref).max() <= TOL[dtype] * np.abs(ref).max()


@pytest.mark.parametrize("dtype,m", WIDTHS)
@pytest.mark.parametrize("diagonals", [False, True])
def test_reverse_sweep(gpu, dtype, m, diagonals):
    """Gradients of every parameterised kind (and their adjoints) under 0-2
    controls of either value, blocks of diagonal gates among them, against the
    oracle's shift rules at 1e-8 (complex128).  complex64 states: every
    amplitude error of the library's 1e-5 enters a term 2 Re <lambda|A|psi>,
    |lambda| <= sum|coef|, once from each state and for each of a parameter's
    gates."""
    gpu.sv_tune_set("tile_log2_" + dtype, m)
    n, P = m + 1 if m < 13 else m, 10
    rng = np.random.default_rng(50 * m + diagonals)
    kinds = ("RZ", "P", "~RZ", "~P", "RZ", "Z") if diagonals else ("RX", "RY", "RZ", "P", "~RX", "~RY", "H", "X", "U")
    gates = [W.Gate("RY", q, theta=float(rng.uniform(0, 6))) for q in range(n)]
    for i in range(40):
        kind = "H" if diagonals and i % 14 == 13 else kinds[i % len(kinds)]
        t = int(rng.integers(n))
        nc = int(rng.integers(0, 3))
        ctrls = tuple(int(q) for q in rng.choice([q for q in range(n) if q != t], size=nc, replace=False))
        p = int(rng.integers(P)) if kind[-1] in "XYZP" and len(kind.strip("~")) == (1 if kind[-1] == "P" else 2) else -1
        gates.append(W.Gate(kind, t, ctrls, tuple(int(v) for v in rng.integers(0, 2, size=nc)),
                            float(rng.uniform(0, 6)), p, _matrix(rng, "general") if kind == "U" else None))
    c = W.Circuit(n, gates, rng.uniform(0, 6.28, P))
    terms = W.zz_x_hamiltonian(n, 3)
    ref = oracle.grad_param_shift(c, c.params, terms)
    code, tdt = (gpu.SV_C128, torch.complex128) if dtype == "c128" else (gpu.SV_C64, torch.complex64)
    params = torch.tensor(c.params, device="cuda")
    psi = torch.zeros(1 << n, dtype=tdt, device="cuda")
    psi[0] = 1
    gpu.Circuit(n, c, dtype=code, nparams=P).run(psi, params)
    grad, _ = gpu.AdjointPlan(n, c, terms, P, dtype=code).run(psi, torch.empty_like(psi), params)
    l1 = sum(abs(t.coef) for t in terms)
    uses = max(sum(g.param == j for g in gates) for j in range(P))
    tol = 1e-8 * max(1.0, np.abs(ref).max()) if dtype == "c128" else 2e-5 * l1 * uses
    assert np.abs(grad.cpu().numpy() - ref).max() <= tol
    psi[0] -= 1  # the sweep un-applies every gate
    assert psi.abs().max().item() <= TOL[dtype]


@pytest.mark.parametrize("dtype,n", [("c128", 12), ("c128", 14), ("c64", 13), ("c64", 15), ("c64", 17)])
def test_runs_of_x_only(gpu, dtype, n):
    """Runs that only permute (a gather through LDS tiles, or register tiles):
    amplitudes move exactly."""
    rng = np.random.default_rng(n)
    gates = []
    for _ in range(40):
        t, nc = int(rng.integers(n)), int(rng.integers(0, 5))
        ctrls = tuple(int(q) for q in rng.choice([q for q in range(n) if q != t], size=nc, replace=False))
        gates.append(W.Gate("X", t, ctrls, tuple(int(v) for v in rng.integers(0, 2, size=nc))))
    for c in (W.Circuit(n, gates), W.stream(n)):
        tdt = torch.complex128 if dtype == "c128" else torch.complex64
        psi = torch.tensor(W.random_state(n, 4), device="cuda").to(tdt)
        ref = oracle.run_circuit(c, psi0=psi.cpu().numpy().astype(np.complex128))
        gpu.Circuit(n, c, dtype=gpu.SV_C128 if dtype == "c128" else gpu.SV_C64).run(psi)
        assert np.array_equal(psi.cpu().numpy().astype(np.complex128), ref)


@pytest.mark.parametrize("dtype,m", [("c128", m) for m in (8, 10, 11, 12)] + [("c64", m) for m in (8, 11, 12, 13)])
def test_batched(gpu, dtype, m):
    """Batched circuits on a workgroup of 256 lanes: tiles that leave part of
    a wavefront or whole wavefronts idle, states of one tile and of many, the
    smallest states on register tiles and the largest that stay in LDS."""
    gpu.sv_tune_set("tile_log2_" + dtype, m)
    ns = [9, 10, 11, 12, 13, 14, 15, 10]
    circs = [_random_circuit(n, 90, 50 * m + i, params=8) for i, n in enumerate(ns)]
    circs[-1] = W.Circuit(ns[-1], _diagonal_circuit(ns[-1], 60, m).gates, np.zeros(0))
    psi0 = [W.random_state(n, 5 + i) for i, n in enumerate(ns)]
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    psis = [torch.tensor(p, device="cuda").to(tdt) for p in psi0]
    starts = [p.cpu().numpy().astype(np.complex128) for p in psis]
    params = torch.tensor(np.concatenate([c.params for c in circs]), device="cuda")
    gpu.sv_apply_circuits_batched(psis, circs, params)
    for c, psi, start in zip(circs, psis, starts):
        ref = oracle.run_circuit(c, params=c.params, psi0=start)
        got = psi.cpu().numpy().astype(np.complex128)
        slack = 2 * np.pi * 60 ** 2 * 2.0 ** -53 if c is circs[-1] else 0.0
        assert np.abs(got - ref).max() <= (TOL[dtype] + slack) * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("m", [7, 9, 13])
def test_batched_gradients(gpu, dtype, m):
    """Batched reverse sweeps: states swept in LDS, tiles that leave lanes
    idle, one tile and many, angles that several gates share, diagonal and
    single-gate passes; in a batch of few circuits the wide ones are split
    over workgroups, with the same gradients however far.  Tolerances as for
    the single sweep above."""
    gpu.sv_tune_set("tile_log2_" + dtype, m)
    ns = [2, 4, 5, 7, 10, 12, 13, 15]
    circs = [_random_circuit(n, 40, 30 * m + i, params=4) if n > 3 else W.hea(n, 2, seed=i) for i, n in enumerate(ns)]
    for c in circs:  # unitary gates only
        c.gates[:] = [g for g in c.gates if g.kind[-1] != "U"]
    hams = [W.zz_x_hamiltonian(n, 70 + n) for n in ns]
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    params = torch.tensor(np.concatenate([c.params for c in circs]), device="cuda")
    finals = [torch.tensor(oracle.run_circuit(c, params=c.params), device="cuda").to(tdt) for c in circs]
    got = []
    for split in (1, 64):
        gpu.sv_tune_set("batch_split", split)
        psis = [f.clone() for f in finals]
        lams = [torch.empty_like(f) for f in finals]
        grad, loss = gpu.sv_adjoint_grad_batched(psis, lams, circs, params, hams)
        got.append((grad.cpu().numpy(), loss.cpu().numpy(), psis))
    off = 0
    for i, (c, h) in enumerate(zip(circs, hams)):
        p = slice(off, off + c.nparams)
        off += c.nparams
        l1 = sum(abs(t.coef) for t in h)
        uses = max(sum(g.param == j for g in c.gates) for j in range(c.nparams))
        # the same terms in other partial sums: at most 2^15 additions of 53 bits
        assert np.abs(got[0][0][p] - got[1][0][p]).max() <= 2.0 ** -37 * l1 * uses
        assert abs(got[0][1][i] - got[1][1][i]) <= 2.0 ** -37 * l1
        assert torch.equal(got[0][2][i], got[1][2][i])
        ref = oracle.grad_param_shift(c, c.params, h)
        tol = 1e-8 * max(1.0, np.abs(ref).max()) if dtype == "c128" else 2e-5 * l1 * uses
        assert np.abs(got[0][0][p] - ref).max() <= tol, c.n
        assert abs(got[0][1][i] - oracle.loss(c, c.params, h)) <= (1e-10 if dtype == "c128" else 2e-5 * l1)


def test_default_complex64_tiles_with_full_lanes(gpu):
    """Random gates on the default complex64 width, 2^13, with more tiles than
    CUs: 256 lanes of 32 amplitudes each, where up to 256 tiles have 512 of 16."""
    gpu.sv_tune_set("tile_log2_c64", 13)
    _check(gpu, _random_circuit(22, 60, 1322), "c64")
