"""Batches of small states: register tiles where the batch is planned, gate by
gate in LDS where it runs once, against the oracle at the library's 1e-12
(complex128) and 1e-5 (complex64) of the largest amplitude."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 1e-5}


def _circuit(n, count, seed):
    rng = np.random.default_rng(seed)
    kinds = ["X", "Y", "Z", "H", "RX", "RY", "RZ", "P", "U", "~RX", "~RZ", "~P", "~U"]
    gates, params = [], rng.uniform(0, 6.28, 6)
    for _ in range(count):
        kind, t = kinds[int(rng.integers(len(kinds)))], int(rng.integers(n))
        others = [q for q in range(n) if q != t]
        nc = int(rng.integers(0, min(3, n - 1) + 1))
        ctrls = tuple(int(q) for q in rng.choice(others, size=nc, replace=False)) if nc else ()
        vals = tuple(int(v) for v in rng.integers(0, 2, size=nc))
        p = int(rng.integers(6)) if kind in ("RX", "RY", "RZ", "P") and rng.random() < 0.5 else -1
        mat = W.haar_unitary_2x2(int(rng.integers(1 << 30))) if kind[-1] == "U" else None
        gates.append(W.Gate(kind, t, ctrls, vals, float(rng.uniform(0, 6.28)) if p < 0 else 0.0, p, mat))
    return W.Circuit(n, gates, params)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("ns", [[1, 2, 3, 4, 5, 6, 7], [4, 7, 9, 10, 11, 12], [12, 13, 8], [11, 12, 13, 14, 5]],
                         ids=["tiny", "small", "edge", "mixed"])
def test_small_states(gpu, dtype, ns):
    """Widths around what LDS holds (12 qubits of complex128, 13 of complex64;
    half of it beside wider circuits) and around the smallest register tiles."""
    circs = [_circuit(n, 70, 100 * n + len(ns)) for n in ns]
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    params = torch.tensor(np.concatenate([c.params for c in circs]), device="cuda")
    start = [torch.tensor(W.random_state(n, n), device="cuda").to(tdt) for n in ns]
    refs = [oracle.run_circuit(c, params=c.params, psi0=s.cpu().numpy().astype(np.complex128))
            for c, s in zip(circs, start)]
    once = [s.clone() for s in start]
    gpu.sv_apply_circuits_batched(once, circs, params)
    kept = [s.clone() for s in start]
    batch = gpu.Batch(kept, circs)
    batch.run(params)
    batch.close()
    for n, ref, a, b in zip(ns, refs, once, kept):
        for got in (a, b):
            assert np.abs(got.cpu().numpy() - ref).max() <= TOL[dtype] * np.abs(ref).max(), n


@pytest.mark.parametrize("once", [False, True])
def test_complex64_angles_round_alike_with_and_without_gradients(gpu, once):
    """A parameterised complex64 batch gives the same bits whether or not it
    has lambda states to take gradients with."""
    ns = [9, 13, 14, 15]
    circs = [_circuit(n, 90, 30 + n) for n in ns]
    for c in circs:  # unitary gates only
        c.gates[:] = [g for g in c.gates if g.kind[-1] != "U"]
    params = torch.tensor(np.concatenate([c.params for c in circs]), device="cuda")
    start = [torch.tensor(W.random_state(n, n), device="cuda").to(torch.complex64) for n in ns]
    plain, both = [s.clone() for s in start], [s.clone() for s in start]
    if once:
        gpu.sv_apply_circuits_batched(plain, circs, params)
    else:
        batch = gpu.Batch(plain, circs)
        batch.run(params)
        batch.close()
    batch = gpu.Batch(both, circs, lam_states=[torch.empty_like(s) for s in start],
                      hamiltonians=[W.zz_x_hamiltonian(n, n) for n in ns])
    batch.run(params)
    batch.close()
    for a, b in zip(plain, both):
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
