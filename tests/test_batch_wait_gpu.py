"""Waits between the workgroups of a split circuit: they outlast chunks that
take long, and where one gives up all the same, gradients say so."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _batch(gpu, dtype, n, ncirc, terms, split):
    gpu.sv_tune_set("batch_split", split)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    circs = [W.hea(n, 2, seed=i) for i in range(ncirc)]
    psi = torch.zeros(ncirc, 1 << n, dtype=tdt, device="cuda")
    lam = torch.empty_like(psi)
    params = torch.tensor(np.concatenate([c.params for c in circs]), device="cuda")
    b = gpu.Batch(list(psi), circs, lam_states=list(lam), hamiltonians=[terms] * ncirc)
    return b, psi, params, circs[0].nparams


def _gradients(b, psi, params, ncirc):
    psi.zero_()
    psi[:, 0] = 1
    b.run(params)
    grad, loss = b.adjoint(params)
    return grad.cpu().numpy().reshape(ncirc, -1), loss.cpu().numpy()


def _reference(gpu, dtype, n, ncirc, terms):
    b, psi, params, _ = _batch(gpu, dtype, n, ncirc, terms, 1)
    try:
        return _gradients(b, psi, params, ncirc)
    finally:
        b.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_chunks_that_outlast_the_knob(gpu, dtype):
    """30,000 terms on 15 qubits: a chunk of H psi (1024 or more amplitudes)
    takes milliseconds, more than the shortest wait there is, and the limit
    follows it.  Tolerance: the same terms in other partial sums, at most 2^15
    additions of 53 bits."""
    n, ncirc = 15, 2
    rng = np.random.default_rng(3)
    terms = [W.PauliTerm(float(rng.uniform(-1, 1)), int(rng.integers(1 << n)), 0) for _ in range(30000)]
    ref = _reference(gpu, dtype, n, ncirc, terms)
    gpu.sv_tune_set("batch_wait_ms", 1)
    b, psi, params, _ = _batch(gpu, dtype, n, ncirc, terms, 64)
    try:
        grad, loss = _gradients(b, psi, params, ncirc)
        assert b.wait_timeouts() == 0
    finally:
        b.close()
    l1 = sum(abs(t.coef) for t in terms)
    assert np.abs(grad - ref[0]).max() <= 2.0 ** -37 * l1
    assert np.abs(loss - ref[1]).max() <= 2.0 ** -37 * l1


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gradients_after_a_wait_gave_up(gpu, dtype):
    """Waits that give up at once ("batch_wait_ms" 0): every circuit's loss and
    gradients are NaN, or, where no wait of its own gave up, right."""
    n, ncirc = 15, 6
    terms = W.zz_x_hamiltonian(n, 3)
    ref = _reference(gpu, dtype, n, ncirc, terms)
    gpu.sv_tune_set("batch_wait_ms", 0)
    b, psi, params, _ = _batch(gpu, dtype, n, ncirc, terms, 64)
    l1 = sum(abs(t.coef) for t in terms)
    try:
        # final states without a wait, for sweeps that have them
        gpu.sv_tune_set("batch_wait_ms", 10000)
        fwd, fpsi, _, _ = _batch(gpu, dtype, n, ncirc, terms, 1)
        fpsi.zero_()
        fpsi[:, 0] = 1
        fwd.run(params)
        fwd.close()
        gone = 0
        for _ in range(5):
            psi.copy_(fpsi)
            grad, loss = b.adjoint(params)
            grad, loss = grad.cpu().numpy().reshape(ncirc, -1), loss.cpu().numpy()
            for i in range(ncirc):
                if np.isnan(loss[i]):
                    assert np.isnan(grad[i]).all()
                    gone += 1
                else:
                    assert np.abs(grad[i] - ref[0][i]).max() <= 2.0 ** -37 * l1
                    assert abs(loss[i] - ref[1][i]) <= 2.0 ** -37 * l1
        assert (gone > 0) == (b.wait_timeouts() > 0)
        print("circuits without gradients", gone, "waits", b.wait_timeouts(), flush=True)
    finally:
        b.close()
