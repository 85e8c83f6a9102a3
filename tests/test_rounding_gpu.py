"""Rounding of the kernels where a looser one would pass the oracle tests:
bounds counted from the roundings each result may have."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def test_expectation_sums_by_pairs(gpu):
    """2^18 amplitudes of equal |psi_k|^2 = v: a sum of two equal numbers is
    exact in binary, so tiles, lanes and workgroups that add by pairs give
    exactly 2^18 v (one after another, the third addend already rounds)."""
    n = 18
    for a in np.random.default_rng(2).uniform(0.5, 1.0, 16):
        psi = torch.full((1 << n,), complex(a), dtype=torch.complex128, device="cuda")
        got = float(gpu.sv_expect(psi, gpu.pauli_terms([W.PauliTerm(1.0, 0, 0)]))[0])
        assert got == (1 << n) * (a * a), a


def _phases(n, count, controls, seed):
    """Diagonal gates on every qubit in turn, each under `controls` controls of
    either value, and the phase they give every basis state."""
    rng = np.random.default_rng(seed)
    k = np.arange(1 << n)
    gates, phase = [], np.zeros(1 << n)
    for i in range(count):
        kind, t, theta = ("P", "RZ", "P")[i % 3], i % n, float(rng.uniform(-np.pi, np.pi))
        nc = int(rng.integers(0, controls + 1))
        ctrls = tuple(int(q) for q in rng.choice([q for q in range(n) if q != t], size=nc, replace=False))
        vals = tuple(int(v) for v in rng.integers(0, 2, size=nc))
        gates.append(W.Gate(kind, t, ctrls, vals, theta))
        on = np.ones(1 << n, dtype=bool)
        for c, v in zip(ctrls, vals):
            on &= ((k >> c) & 1) == v
        bit = (k >> t) & 1
        phase += np.where(on, theta * bit if kind == "P" else theta * (bit - 0.5), 0.0)
    return W.Circuit(n, gates), phase


@pytest.mark.parametrize("m", [11, 12, 13, 14])
@pytest.mark.parametrize("extra", [0, 9])
@pytest.mark.parametrize("controls", [0, 1, 3])
def test_complex64_phase_block_rounds_once(gpu, m, extra, controls):
    """However many diagonal gates a block has, an amplitude a of a complex64
    state is multiplied by one factor f: with u = 2^-24, each part of f is off
    by u / 2 at most (|f| <= 1: sqrt(2)/2 u |a| in all), a part of the product
    by u (|f_i a_i| + |result|), which is at most 2 u |a| for both; the factor
    itself is formed in double, to 1e-7 u.  One tile per workgroup and more
    tiles than CUs (other numbers of amplitudes per lane), no controls, one,
    and up to three."""
    if m + extra > 21:
        extra = 21 - m
    n = m + extra
    gpu.sv_tune_set("tile_log2_c64", m)
    c, phase = _phases(n, 4 * n, controls, 10 * m + controls)
    psi = torch.tensor(W.random_state(n, m), device="cuda").to(torch.complex64)
    a = psi.cpu().numpy().astype(np.complex128)
    gpu.Circuit(n, c, dtype=gpu.SV_C64).run(psi)
    err = np.abs(psi.cpu().numpy() - a * np.exp(1j * phase))
    assert (err <= 2.75 * 2.0 ** -24 * np.abs(a)).all(), (err / np.abs(a)).max() * 2.0 ** 24


@pytest.mark.parametrize("m", [10, 12])
@pytest.mark.parametrize("extra", [0, 9])
def test_complex128_phase_sums(gpu, m, extra):
    """RZ on every qubit, u = 2^-53: each gate's phase is off by the rounding of
    its entries and of their angle, at most u / 2 rms together; the block's sums
    add nothing, and its two factors per amplitude (of the lane and of the
    register) and their products round 0.65 u rms each.  (A sum in double of
    nine phases of several radians would add 5 u.)"""
    n = m + extra
    gpu.sv_tune_set("tile_log2_c128", m)
    worst = 0.0
    for seed in range(6):
        rng = np.random.default_rng(100 * m + seed)
        theta = rng.uniform(np.pi / 2, 2 * np.pi, n)  # long sums
        k = np.arange(1 << n)
        phase = sum(np.longdouble(t) * (((k >> q) & 1) - np.longdouble(0.5)) for q, t in enumerate(theta))
        exact = np.cos(phase) + 1j * np.sin(phase)
        psi = torch.ones(1 << n, dtype=torch.complex128, device="cuda")
        gpu.Circuit(n, W.Circuit(n, [W.Gate("RZ", q, theta=float(t)) for q, t in enumerate(theta)])).run(psi)
        err = (psi.cpu().numpy() - exact).astype(np.complex128)
        worst = max(worst, float(np.sqrt((np.abs(err) ** 2).mean())))
    assert worst <= np.sqrt(n * 0.25 + 2 * 0.65 ** 2) * 2.0 ** -53, worst * 2.0 ** 53


@pytest.mark.parametrize("controls", [0, 1, 3])
def test_complex64_phase_block_rounds_once_in_batches(gpu, controls):
    """The same bound for planned batches, whose tiles are loaded by workgroups
    of one size: states of a part of a tile, one, and many."""
    ns = [8, 10, 13, 14, 16]
    made = [_phases(n, 4 * n, controls, n + controls) for n in ns]
    psis = [torch.tensor(W.random_state(n, n), device="cuda").to(torch.complex64) for n in ns]
    starts = [p.cpu().numpy().astype(np.complex128) for p in psis]
    batch = gpu.Batch(psis, [c for c, _ in made])
    batch.run()
    batch.close()
    for n, (_, phase), psi, a in zip(ns, made, psis, starts):
        err = np.abs(psi.cpu().numpy() - a * np.exp(1j * phase))
        assert (err <= 2.75 * 2.0 ** -24 * np.abs(a)).all(), (n, (err / np.abs(a)).max() * 2.0 ** 24)
