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
