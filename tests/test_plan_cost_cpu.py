"""Host time of planning (no device: the calls end with an error where they
would allocate).  Ratios of times on one machine, with margins of several
times what is measured."""
import ctypes
import time

import pytest

import paper_2411_18354_amd as sv
import workloads as W
from paper_2411_18354_amd import batched


@pytest.fixture(autouse=True)
def _host_only():
    import torch
    if torch.cuda.is_available():
        pytest.skip("states here are addresses that no kernel may touch")


def _arguments(circs):
    states = (sv.sv_state_t * len(circs))(*[sv.sv_state_t(1 << 20, c.n, sv.SV_C128) for c in circs])
    gates, offsets = batched._concat_gates(circs)
    return states, gates, offsets, batched._offsets([0] * len(circs))


def _seconds(call, repeats=5):
    best = 1e9
    for _ in range(repeats):
        t = time.perf_counter()
        assert call() in (sv.SV_EHIP, sv.SV_ENOMEM)
        best = min(best, time.perf_counter() - t)
    return best


def _plan_seconds(circs):
    states, gates, offsets, params = _arguments(circs)
    return _seconds(lambda: sv._L.sv_batch_create(states, None, len(circs), gates, offsets, params, 0, None, None,
                                                  ctypes.byref(ctypes.c_void_p())))


@pytest.mark.parametrize("n", [10, 12])
def test_long_circuits_on_one_tile(n):
    """One run of 4,000 and of 32,000 gates on a state of one register tile:
    8 times the gates take about 8 times as long (64 times where every segment
    looks through the whole run)."""
    short, long = [_plan_seconds([W.random_gates_n12(seed=n, n=n, ngates=g)]) for g in (4000, 32000)]
    assert long <= 24 * short, (short, long)


def test_one_shot_batches_of_small_states_need_no_plan():
    """States that fit a workgroup's LDS run gate by gate when the batch runs
    once: a plan as kept batches have costs several times their whole call."""
    circs = [W.random_gates_n12(seed=i, n=8 + i % 5, ngates=150) for i in range(400)]
    states, gates, offsets, params = _arguments(circs)
    once = _seconds(lambda: sv._L.sv_apply_circuits_batched(states, len(circs), gates, offsets, None, params, 0, None))
    kept = _plan_seconds(circs)
    assert once <= 0.5 * kept, (once, kept)
