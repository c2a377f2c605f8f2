"""dprc_trace_launches records every launch of a call, also where one step of a call
takes several: each with its own kind and events."""

import ctypes

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_24879_amd import dprc
    dprc.lib()
    return dprc


def _trace(D, fn, capacity=32):
    """(kinds, milliseconds) of the launches of fn()."""
    events = [torch.cuda.Event(enable_timing=True) for _ in range(2 * capacity)]
    for e in events:
        e.record()                                     # torch creates an event when it is first recorded
    torch.cuda.synchronize()
    ptrs = (ctypes.c_void_p * len(events))(*[e.cuda_event for e in events])
    kinds, count = (ctypes.c_int32 * capacity)(), ctypes.c_int32(0)
    D.dprc_trace_launches(ctypes.cast(ptrs, ctypes.c_void_p), ctypes.cast(kinds, ctypes.c_void_p), capacity,
                          ctypes.cast(ctypes.byref(count), ctypes.c_void_p))
    try:
        fn()
    finally:
        n = count.value
        D.dprc_trace_launches(None, None, 0, None)
    torch.cuda.synchronize()
    return [D.KERNEL_NAMES[k] for k in kinds[:n]], [events[2 * j].elapsed_time(events[2 * j + 1]) for j in range(n)]


def _f64(*x):
    return torch.tensor(x, dtype=torch.float64, device="cuda")


def _one_by_one(j):
    """A layer of one token and one feature on either side: it takes element loads, which batched
    projections leave to a launch per layer."""
    return workloads.draw(1, 1, 1, 1, dtype="bf16", law="lognormal", seed=0, layer=j, device="cuda") + (j,)


CALLS = {
    "fold": (lambda D: D.dprc_pld_fold(torch.rand(80001, dtype=torch.float64, device="cuda"), 40001, _f64(0.1), _f64(0.1)),
             ["pld"] * 3),
    "fold, one workgroup": (lambda D: D.dprc_pld_fold(_f64(0.2, 0.3, 0.1), 1, _f64(0.1), _f64(0.1)), ["pld"]),
    "step": (lambda D: D.dprc_pld_step(1.0, 0.1, 0.01, 300), ["pld"] * 2),
    "envelope": (lambda D: D.dprc_envelope_middle(_f64(1.1), 4, 5, 3), ["envelope"] * 2),
    "element loads": (lambda D: D.dprc_norm_hutch([_one_by_one(j) for j in range(3)], 4, 1),
                      ["project"] * 3 + ["token_reduce", "sample_sum"]),
}


@pytest.mark.parametrize("call", CALLS)
def test_every_launch_is_recorded(D, call):
    fn, expected = CALLS[call]
    kinds, ms = _trace(D, lambda: fn(D))
    assert kinds == expected
    assert all(0.0 < t < 100.0 for t in ms)


def test_recording_stops_at_the_capacity(D):
    fn, expected = CALLS["element loads"]
    kinds, ms = _trace(D, lambda: fn(D), capacity=2)
    assert kinds == expected[:2] and all(t > 0.0 for t in ms)
