"""Host-side checks of libdprc that need no GPU: the library loads, exports every
entry point declared in include/dprc.h, and rejects bad arguments before it
enqueues anything (so these calls never reach a kernel)."""

import ctypes
import os
import re
import types

import pytest
import torch

from paper_2605_24879_amd import dprc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "dprc.h")

pytestmark = pytest.mark.skipif(not os.path.exists(dprc.LIB_PATH), reason="libdprc.so not built")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dprc_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = declared_functions()
    assert len(names) >= 11
    L = dprc.lib()
    for n in names:
        assert hasattr(L, n), n
    assert set(names) == set(dprc.EXPORTS)


def test_version_and_status_strings():
    assert "gfx950" in dprc.dprc_version()
    L = dprc.lib()
    for code in range(5):
        assert L.dprc_status_string(code).decode().startswith("DPRC_")


def _fake_layer(**kw):
    # device pointers are never dereferenced on the host; these calls fail validation first
    base = dict(A=0x10000, E=0x20000, B=2, T=64, d=64, p=48, lda=64, lde=48, dtype=dprc.BF16, layer_id=0)
    base.update(kw)
    return dprc.Layer(base["A"], base["E"], base["B"], base["T"], base["d"], base["p"], base["lda"],
                      base["lde"], base["dtype"], base["layer_id"])


def _hutch(layer, k=4, ws_bytes=0, ws=0x30000, n2=0x40000, side=0, probe=0, nl=1):
    L = dprc.lib()
    arr = (dprc.Layer * 1)(layer)
    return L.dprc_norm_hutch(arr, nl, k, probe, 0, side, n2, None, 0, ws, ws_bytes, None)


def test_hutch_argument_validation():
    L = dprc.lib()
    assert L.dprc_norm_hutch(None, 1, 4, 0, 0, 0, 0x40000, None, 0, 0x30000, 1 << 30, None) == 1
    assert _hutch(_fake_layer(), nl=0, ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(B=0), ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(T=-1), ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(lda=32), ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(dtype=7), ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(A=0), ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(), k=0, ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(), k=257, ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(), n2=0, ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(), side=5, ws_bytes=1 << 30) == 1
    assert _hutch(_fake_layer(), probe=9, ws_bytes=1 << 30) == 1
    # element alignment (any row stride is accepted; 16-byte aligned rows take the vector path)
    assert _hutch(_fake_layer(A=0x10001), ws_bytes=1 << 30) == 2
    assert _hutch(_fake_layer(E=0x20003), ws_bytes=1 << 30) == 2
    assert _hutch(_fake_layer(dtype=dprc.F32, A=0x10002), ws_bytes=1 << 30) == 2
    # workspace
    need = L.dprc_norm_hutch_workspace((dprc.Layer * 1)(_fake_layer()), 1, 4, dprc.PROBE_RADEMACHER, 0)
    assert need > 0
    assert _hutch(_fake_layer(), ws_bytes=need - 1) == 3
    assert _hutch(_fake_layer(), ws=0, ws_bytes=need) == 1
    assert _hutch(_fake_layer(), ws=0x30010, ws_bytes=need) == 1        # not 256-byte aligned


def test_gaussian_probe_validation():
    L = dprc.lib()
    arr = (dprc.Layer * 1)(_fake_layer())
    G = dprc.PROBE_GAUSSIAN
    # Gaussian probes are dense columns: k <= 32, and the workspace holds them
    assert _hutch(_fake_layer(), k=33, probe=G, ws_bytes=1 << 30) == 2
    assert L.dprc_norm_hutch_workspace(arr, 1, 33, G, 0) == 0
    assert L.dprc_norm_hutch_workspace(arr, 1, 4, 9, 0) == 0
    for dt in (dprc.BF16, dprc.F32):
        a1 = (dprc.Layer * 1)(_fake_layer(dtype=dt))
        g = L.dprc_norm_hutch_workspace(a1, 1, 32, G, 0)
        r = L.dprc_norm_hutch_workspace(a1, 1, 32, dprc.PROBE_RADEMACHER, 0)
        assert g > r > 0
        assert _hutch(_fake_layer(dtype=dt), k=32, probe=G, ws_bytes=g - 1) == 3
    # values export
    assert L.dprc_probe_gaussian(1, 0, 100, 4, None, None) == 1
    assert L.dprc_probe_gaussian(1, 0, 0, 4, 0x40000, None) == 1
    assert L.dprc_probe_gaussian(1, 0, 100, 0, 0x40000, None) == 1
    assert L.dprc_probe_gaussian(1, 0, 100, 257, 0x40000, None) == 1
    assert L.dprc_probe_gaussian(1, 0, 100, 4, 0x40002, None) == 1


def test_hutchpp_and_accumulate_validation():
    L = dprc.lib()
    arr = (dprc.Layer * 1)(_fake_layer())
    assert L.dprc_norm_hutchpp_workspace(arr, 1, 16, 32, 0) > 0
    assert L.dprc_norm_hutchpp(arr, 1, 33, 4, 0, 0, 0x40000, None, 0, 0x30000, 1 << 30, None) == 1
    assert L.dprc_norm_hutchpp(arr, 1, 4, 0, 0, 0, 0x40000, None, 0, 0x30000, 1 << 30, None) == 1
    assert L.dprc_norm_hutchpp(arr, 1, 49, 4, 0, 0, 0x40000, None, 0, 0x30000, 1 << 30, None) == 1  # s > p
    assert L.dprc_norm_hutchpp(arr, 1, 4, 4, 0, 0, 0x40000, None, 0, 0x30000, 0, None) == 3
    # a sketched width of 2^22 rows needs a QR tree deeper than eight levels
    wide = (dprc.Layer * 1)(_fake_layer(p=1 << 22, lde=1 << 22))
    assert L.dprc_norm_hutchpp(wide, 1, 32, 4, 0, 0, 0x40000, None, 0, 0x30000, 1 << 40, None) == 2
    lay = _fake_layer()
    assert L.dprc_clip_accumulate(ctypes.byref(lay), None, 0x50000, 48, 0, None, 0, None) == 1
    assert L.dprc_clip_accumulate(ctypes.byref(lay), 0x60000, 0x50000, 47, 0, None, 0, None) == 1
    # several layers in one call: validated before any launch
    two = (dprc.Layer * 2)(_fake_layer(), _fake_layer())
    ptrs = (ctypes.c_void_p * 2)(0x50000, 0x58000)
    lds = (ctypes.c_int64 * 2)(48, 48)
    acc = L.dprc_clip_accumulate_layers
    assert acc(two, 2, None, ptrs, lds, 0, None) == 1                      # no clip factors
    assert acc(two, 2, 0x60000, None, lds, 0, None) == 1                   # no gradient list
    assert acc(two, -1, 0x60000, ptrs, lds, 0, None) == 1
    assert acc(two, 2, 0x60000, ptrs, (ctypes.c_int64 * 2)(48, 47), 0, None) == 1   # ldg < p
    assert acc(two, 2, 0x60000, (ctypes.c_void_p * 2)(0x50000, None), lds, 0, None) == 1
    other_b = (dprc.Layer * 2)(_fake_layer(), _fake_layer(B=3))
    assert acc(other_b, 2, 0x60000, ptrs, lds, 0, None) == 1               # one batch
    f32 = (dprc.Layer * 2)(_fake_layer(), _fake_layer(dtype=dprc.F32, A=0x10000))
    assert acc(f32, 2, 0x60000, ptrs, lds, 0, None) == 2
    assert acc(two, 0, 0x60000, ptrs, lds, 0, None) == 0                   # nothing to do


def test_clip_noise_bits_validation():
    L = dprc.lib()
    assert L.dprc_clip_scale(0x1000, 4, 0.0, 0x2000, None) == 1
    assert L.dprc_clip_scale(0x1000, 4, float("inf"), 0x2000, None) == 1
    assert L.dprc_clip_scale(None, 4, 1.0, 0x2000, None) == 1
    assert L.dprc_clip_scale(0x1000, 0, 1.0, 0x2000, None) == 1
    assert L.dprc_add_noise(0x1000, -1, 0.8, 1.0, 0, 0, None) == 1
    assert L.dprc_add_noise(0x1000, 10, -0.1, 1.0, 0, 0, None) == 1
    assert L.dprc_add_noise(0x1000, 10, float("nan"), 1.0, 0, 0, None) == 1
    assert L.dprc_add_noise(0x1000, 10, 0.8, 0.0, 0, 0, None) == 1
    assert L.dprc_add_noise(0x1002, 10, 0.8, 1.0, 0, 0, None) == 2
    assert L.dprc_add_noise(None, 0, 0.8, 1.0, 0, 0, None) == 0          # empty: nothing to do
    assert L.dprc_probe_bits(0, 0, 0, 0, 0, 4, 0x1000, None) == 1
    assert L.dprc_probe_bits(0, 0, 0, 0, 32, 0, 0x1000, None) == 1
    assert L.dprc_probe_bits(3, 0, 0, 0, 32, 4, 0x1000, None) == 1


def test_private_adamw_validation():
    L = dprc.lib()
    hp = dprc.AdamWParams(1e-3, 0.9, 0.999, 1e-8, 0.0, 1)
    T, M, V, G = 0x10000, 0x20000, 0x30000, 0x40000

    def call(ldt=8, ldg=8, d=4, p=8, sigma=1.0, C=1.0, inv=0.25, h=hp, w=None, ldw=0, theta=T):
        return L.dprc_private_adamw(theta, M, V, ldt, G, ldg, d, p, sigma, C, 0, 0, inv, ctypes.byref(h) if h else None,
                                    w, ldw, None)
    assert call(theta=0) == 1
    assert call(ldt=7) == 1
    assert call(ldg=7) == 1
    assert call(sigma=-1.0) == 1
    assert call(C=0.0) == 1
    assert call(inv=float("inf")) == 1
    assert call(h=None) == 1
    assert call(w=0x50000, ldw=3) == 1
    assert call(theta=T + 2) == 1                 # fp32 pointers 4-byte aligned
    for bad in (dprc.AdamWParams(-1.0, 0.9, 0.999, 1e-8, 0.0, 1), dprc.AdamWParams(1e-3, 1.0, 0.999, 1e-8, 0.0, 1),
                dprc.AdamWParams(1e-3, 0.9, 0.999, 0.0, 0.0, 1), dprc.AdamWParams(1e-3, 0.9, 0.999, 1e-8, 0.0, 0)):
        assert call(h=bad) == 1
    assert call(d=0) == 0                         # nothing to do, nothing enqueued


def test_hutch_clip_validation():
    L = dprc.lib()
    arr = (dprc.Layer * 1)(_fake_layer())

    def call(C=1.0, c=0x50000, ws_bytes=1 << 30):
        return L.dprc_norm_hutch_clip(arr, 1, 4, 0, 0, 0, C, 0x40000, c, None, 0, 0x30000, ws_bytes, None)
    assert call(C=0.0) == 1
    assert call(C=float("inf")) == 1
    assert call(c=None) == 1
    need = L.dprc_norm_hutch_workspace(arr, 1, 4, 0, 0)
    assert call(ws_bytes=need - 1) == 3


def test_batched_workspaces_grow_with_the_groups_they_hold():
    # Hutchinson over bf16 layers with their own activations: up to 32 groups per batch keep
    # their own projected Y (hi + lo planes, 16 columns, T rounded up to 64) besides the
    # shared scratch, and every group of the call keeps its tile sums until the per-sample
    # sums at the end (one 256-byte-aligned slice each here); Hutch++ keeps up to eight
    # layers' buffers.  Workspace queries run on the host.
    L = dprc.lib()
    B, T, k = 2, 100, 16
    layers = [_fake_layer(A=0x100000 + 0x10000 * j, E=0x900000 + 0x10000 * j, B=B, T=T, layer_id=j)
              for j in range(40)]
    arr = (dprc.Layer * 40)(*layers)
    ws = lambda n, probe=dprc.PROBE_RADEMACHER: L.dprc_norm_hutch_workspace(arr, n, k, probe, 0)
    y = 2 * 16 * B * 128 * 2
    assert ws(10) >= ws(1) + 8 * y
    assert ws(32) >= ws(2) + 30 * y
    assert ws(40) == ws(32) + 8 * 256                 # a second batch reuses the first one's space
    # a call with one byte less is refused before anything is enqueued
    n2 = 0x40000
    assert L.dprc_norm_hutch(arr, 10, k, dprc.PROBE_RADEMACHER, 0, 0, n2, None, 0, 0x30000, ws(10) - 1,
                             None) == 3
    hpp = lambda n: L.dprc_norm_hutchpp_workspace(arr, n, 4, 8, 0)
    assert hpp(8) > hpp(4) > hpp(1) > 0
    assert hpp(16) == hpp(8)


def test_static_scratch_entry_point_limits():
    # dprc_norm_hutch_clip_static validates like dprc_norm_hutch_clip, and a call whose
    # workspace query exceeds the static scratch is refused before anything is enqueued
    L = dprc.lib()
    small = (dprc.Layer * 1)(_fake_layer())

    def call(arr, n=1, C=1.0, c=0x50000):
        return L.dprc_norm_hutch_clip_static(arr, n, 4, 0, 0, 0, C, 0x40000, c, None, 0, None)
    assert call(small, C=0.0) == 1
    assert call(small, c=None) == 1
    assert call(small, n=0) == 1
    limit = 256 << 20
    big = (dprc.Layer * 1)(_fake_layer(B=64, T=65536, d=4096, p=4096, lda=4096, lde=4096))
    assert L.dprc_norm_hutch_workspace(big, 1, 256, 0, 0) > limit
    assert L.dprc_norm_hutch_clip_static(big, 1, 256, 0, 0, 0, 1.0, 0x40000, 0x50000, None, 0, None) == 5
    assert L.dprc_status_string(5).decode().startswith("DPRC_ERROR_SCRATCH_LIMIT")


def test_static_scratch_holds_what_needs_no_more():
    # split partials are reserved for the splits that a batch of layers runs with, in both forms of
    # a Gaussian call: no form's need exceeds the query.  (An unaligned workspace is refused
    # with 1, after a too small one with 3, so nothing is enqueued here.)
    L = dprc.lib()
    limit = 256 << 20

    def layers(n, share, **kw):
        return (dprc.Layer * n)(*[_fake_layer(A=0x1000000 + 0x10000 * (j // share), E=0x90000000 + 0x10000 * j,
                                              layer_id=j, **kw) for j in range(n)])
    # 32 Gaussian layers: 1024 pairs of samples and tiles and more, so no splits
    arr = layers(32, 1, B=5, T=512, d=6528, p=2048, lda=6528, lde=2048)
    need = L.dprc_norm_hutch_workspace(arr, 32, 32, dprc.PROBE_GAUSSIAN, 0)
    assert need < 32 << 20
    for size in (need, need - 1, limit):
        assert L.dprc_norm_hutch(arr, 32, 32, dprc.PROBE_GAUSSIAN, 0, 0, 0x40000, None, 0, 0x30010, size, None) == 1
    assert L.dprc_norm_hutch(arr, 32, 32, dprc.PROBE_GAUSSIAN, 0, 0, 0x40000, None, 0, 0x30010, need // 64, None) == 3
    # sign probes: a batch of 32 narrow groups of the stack reserves the splits that it runs with
    stack = []
    for j in range(200):
        d, p = ((19183, 110)[j // 3 % 2], (274, 1351)[j % 2])
        stack.append(_fake_layer(A=0x1000000 + 0x10000 * (j // 3), E=0x90000000 + 0x10000 * j, B=9, T=708, d=d, p=p,
                                 lda=d, lde=p, layer_id=j))
    assert L.dprc_norm_hutch_workspace((dprc.Layer * 200)(*stack), 200, 128, dprc.PROBE_RADEMACHER, 2) <= limit


def test_accountant_entry_points_validation():
    L = dprc.lib()
    P = 0x10000
    assert L.dprc_envelope_bins(P, 0, 0.0, 1.0, P, P, None) == 1          # no bins
    assert L.dprc_envelope_bins(P, 4, 1.0, 1.0, P, P, None) == 1          # empty range
    assert L.dprc_envelope_bins(None, 4, 0.0, 1.0, P, P, None) == 1
    assert L.dprc_pld_step_workspace(0) == 0
    need = L.dprc_pld_step_workspace(1000)
    assert need >= 2000 * 8
    args = lambda **kw: dict(dict(sigma=1.0, p=0.1, h=1e-3, n=1000, ybar=None, w=None, nb=0, ws_bytes=need), **kw)

    def step(a):
        return L.dprc_pld_step(a["sigma"], a["p"], a["h"], a["n"], a["ybar"], a["w"], a["nb"], P, P + 8192,
                               0x40000, a["ws_bytes"], None)
    assert step(args(sigma=0.0)) == 1
    assert step(args(p=0.0)) == 1
    assert step(args(p=1.5)) == 1
    assert step(args(h=-1.0)) == 1
    assert step(args(nb=3)) == 1                                             # bins without arrays
    assert step(args(ws_bytes=need - 1)) == 3
    assert L.dprc_pld_fold(P, 10, P, P, P, P, None) == 1                     # even L
    assert L.dprc_pld_delta(P, 11, 1e-3, P, P, 0, P, None) == 1              # no eps
    assert L.dprc_pld_delta(P, 11, 0.0, P, P, 3, P, None) == 1               # h = 0


def test_tensors_that_are_not_on_a_gpu_are_refused(monkeypatch):
    # the binding takes the stream of a tensor's device: a host tensor has none, also where a GPU is current
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 0, raising=False)
    monkeypatch.setattr(dprc, "_raw_stream", lambda index: 0, raising=False)
    assert dprc._stream(torch.device("cuda")).value is None and dprc._stream(torch.device("cuda", 0)).value is None
    with pytest.raises(ValueError):
        dprc._stream(torch.device("cpu"))
    monkeypatch.setattr(dprc, "_lib", None)            # nothing may be enqueued: no entry point is looked up
    monkeypatch.setattr(dprc, "lib", lambda: types.SimpleNamespace(
        **{n: (lambda *a, n=n: 1 << 20 if n.endswith("_workspace") else pytest.fail(n)) for n in dprc.EXPORTS}))
    host = torch.zeros(4, 8)
    for call in (lambda: dprc.dprc_clip_scale(host[0], 1.0), lambda: dprc.dprc_add_noise(host, 1.0, 1.0, 0, 0),
                 lambda: dprc.dprc_private_adamw(host, host.clone(), host.clone(), host.clone(), 1.0, 1.0, 0, 0, 1.0,
                                                 1e-3, 0.9, 0.999, 1e-8, 0.0, 1),
                 lambda: dprc.dprc_envelope_middle(host[0].double(), 4, 3, 5), lambda: dprc.dprc_chi2_cdf(host[0].double(), 4),
                 lambda: dprc.dprc_probe_bits(0, 0, 0, 0, 32, 4, out=torch.zeros(4, 1, dtype=torch.int32)),
                 lambda: dprc.dprc_probe_gaussian(0, 0, 8, 4, out=host), lambda: dprc.dprc_pld_step(1.0, 0.1, 0.1, 3, device="cpu"),
                 lambda: dprc.dprc_pld_step(1.0, 0.1, 0.1, 3, device="cpu:0"),
                 lambda: dprc.dprc_norm_hutch([(host[None], host[None], 0)], 4, 0)):
        with pytest.raises(ValueError):
            call()
