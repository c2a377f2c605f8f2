"""GPU parity of libdprc against the CPU oracle on identical seeded inputs.

Sizes span several tiles with ragged tails (token counts, widths and probe
counts that are not multiples of the kernels' tiles).  Tolerances: probe bits
bit-exact; squared-norm estimates 1e-3 relative; clipped gradients 2e-3
relative Frobenius; noise 1e-5 * sigma * C absolute on the added term.
"""

import math

import numpy as np
import pytest
import torch

from oracle import philox
from oracle import estimators as est
import workloads

pytestmark = pytest.mark.gpu

NORM_RTOL = 1e-3
GRAD_RTOL = 2e-3


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_24879_amd import dprc
    dprc.lib()
    return dprc


def _draw(B, T, d, p, dtype="bf16", law="lognormal", layer=0, seed=0, **kw):
    return workloads.draw(B, T, d, p, dtype=dtype, law=law, seed=seed, layer=layer, device="cuda", **kw)


def _np(x):
    return est.as_f64(x)


def _rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return np.abs(a - b) / np.maximum(np.abs(b), 1e-300)


def _hadamard_words(m, k):
    H = philox.hadamard_matrix(m, k)           # +-1
    bits = (H < 0).astype(np.uint64).T         # [k, m]
    nw = (m + 31) // 32
    out = np.zeros((k, nw), dtype=np.uint64)
    for u in range(m):
        out[:, u // 32] |= bits[:, u] << np.uint64(u % 32)
    return out.astype(np.uint32)


# ---- probe bits --------------------------------------------------------------------------

@pytest.mark.parametrize("seed,layer,stream,m,k", [
    (0, 0, 0, 48, 4), (0, 3, 1, 2048, 16), (12345678901234, 7, 0, 45, 3), (5, 112, 0, 128256, 2),
    (2**64 - 1, 2**32 - 1, 2, 100, 33), (9, 1, 0, 1, 1), (9, 1, 0, 130, 1)])
def test_probe_bits_bitexact(D, seed, layer, stream, m, k):
    got = D.dprc_probe_bits(D.PROBE_RADEMACHER, seed, layer, stream, m, k).cpu().numpy().view(np.uint32)
    ref = philox.rademacher_words(seed, layer, stream, m, k)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("m,k", [(64, 64), (48, 64), (100, 7)])
def test_hadamard_bits_bitexact(D, m, k):
    got = D.dprc_probe_bits(D.PROBE_HADAMARD, 0, 0, 0, m, k).cpu().numpy().view(np.uint32)
    assert np.array_equal(got, _hadamard_words(m, k))


@pytest.mark.parametrize("seed,layer,m,k", [
    (0, 0, 48, 4), (7, 3, 130, 33), (2**64 - 1, 2**32 - 1, 1, 1), (11, 5, 4097, 2)])
def test_gaussian_probe_values(D, seed, layer, m, k):
    # fp32 Box-Muller on the GPU against the fp64 transform of the same Philox words
    got = D.dprc_probe_gaussian(seed, layer, m, k).cpu().numpy().astype(np.float64).T
    ref = philox.gaussian_probe_matrix(seed, layer, m, k)
    assert got.shape == ref.shape
    assert np.all(np.abs(got - ref) <= 2e-6 * np.maximum(1.0, np.abs(ref)))


# ---- Hutchinson ---------------------------------------------------------------------------

@pytest.mark.parametrize("B,T,d,p,k,side", [
    (3, 200, 300, 260, 16, 0),     # ragged tokens / widths, 3 x 3 tiles
    (2, 130, 72, 520, 5, 1),       # side IN, odd k
    (2, 96, 520, 72, 33, 2),       # AUTO -> IN (d > p), 3 column blocks
    (1, 1, 8, 8, 1, 0),            # a single token
    (2, 64, 64, 48, 4, 0),         # the tiny workload's shape in bf16
])
def test_hutch_parity_bf16(D, B, T, d, p, k, side):
    A, E = _draw(B, T, d, p, layer=1)
    n2l = torch.zeros(1, B, device="cuda")
    n2 = D.dprc_norm_hutch([(A, E, 1)], k, 42, side=side, n2_layers=n2l)
    ref = est.hutch_layer(_np(A), _np(E), k, 42, 1, side=side)
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)
    assert torch.equal(n2, n2l[0])


@pytest.mark.parametrize("B,T,d,p,k,side,dtype", [
    (3, 200, 300, 260, 16, 0, "bf16"),    # ragged tokens / widths
    (2, 130, 72, 1100, 5, 1, "bf16"),     # side IN, odd k, wide reduced operand
    (2, 96, 1100, 72, 32, 2, "bf16"),     # AUTO -> IN, 1100 sketched columns (3 stages), k at its maximum
    (1, 1, 8, 8, 1, 0, "bf16"),           # a single token
    (2, 64, 64, 48, 4, 0, "f32"),
    (2, 100, 130, 70, 32, 1, "f32"),
])
def test_hutch_gaussian_parity(D, B, T, d, p, k, side, dtype):
    A, E = _draw(B, T, d, p, dtype=dtype, layer=6)
    n2 = D.dprc_norm_hutch([(A, E, 4)], k, 77, side=side, probe=D.PROBE_GAUSSIAN)
    ref = est.hutch_layer(_np(A), _np(E), k, 77, 4, side=side, probe="gaussian")
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)


@pytest.mark.parametrize("n", [5, 37])
def test_hutch_gaussian_batched_launches(D, n):
    # Gaussian layers in one call: one probe launch, batched projections and reductions (37
    # layers: two batches), against calls of one layer bit for bit; and in a workspace
    # that only holds the unbatched form, with the same results
    B, T, k = 2, 130, 20
    pairs = [_draw(B, T, 40 + 8 * (j % 3), 56 + 100 * (j % 4), layer=600 + j) + (j,) for j in range(n)]
    need = D.dprc_norm_hutch_workspace(pairs, k, probe=D.PROBE_GAUSSIAN)
    per = torch.zeros(n, B, device="cuda")
    n2, c = D.dprc_norm_hutch_clip(pairs, k, 5, 0.5, probe=D.PROBE_GAUSSIAN, n2_layers=per)
    solo = torch.stack([D.dprc_norm_hutch([q], k, 5, probe=D.PROBE_GAUSSIAN) for q in pairs])
    assert torch.equal(per, solo)
    for j in (0, n - 1):
        A, E, _ = pairs[j]
        assert np.all(_rel(per[j].cpu().numpy(), est.hutch_layer(_np(A), _np(E), k, 5, j, probe="gaussian")) < NORM_RTOL)
    arr, nl, _, dev = D._layers(pairs)
    small = need - 2 * k * 128 * 2               # one layer's probe columns short of batched launches
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    m2, mc, mper = torch.zeros_like(n2), torch.zeros_like(c), torch.zeros_like(per)
    status = D.lib().dprc_norm_hutch_clip(arr, nl, k, D.PROBE_GAUSSIAN, 5, 0, 0.5, m2.data_ptr(), mc.data_ptr(),
                                          mper.data_ptr(), 0, ws.data_ptr(), small, D._stream(dev))
    assert status == D.SUCCESS
    assert torch.equal(m2, n2) and torch.equal(mc, c) and torch.equal(mper, per)


@pytest.mark.parametrize("n,B,T,d,p,k", [
    (8, 32, 1024, 8, 72, 1),        # 256 pairs of samples and tiles: four token splits of 4 stages become one
    (3, 90, 4096, 8, 40, 1),        # 270 pairs, 64 stages: splits of at least 16 stages
    (32, 5, 512, 6528, 128, 32),    # 1024 pairs and more: none
])
def test_hutch_gaussian_forms_agree_where_splits_are_limited(D, n, B, T, d, p, k):
    # batched launches, the smaller workspace's launches per group and the static scratch all
    # split the tokens alike, so their estimates agree bit for bit (few entries per sample: a
    # different split would show)
    pairs = [_draw(B, T, d, p, layer=700 + j) + (j,) for j in range(n)]
    arr, nl, _, dev = D._layers(pairs)
    need = D.dprc_norm_hutch_workspace(pairs, k, probe=D.PROBE_GAUSSIAN)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    outs = []
    for form in ("batched", "per group", "static"):
        n2, c, per = (torch.full(s, -1.0, device="cuda") for s in ((B,), (B,), (n, B)))
        out = (n2.data_ptr(), c.data_ptr(), per.data_ptr(), 0)
        if form == "static":
            status = D.lib().dprc_norm_hutch_clip_static(arr, nl, k, D.PROBE_GAUSSIAN, 5, 0, 0.5, *out, D._stream(dev))
        else:
            status = D.lib().dprc_norm_hutch_clip(arr, nl, k, D.PROBE_GAUSSIAN, 5, 0, 0.5, *out, ws.data_ptr(),
                                                  need - (form == "per group"), D._stream(dev))
        assert status == D.SUCCESS, form
        outs.append(torch.cat([n2, c, per.flatten()]))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    A, E, _ = pairs[1]
    ref = est.hutch_layer(_np(A[:2]), _np(E[:2]), k, 5, 1, probe="gaussian")
    assert np.all(_rel(outs[0][2 * B:].view(n, B)[1, :2].cpu().numpy(), ref) < NORM_RTOL)


def test_hutch_gaussian_multilayer_accumulate(D):
    # per-layer probes differ (layer id in the counter); the workspace is reused across layers
    A1, E1 = _draw(2, 300, 256, 200, layer=0)
    A2, E2 = _draw(2, 150, 136, 700, layer=1)
    n2 = torch.tensor([0.5, 1.0], device="cuda")
    n2l = torch.zeros(2, 2, device="cuda")
    D.dprc_norm_hutch([(A1, E1, 20), (A2, E2, 21)], 8, 3, probe=D.PROBE_GAUSSIAN, n2=n2, n2_layers=n2l,
                      accumulate=True)
    r1 = est.hutch_layer(_np(A1), _np(E1), 8, 3, 20, probe="gaussian")
    r2 = est.hutch_layer(_np(A2), _np(E2), 8, 3, 21, probe="gaussian")
    got = n2l.cpu().numpy()
    assert np.all(_rel(got[0], r1) < NORM_RTOL) and np.all(_rel(got[1], r2) < NORM_RTOL)
    assert np.all(_rel(n2.cpu().numpy(), np.array([0.5, 1.0]) + r1 + r2) < NORM_RTOL)


# ---- short fp32 samples -----------------------------------------------------------------------

@pytest.mark.parametrize("B,d,p", [(2, 64, 48), (11, 130, 37), (37, 3, 5), (9, 1030, 4100), (700, 72, 8)])
@pytest.mark.parametrize("T", [1, 3, 4, 5, 8, 9, 13, 16, 17])
def test_clip_accumulate_short_fp32_samples(D, B, T, d, p):
    # up to 16 tokens a slab holds several samples (8, 4 or 2); the last slab is ragged, samples with
    # factor 0 hold infinities, and the result is written and added to
    A, E = _draw(B, T, d, p, dtype="f32", layer=9)
    c = torch.rand(B, device="cuda")
    c[1::4] = 0.0
    ref = est.clip_accumulate(_np(A), _np(E), _np(c))
    A[1::4] = float("inf")
    E[1::4] = float("nan")
    g = D.dprc_clip_accumulate(A, E, c)
    base = torch.randn(d, p + 3, device="cuda")
    h = base.clone()
    D.dprc_clip_accumulate(A, E, c, grad=h[:, 2:2 + p], accumulate=True)
    norm = np.linalg.norm(ref)
    assert np.linalg.norm(g.cpu().numpy() - ref) < 2e-6 * norm
    err = h[:, 2:2 + p].double().cpu().numpy() - base[:, 2:2 + p].double().cpu().numpy() - ref
    assert np.linalg.norm(err) < 2e-6 * (norm + base.norm().item())
    assert torch.equal(h[:, :2], base[:, :2]) and torch.equal(h[:, 2 + p:], base[:, 2 + p:])


@pytest.mark.parametrize("B,T,d,p,k", [
    (600, 1, 70, 9, 5),          # one wave in both kernels, 38 workgroups of rows of several samples
    (523, 16, 40, 64, 17),       # whole blocks of 16 rows, the widest one-wave projection
    (520, 17, 130, 65, 33),      # two waves in both, rows of several samples
    (60, 130, 600, 128, 70),     # two waves, 10 x 2 tiles
    (600, 257, 8, 129, 4),       # eight waves again
])
@pytest.mark.parametrize("probe", ["rademacher", "gaussian", "hutchpp"])
def test_norms_of_many_short_fp32_samples(D, B, T, d, p, k, probe):
    A, E = _draw(B, T, d, p, dtype="f32", layer=3)
    rows = [0, 1, B // 2, B - 1]
    An, En = _np(A[rows]), _np(E[rows])
    if probe == "hutchpp":
        n2, ref = D.dprc_norm_hutchpp([(A, E, 2)], 4, k, 6), est.hutchpp_layer(An, En, 4, k, 6, 2)
    else:
        k = min(k, 32) if probe == "gaussian" else k
        code = D.PROBE_GAUSSIAN if probe == "gaussian" else D.PROBE_RADEMACHER
        n2, ref = D.dprc_norm_hutch([(A, E, 2)], k, 6, probe=code), est.hutch_layer(An, En, k, 6, 2, probe=probe)
    assert np.all(_rel(n2[rows].cpu().numpy(), ref) < 2e-5)


# ---- routes of batched bf16 launches -----------------------------------------------------------

@pytest.mark.parametrize("probe,k", [("rademacher", 48), ("gaussian", 9), ("gaussian", 32)])
def test_batched_layers_of_every_kind_match_calls_of_one(D, probe, k):
    # one call over layers whose projections take element loads (fewer than 8 elements), any
    # alignment, rows of one 512-column stage and more than one
    code = D.PROBE_GAUSSIAN if probe == "gaussian" else D.PROBE_RADEMACHER
    B, T = 2, 2
    widths = [(3, 1), (90, 1), (40, 64), (56, 512), (9, 513), (24, 1030), (5, 2)]
    pairs = [_draw(B, T, d, p, layer=800 + j) + (j,) for j, (d, p) in enumerate(widths)]
    per = torch.zeros(len(pairs), B, device="cuda")
    D.dprc_norm_hutch(pairs, k, 5, probe=code, n2_layers=per)
    for j, q in enumerate(pairs):
        assert torch.equal(per[j], D.dprc_norm_hutch([q], k, 5, probe=code)), widths[j]
        ref = est.hutch_layer(_np(q[0]), _np(q[1]), k, 5, j, probe=probe)
        assert np.all(_rel(per[j].cpu().numpy(), ref) < NORM_RTOL)


@pytest.mark.parametrize("B,T,d,k,probe", [
    (1500, 3, 384, 24, "rademacher"),     # 4500 workgroups of a tile: launches of their own
    (1500, 3, 384, 24, "gaussian"),
    (1300, 70, 264, 8, "rademacher"),     # two stages, 16 columns
    (128, 2048, 896, 32, "rademacher"),   # 7 tiles in 4 pairs, 32 stages
    (128, 1985, 640, 32, "gaussian"),     # 5 tiles would leave 3 pairs half empty
    (128, 1984, 896, 40, "rademacher"),   # 31 stages
])
def test_batched_reductions_of_many_samples(D, B, T, d, k, probe):
    code = D.PROBE_GAUSSIAN if probe == "gaussian" else D.PROBE_RADEMACHER
    pairs = [_draw(B, T, d, 40 + 8 * j, layer=820 + j) + (j,) for j in range(2)]
    per = torch.zeros(2, B, device="cuda")
    n2 = D.dprc_norm_hutch(pairs, k, 5, probe=code, n2_layers=per)
    rows = [0, B // 2, B - 1]
    for A, E, j in pairs:
        ref = est.hutch_layer(_np(A[rows]), _np(E[rows]), k, 5, j, probe=probe)
        assert np.all(_rel(per[j][rows].cpu().numpy(), ref) < NORM_RTOL)
    assert np.all(_rel(n2.cpu().numpy(), per.sum(0).cpu().numpy()) < 1e-6)


@pytest.mark.parametrize("k", [193, 225, 226])
def test_sign_columns_in_few_and_many_workgroups(D, k):
    # 256 padded columns: from 257 workgroups on the registers are held to two of them per CU where
    # the LDS has room for two (up to 225 columns)
    A, E = _draw(40, 130, 24, 1100, layer=840)
    n2 = D.dprc_norm_hutch([(A, E, 3)], k, 8)
    few = torch.cat([D.dprc_norm_hutch([(A[i:i + 4], E[i:i + 4], 3)], k, 8) for i in range(0, 40, 4)])
    assert np.all(_rel(n2.cpu().numpy(), few.cpu().numpy()) < 1e-6)
    ref = est.hutch_layer(_np(A[-2:]), _np(E[-2:]), k, 8, 3)
    assert np.all(_rel(n2[-2:].cpu().numpy(), ref) < NORM_RTOL)


@pytest.mark.parametrize("s,r", [(4, 5), (5, 200), (16, 33), (32, 64)])
def test_hutchpp_expansions_of_one_and_four_waves(D, s, r):
    # 2 blocks of rows per sample: 1200 workgroups of one wave, 120 of four
    A, E = _draw(600, 9, 24, 200, layer=830)
    n2 = D.dprc_norm_hutchpp([(A, E, 3)], s, r, 8)
    few = D.dprc_norm_hutchpp([(A[:60], E[:60], 3)], s, r, 8)
    assert torch.equal(n2[:60], few)
    ref = est.hutchpp_layer(_np(A[-2:]), _np(E[-2:]), s, r, 8, 3)
    assert np.all(_rel(n2[-2:].cpu().numpy(), ref) < NORM_RTOL)


# ---- rows at any 2-byte alignment -----------------------------------------------------------

def _in_nans(X, pad, lead):
    """The same values as a view into storage whose other elements are all NaN: rows `pad`
    elements apart beyond their width, the first one `lead` elements in, the last one ending
    with the storage."""
    B, T, n = X.shape
    ld = n + pad
    store = torch.full((lead + B * T * ld - pad,), float("nan"), dtype=X.dtype, device=X.device)
    view = store.as_strided((B, T, n), (T * ld, ld, 1), lead)
    view.copy_(X)
    return view


@pytest.mark.parametrize("B,T,d,p,k,pads,lead", [
    (1, 1, 1, 1, 2, (0, 0), 0),           # fewer than 8 elements: element loads
    (2, 3, 3, 5, 4, (1, 2), 1),           # rows shorter than one 16-byte piece
    (3, 17, 8, 9, 16, (1, 0), 1),         # 16-byte widths on odd rows, one more than a piece
    (2, 65, 129, 513, 16, (0, 4), 3),     # one past the tiles of 128 and 512, T one past a stage
    (2, 100, 255, 1031, 33, (7, 1), 5),   # general projection body, 33 columns
    (1, 130, 777, 4099, 80, (0, 0), 1),   # 96 columns, several probe chunks
    (2, 4200, 24, 31, 20, (3, 8), 2),     # 32-row workgroups
])
@pytest.mark.parametrize("side", [0, 1])
def test_any_alignment_hutch_and_accumulate(D, B, T, d, p, k, pads, lead, side):
    A, E = _draw(B, T, d, p, layer=530)
    Av, Ev = _in_nans(A, pads[0], lead), _in_nans(E, pads[1], lead)
    n2 = D.dprc_norm_hutch([(Av, Ev, 3)], k, 6, side=side)
    ref = est.hutch_layer(_np(A), _np(E), k, 6, 3, side=side)
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)
    c = torch.linspace(0.5, 1.0, B, device="cuda")
    g = D.dprc_clip_accumulate(Av, Ev, c)
    refg = est.clip_accumulate(_np(A), _np(E), c.cpu().numpy().astype(np.float64))
    assert np.linalg.norm(g.cpu().numpy() - refg) < 1e-5 * np.linalg.norm(refg)
    # two layers: the batched kernels; the gradients in one launch
    n2l = torch.zeros(2, B, device="cuda")
    D.dprc_norm_hutch([(Av, Ev, 3), (A, E, 3)], k, 6, side=side, n2_layers=n2l)
    assert np.all(_rel(n2l.cpu().numpy(), np.stack([ref, ref])) < NORM_RTOL)
    for q in D.dprc_clip_accumulate_layers([(Av, Ev), (A, E)], c):
        assert np.linalg.norm(q.cpu().numpy() - refg) < 1e-5 * np.linalg.norm(refg)


@pytest.mark.parametrize("B,T,d,p,s,r", [(2, 40, 33, 61, 8, 9), (1, 8200, 35, 131, 20, 12)])
def test_any_alignment_hutchpp_and_gaussian(D, B, T, d, p, s, r):
    # dense projections of unaligned rows (16- and 64-row workgroups), stored reductions
    A, E = _draw(B, T, d, p, law="student_t", layer=540)
    Av, Ev = _in_nans(A, 3, 1), _in_nans(E, 0, 1)
    for pairs in ([(Av, Ev, 2)], [(Av, Ev, 2), (A, E, 5)]):
        n2l = torch.zeros(len(pairs), B, device="cuda")
        D.dprc_norm_hutchpp(pairs, s, r, 7, n2_layers=n2l)
        for q, (_, _, j) in enumerate(pairs):
            assert np.all(_rel(n2l[q].cpu().numpy(), est.hutchpp_layer(_np(A), _np(E), s, r, 7, j)) < NORM_RTOL)
    n2 = D.dprc_norm_hutch([(Av, Ev, 2)], 11, 7, probe=D.PROBE_GAUSSIAN)
    assert np.all(_rel(n2.cpu().numpy(), est.hutch_layer(_np(A), _np(E), 11, 7, 2, probe="gaussian")) < NORM_RTOL)


# fp32 sums of n terms in any order: relative error at most n 2^-24 of the sum of magnitudes;
# with random signs that is about sqrt(n) 2^-24 of the result, and 3e-6 covers n = 1000 tenfold
F32_RTOL = 3e-6


@pytest.mark.parametrize("B,T,d,p,k,probe,pad", [
    (1, 1, 1, 1, 1, "rademacher", 0),           # one entry
    (2, 17, 3, 2, 5, "hadamard", 0),            # rows of less than one 16-byte piece
    (2, 33, 65, 513, 17, "rademacher", 3),      # one past the tiles of 64, 512 and 16; odd strides
    (1, 70, 130, 20000, 64, "rademacher", 0),   # two chunks of probe words, 64 columns
    (3, 40, 70, 131, 130, "rademacher", 1),     # more than 64 columns: three column groups
    (2, 36, 66, 258, 9, "gaussian", 0),
])
def test_f32_norm_edges(D, B, T, d, p, k, probe, pad):
    A, E = _draw(B, T, d, p, dtype="f32", layer=500, row_pad_a=pad, row_pad_e=pad)
    pid = {"rademacher": 0, "hadamard": 1, "gaussian": 2}[probe]
    n2, c = D.dprc_norm_hutch_clip([(A, E, 3)], k, 6, 0.5, probe=pid)
    ref = est.hutch_layer(_np(A), _np(E), k, 6, 3, probe=probe)
    assert np.all(_rel(n2.cpu().numpy(), ref) < 2 * F32_RTOL)
    assert torch.equal(c, D.dprc_clip_scale(n2, 0.5))


@pytest.mark.parametrize("B,T,d,p,pad,accumulate", [
    (1, 1, 1, 1, 0, False),
    (2, 33, 3, 70, 2, True),                    # narrow operand (element loads)
    (3, 31, 33, 34, 1, False),                  # one past a 32-wide tile, tokens short of a slab
    (2, 65, 1025, 1030, 3, True),               # 64-wide tiles, ragged, odd strides
    (2, 40, 2049, 2050, 0, False),              # 128-wide tiles, last ones 1 and 2 wide
    (5, 32, 130, 4, 0, False),
])
def test_f32_accumulate_edges(D, B, T, d, p, pad, accumulate):
    A, E = _draw(B, T, d, p, dtype="f32", layer=510, row_pad_a=pad, row_pad_e=pad)
    c = torch.linspace(0.0, 1.0, B + 1, device="cuda")[1:].contiguous()
    if B > 2:
        c[1] = 0.0
        E.select(0, 1).fill_(float("nan"))      # a dropped sample is not read into the sum
    grad = torch.full((d, p + 3), 0.5, device="cuda")[:, :p]
    D.dprc_clip_accumulate(A, E, c, grad=grad, accumulate=accumulate)
    ref = est.clip_accumulate(_np(A), _np(E), c.cpu().numpy().astype(np.float64)) + (0.5 if accumulate else 0.0)
    err = np.linalg.norm(grad.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err < F32_RTOL


@pytest.mark.parametrize("s,r", [(16, 7), (20, 40)])
def test_f32_hutchpp_mixed_column_blocks(D, s, r):
    # pass 3 projects dense and sign columns that share a block of 16
    A, E = _draw(2, 50, 90, 210, dtype="f32", law="student_t", layer=520)
    n2 = D.dprc_norm_hutchpp([(A, E, 1)], s, r, 2)
    assert np.all(_rel(n2.cpu().numpy(), est.hutchpp_layer(_np(A), _np(E), s, r, 2, 1)) < 1e-4)


# ---- layers sharing their activations (one token reduction over A) -------------------------

def _shared_a(B, T, d, ps, layer0=0):
    """Layers that read the same A (as q, k, v do), each with its own E."""
    A, _ = _draw(B, T, d, 8, layer=layer0)
    Es = [_draw(B, T, 8, p, layer=layer0 + 1 + j)[1] for j, p in enumerate(ps)]
    return A, Es


@pytest.mark.parametrize("B,T,d,ps,k,probe", [
    (2, 200, 300, (260, 72, 72), 16, "rademacher"),     # q, k, v-like widths (ragged)
    (3, 130, 136, (520, 520), 5, "rademacher"),         # gate/up-like pair, k not a multiple of 16
    (2, 700, 256, (200, 100, 64, 48, 30), 16, "rademacher"),   # five sharing layers -> groups of 4 and 1
    (2, 96, 64, (128, 40, 72), 100, "rademacher"),      # 3k > 256 columns -> groups of 2 and 1
    (2, 100, 64, (1100, 600), 16, "rademacher"),        # wide, unequal sketched sides in one group
    (2, 150, 520, (96, 260), 7, "gaussian"),
])
def test_hutch_shared_activations(D, B, T, d, ps, k, probe):
    A, Es = _shared_a(B, T, d, ps)
    pairs = [(A, E, 30 + j) for j, E in enumerate(Es)]
    pid = D.PROBE_GAUSSIAN if probe == "gaussian" else D.PROBE_RADEMACHER
    n2l = torch.zeros(len(Es), B, device="cuda")
    n2 = D.dprc_norm_hutch(pairs, k, 8, probe=pid, n2_layers=n2l)
    refs = [est.hutch_layer(_np(A), _np(E), k, 8, 30 + j, probe=probe) for j, E in enumerate(Es)]
    got = n2l.cpu().numpy()
    for j in range(len(Es)):
        assert np.all(_rel(got[j], refs[j]) < NORM_RTOL), j
    assert np.all(_rel(n2.cpu().numpy(), np.sum(refs, axis=0)) < NORM_RTOL)
    # same estimates as with a private copy of A per layer (no shared reduction)
    n2l_sep = torch.zeros_like(n2l)
    n2_sep = D.dprc_norm_hutch([(A.clone(), E, 30 + j) for j, E in enumerate(Es)], k, 8, probe=pid,
                               n2_layers=n2l_sep)
    assert np.all(_rel(got, n2l_sep.cpu().numpy()) < 1e-6)
    assert np.all(_rel(n2.cpu().numpy(), n2_sep.cpu().numpy()) < 1e-6)
    if k % 16 == 0:
        assert torch.equal(n2l, n2l_sep)


def test_hutch_shared_activations_mixed_sides(D):
    # AUTO: q (d == p) sketches OUT, k/v (d > p) sketch IN; only OUT layers share a reduction
    A, Es = _shared_a(2, 160, 256, (256, 64, 64))
    pairs = [(A, E, 40 + j) for j, E in enumerate(Es)]
    n2l = torch.zeros(3, 2, device="cuda")
    D.dprc_norm_hutch(pairs, 16, 2, side=2, n2_layers=n2l)
    for j, E in enumerate(Es):
        ref = est.hutch_layer(_np(A), _np(E), 16, 2, 40 + j, side=2)
        assert np.all(_rel(n2l[j].cpu().numpy(), ref) < NORM_RTOL), j


@pytest.mark.parametrize("k,probe", [(16, "rademacher"), (12, "hadamard"), (40, "rademacher"),
                                     (100, "rademacher")])
def test_hutch_many_groups_batched(D, k, probe):
    # 15 bf16 layers in 11 activation groups (one batch of up to 32): shared groups of
    # three and two layers between single layers, so one batch holds more than eight
    # projections and token reductions of several column counts (k = 40: groups over 64
    # columns, still batched; k = 100: projections over 64 columns, one launch each)
    B, T = 2, 150
    groups = [(96, (130, 72, 72)), (64, (300,)), (136, (520, 260)), (48, (90,)), (80, (200,)),
              (72, (64,)), (40, (150,)), (88, (110, 96)), (56, (70,)), (64, (260,)), (120, (100,))]
    pairs, lid = [], 0
    for g, (d, ps) in enumerate(groups):
        A, Es = _shared_a(B, T, d, ps, layer0=60 + 10 * g)
        for E in Es:
            pairs.append((A, E, lid))
            lid += 1
    pid = D.PROBE_HADAMARD if probe == "hadamard" else D.PROBE_RADEMACHER
    n2l = torch.zeros(len(pairs), B, device="cuda")
    n2 = D.dprc_norm_hutch(pairs, k, 3, probe=pid, n2_layers=n2l)
    refs = [est.hutch_layer(_np(A), _np(E), k, 3, j, probe=probe) for (A, E, j) in pairs]
    got = n2l.cpu().numpy()
    for j in range(len(pairs)):
        assert np.all(_rel(got[j], refs[j]) < NORM_RTOL), j
    assert np.all(_rel(n2.cpu().numpy(), np.sum(refs, axis=0)) < NORM_RTOL)
    # each layer's estimate as from a call of its own (no batching, no shared reduction)
    solo = torch.stack([D.dprc_norm_hutch([(A.clone(), E, j)], k, 3, probe=pid) for (A, E, j) in pairs])
    assert np.all(_rel(got, solo.cpu().numpy()) < 1e-6)
    if k % 16 == 0:
        assert torch.equal(n2l, solo)


@pytest.mark.parametrize("T,ngroups,k,G", [
    (200, 8, 32, 3),      # 1056 (sample, tile) pairs: unsplit, 96 columns
    (520, 2, 25, 3),      # two token splits, 75 columns in 80 (an odd number of column blocks)
    (520, 2, 32, 4),      # 128 columns
])
def test_hutch_wide_groups_two_tiles(D, T, ngroups, k, G):
    # activation groups of more than 64 columns with enough tile pairs for two-tile workgroups;
    # 4104-wide activations have an odd number of tiles, the last one 8 columns wide
    B, d = 4, 4104
    pairs = []
    for g in range(ngroups):
        A, Es = _shared_a(B, T, d, (40, 72, 24, 56)[:G], layer0=400 + 10 * g)
        pairs += [(A, E, 10 * g + j) for j, E in enumerate(Es)]
    n2l = torch.zeros(len(pairs), B, device="cuda")
    D.dprc_norm_hutch(pairs, k, 4, n2_layers=n2l)
    solo = torch.stack([D.dprc_norm_hutch([(A.clone(), E, j)], k, 4) for (A, E, j) in pairs])
    assert np.all(_rel(n2l.cpu().numpy(), solo.cpu().numpy()) < 1e-5)
    for q in (0, G - 1, len(pairs) - 1):
        A, E, j = pairs[q]
        assert np.all(_rel(n2l[q].cpu().numpy(), est.hutch_layer(_np(A), _np(E), k, 4, j)) < NORM_RTOL), q


def test_hutchpp_wide_store_two_tiles(D):
    # s + r = 80 columns stored (not squared) by two-tile workgroups over four token splits,
    # 2056-wide activations (17 tiles)
    B, T, s, r = 4, 1030, 16, 64
    pairs = [_draw(B, T, 2056, p, law="student_t", layer=450 + j) + (j,) for j, p in enumerate((100, 72))]
    n2l = torch.zeros(len(pairs), B, device="cuda")
    D.dprc_norm_hutchpp(pairs, s, r, 9, n2_layers=n2l)
    for q, (A, E, j) in enumerate(pairs):
        assert np.all(_rel(n2l[q].cpu().numpy(), est.hutchpp_layer(_np(A), _np(E), s, r, 9, j)) < NORM_RTOL), q


@pytest.mark.parametrize("accumulate", [False, True])
def test_hutch_more_groups_than_one_sample_sum(D, accumulate):
    # 131 single-layer groups (the per-sample sums of a call take 128 groups per launch, so
    # a second launch continues n2), ragged widths; each layer's estimate equals that of a
    # call of its own bit for bit, n2 their sum in layer order, the clip factors follow n2
    B, T, k, C = 3, 70, 16, 0.5
    pairs = []
    for j in range(131):
        d, p = 40 + 8 * (j % 5), 24 + 16 * (j % 7)
        A, E = _draw(B, T, d, p, layer=300 + j)
        pairs.append((A, E, j))
    n2l = torch.zeros(len(pairs), B, device="cuda")
    n2 = torch.full((B,), 0.25, device="cuda")
    c = torch.zeros(B, device="cuda")
    D.dprc_norm_hutch_clip(pairs, k, 9, C, n2=n2, c=c, n2_layers=n2l, accumulate=accumulate)
    solo = torch.stack([D.dprc_norm_hutch([(A, E, j)], k, 9) for (A, E, j) in pairs])
    assert torch.equal(n2l, solo)
    ref = np.full(B, 0.25 if accumulate else 0.0, dtype=np.float32)
    for j in range(len(pairs)):                       # float adds in layer order
        ref = (ref + solo[j].cpu().numpy()).astype(np.float32)
    assert np.array_equal(n2.cpu().numpy(), ref)
    assert np.allclose(c.cpu().numpy(), est.clip_scale(ref.astype(np.float64), C), rtol=1e-6)
    for j in (0, 64, 127, 128, 130):                  # against the oracle
        A, E, _ = pairs[j]
        assert np.all(_rel(n2l[j].cpu().numpy(), est.hutch_layer(_np(A), _np(E), k, 9, j)) < NORM_RTOL), j


@pytest.mark.parametrize("k", [32, 20])
def test_hutch_large_batch_unsplit(D, k):
    # a batch of eight layers with 1028 (sample, 128-column tile) pairs: its token reductions
    # run without token splits (one workgroup per pair of tiles over all 200 tokens, a ragged
    # last stage; the last layer has an odd number of tiles, its last one 8 columns wide), the
    # layers ragged in both widths; a second call of one layer runs split
    B, T = 4, 200
    shapes = [(4000, 300), (4096, 130), (4000, 520), (4096, 96), (4000, 72), (4096, 260), (4000, 1000), (4104, 40)]
    pairs = []
    for j, (d, p) in enumerate(shapes):
        A, E = _draw(B, T, d, p, layer=200 + j)
        pairs.append((A, E, j))
    n2l = torch.zeros(len(pairs), B, device="cuda")
    n2 = D.dprc_norm_hutch(pairs, k, 11, n2_layers=n2l)
    refs = [est.hutch_layer(_np(A), _np(E), k, 11, j) for (A, E, j) in pairs]
    got = n2l.cpu().numpy()
    for j in range(len(pairs)):
        assert np.all(_rel(got[j], refs[j]) < NORM_RTOL), j
    assert np.all(_rel(n2.cpu().numpy(), np.sum(refs, axis=0)) < NORM_RTOL)
    A, E, j = pairs[0]
    solo = D.dprc_norm_hutch([(A, E, j)], k, 11).cpu().numpy()     # 128 pairs: four token splits
    assert np.all(_rel(got[0], solo) < 1e-5)


@pytest.mark.parametrize("case,probe", [("narrow", "rademacher"), ("chunked", "rademacher"), ("narrow", "hadamard")])
def test_hutch_row_blocks_per_workgroup(D, case, probe):
    # a batch of 32 layers with enough row blocks that each projection workgroup streams
    # several of them (narrow: 512-wide E, four 32-row blocks per workgroup, one probe chunk
    # per row; chunked: 8200-wide E, four 16-row blocks per workgroup, three probe chunks per
    # row and a ragged last stage); a call of one layer gives each workgroup one block
    k = 32
    if case == "narrow":
        B, T, d, p, check = 8, 1024, 64, 512, range(32)
    else:
        B, T, d, p, check = 4, 1024, 48, 8200, (0, 17, 31)
    pairs = []
    for j in range(32):
        A, E = _draw(B, T, d, p, layer=400 + j)
        pairs.append((A, E, j))
    pid = D.PROBE_HADAMARD if probe == "hadamard" else D.PROBE_RADEMACHER
    n2l = torch.zeros(len(pairs), B, device="cuda")
    n2 = D.dprc_norm_hutch(pairs, k, 21, n2_layers=n2l, probe=pid)
    torch.cuda.synchronize()
    got = n2l.cpu().numpy()
    solo = torch.stack([D.dprc_norm_hutch([(A, E, j)], k, 21, probe=pid) for (A, E, j) in pairs]).cpu().numpy()
    assert np.all(_rel(got, solo) < 1e-5)
    assert np.all(_rel(n2.cpu().numpy(), got.astype(np.float64).sum(axis=0)) < 1e-5)
    for j in check:
        A, E, _ = pairs[j]
        assert np.all(_rel(got[j], est.hutch_layer(_np(A), _np(E), k, 21, j, probe=probe)) < NORM_RTOL), j


@pytest.mark.parametrize("B,T,p,k", [(1, 64, 4100, 16), (2, 40, 2600, 5), (1, 200, 4096, 32)])
def test_hutch_few_rows_wide_sketch(D, B, T, p, k):
    # few token rows and a wide sketched side (many 512-column stages per workgroup, ragged end)
    A, E = _draw(B, T, 72, p, layer=9)
    n2 = D.dprc_norm_hutch([(A, E, 3)], k, 5)
    ref = est.hutch_layer(_np(A), _np(E), k, 5, 3)
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)


@pytest.mark.parametrize("case", ["bf16", "shared", "gaussian", "fp32", "accumulate"])
def test_hutch_clip_fused_matches_separate_calls(D, case):
    C = 0.3
    if case == "shared":
        A, Es = _shared_a(3, 150, 200, (200, 64, 64))
        pairs = [(A, E, j) for j, E in enumerate(Es)]
    elif case == "fp32":
        A, E = _draw(2, 64, 64, 48, dtype="f32", layer=2)
        pairs = [(A, E, 0)]
    else:
        A, E = _draw(3, 130, 96, 300, layer=2)
        pairs = [(A, E, 0)]
    probe = D.PROBE_GAUSSIAN if case == "gaussian" else D.PROBE_RADEMACHER
    prior = torch.tensor([0.5, 0.01, 2.0][:pairs[0][0].shape[0]], device="cuda")
    acc = case == "accumulate"
    n2f, cf = D.dprc_norm_hutch_clip(pairs, 16, 4, C, probe=probe, n2=prior.clone() if acc else None, accumulate=acc)
    n2 = D.dprc_norm_hutch(pairs, 16, 4, probe=probe, n2=prior.clone() if acc else None, accumulate=acc)
    c = D.dprc_clip_scale(n2, C)
    assert torch.equal(n2f, n2) and torch.equal(cf, c)
    assert np.allclose(cf.cpu().numpy(), est.clip_scale(n2.cpu().numpy().astype(np.float64), C), rtol=1e-6)


def test_hutch_tiny_workload_fp32(D):
    cfg = workloads.BY_NAME["tiny"]
    A, E = workloads.layer_inputs(cfg, 0, device="cuda")
    n2 = D.dprc_norm_hutch([(A, E, 0)], cfg["k"], 0)
    ref = est.hutch_layer(_np(A), _np(E), cfg["k"], 0, 0)
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("side", [0, 1])
def test_hutch_hadamard_probes_give_exact_norm(D, dtype, side):
    # 64 Sylvester-Hadamard columns span the sketched dimension (<= 64): estimate == ||A_i^T E_i||^2
    A, E = _draw(2, 150, 64, 48, dtype=dtype, layer=3)
    n2 = D.dprc_norm_hutch([(A, E, 0)], 64, 0, side=side, probe=D.PROBE_HADAMARD)
    exact = est.exact_layer(_np(A), _np(E))
    assert np.all(_rel(n2.cpu().numpy(), exact) < NORM_RTOL)


def test_hutch_token_splits_and_multilayer(D):
    # long token range -> several token splits per tile; two layers summed on top of a prior n2
    A1, E1 = _draw(2, 3000, 256, 200, layer=0)
    A2, E2 = _draw(2, 700, 136, 1100, layer=1)
    n2 = torch.tensor([1.5, 2.5], device="cuda")
    n2l = torch.zeros(2, 2, device="cuda")
    D.dprc_norm_hutch([(A1, E1, 10), (A2, E2, 11)], 16, 7, n2=n2, n2_layers=n2l, accumulate=True)
    r1 = est.hutch_layer(_np(A1), _np(E1), 16, 7, 10)
    r2 = est.hutch_layer(_np(A2), _np(E2), 16, 7, 11)
    got = n2l.cpu().numpy()
    assert np.all(_rel(got[0], r1) < NORM_RTOL) and np.all(_rel(got[1], r2) < NORM_RTOL)
    assert np.all(_rel(n2.cpu().numpy(), np.array([1.5, 2.5]) + r1 + r2) < NORM_RTOL)


def test_hutch_strided_rows(D):
    A, E = _draw(2, 100, 120, 90, layer=5, row_pad_a=8, row_pad_e=38)
    assert A.stride(1) == 128 and E.stride(1) == 128
    n2 = D.dprc_norm_hutch([(A, E, 2)], 8, 1)
    ref = est.hutch_layer(_np(A), _np(E), 8, 1, 2)
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)


def test_hutch_deterministic(D):
    A, E = _draw(2, 2048, 512, 384, layer=4)
    a = D.dprc_norm_hutch([(A, E, 3)], 16, 9)
    b = D.dprc_norm_hutch([(A, E, 3)], 16, 9)
    assert torch.equal(a, b)


# ---- Hutch++ ------------------------------------------------------------------------------

# The QR tree factors 128-row blocks and stacks their s x s R factors: the cases
# below take 2 and 3 levels, odd s (s = 5, padded to 8 register columns), s = 1
# and s = 32 (the largest), with ragged last blocks.
@pytest.mark.parametrize("B,T,d,p,s,r,side,dtype", [
    (2, 300, 200, 150, 8, 12, 0, "bf16"),
    (1, 520, 136, 300, 16, 32, 1, "bf16"),
    (2, 64, 64, 48, 4, 4, 0, "f32"),
    (1, 200, 600, 96, 32, 16, 1, "bf16"),      # m = 600: 5 blocks -> 160 rows -> 2 -> 1 (3 levels)
    (2, 150, 64, 1100, 5, 7, 0, "bf16"),       # m = 1100: 9 blocks -> 45 rows -> 1
    (2, 100, 50, 260, 1, 3, 0, "bf16"),        # s = 1
    (1, 180, 72, 130, 6, 40, 0, "bf16"),       # r = 40: the finalize's residual columns take two passes
])
def test_hutchpp_parity(D, B, T, d, p, s, r, side, dtype):
    A, E = _draw(B, T, d, p, dtype=dtype, law="student_t", layer=2)
    n2 = D.dprc_norm_hutchpp([(A, E, 6)], s, r, 3, side=side)
    ref = est.hutchpp_layer(_np(A), _np(E), s, r, 3, 6, side=side)
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_hutchpp_low_rank_is_exact(D, dtype):
    A, E = _draw(2, 12, 80, 96, dtype=dtype, layer=7)      # rank(A_i^T E_i) <= 12 <= s
    n2 = D.dprc_norm_hutchpp([(A, E, 0)], 16, 8, 11)
    exact = est.exact_layer(_np(A), _np(E))
    assert np.all(_rel(n2.cpu().numpy(), exact) < NORM_RTOL)


@pytest.mark.parametrize("side", [0, 1])
def test_hutchpp_low_rank_is_exact_deep_tree(D, side):
    # rank(A_i^T E_i) <= 12 <= s; the sketched width 1500 takes a 3-level QR tree
    A, E = _draw(2, 12, 1500 if side == 1 else 80, 80 if side == 1 else 1500, layer=9)
    n2 = D.dprc_norm_hutchpp([(A, E, 0)], 16, 8, 13, side=side)
    exact = est.exact_layer(_np(A), _np(E))
    assert np.all(_rel(n2.cpu().numpy(), exact) < NORM_RTOL)


@pytest.mark.parametrize("estimator", ["hutchpp", "gaussian"])
def test_dense_columns_many_rows(D, estimator):
    # B*T >= 16384 token rows: the passes with dense columns (Hutch++ W_S and Q, Gaussian
    # probes) take 64-row projection workgroups; T is ragged
    B, T, d, p = 2, 8200, 72, 200
    A, E = _draw(B, T, d, p, law="student_t", layer=12)
    if estimator == "hutchpp":
        n2 = D.dprc_norm_hutchpp([(A, E, 5)], 8, 12, 6)
        ref = est.hutchpp_layer(_np(A), _np(E), 8, 12, 6, 5)
    else:
        n2 = D.dprc_norm_hutch([(A, E, 5)], 16, 6, probe=D.PROBE_GAUSSIAN)
        ref = est.hutch_layer(_np(A), _np(E), 16, 6, 5, probe="gaussian")
    assert np.all(_rel(n2.cpu().numpy(), ref) < NORM_RTOL)


def test_hutchpp_many_layers_grouped(D):
    # 10 layers: two groups of the batched QR, sketched widths that take 1, 2 and 3 tree levels
    B, T = 2, 160
    shapes = [(64, 100), (96, 300), (48, 1500), (80, 130), (72, 640), (64, 90), (56, 2100), (40, 200),
              (88, 120), (64, 700)]
    pairs = []
    for li, (d, p) in enumerate(shapes):
        A, E = _draw(B, T, d, p, law="student_t", layer=20 + li)
        pairs.append((A, E, li))
    n2l = torch.zeros(len(pairs), B, device="cuda")
    n2 = D.dprc_norm_hutchpp(pairs, 8, 12, 4, n2_layers=n2l)
    ref_l = [est.hutchpp_layer(_np(A), _np(E), 8, 12, 4, li) for (A, E, li) in pairs]
    got_l = n2l.cpu().numpy()
    for li in range(len(pairs)):
        assert np.all(_rel(got_l[li], ref_l[li]) < NORM_RTOL), li
    assert np.all(_rel(n2.cpu().numpy(), sum(ref_l)) < NORM_RTOL)


def test_hutchpp_grouped_wide_passes(D):
    # three bf16 layers with s + r = 80 > 64 columns: the grouped passes take one projection
    # launch per layer (wider than the batched kernel) and one token reduction
    B, T, s, r = 2, 300, 16, 64
    shapes = [(120, 260), (72, 500), (200, 136)]
    pairs = []
    for li, (d, p) in enumerate(shapes):
        A, E = _draw(B, T, d, p, law="student_t", layer=40 + li)
        pairs.append((A, E, li))
    n2l = torch.zeros(len(pairs), B, device="cuda")
    n2 = D.dprc_norm_hutchpp(pairs, s, r, 8, n2_layers=n2l)
    ref_l = [est.hutchpp_layer(_np(A), _np(E), s, r, 8, li) for (A, E, li) in pairs]
    got_l = n2l.cpu().numpy()
    for li in range(len(pairs)):
        assert np.all(_rel(got_l[li], ref_l[li]) < NORM_RTOL), li
    assert np.all(_rel(n2.cpu().numpy(), sum(ref_l)) < NORM_RTOL)


def test_hutchpp_without_sketch_equals_hutch(D):
    A, E = _draw(2, 300, 100, 180, layer=8)
    a = D.dprc_norm_hutchpp([(A, E, 4)], 0, 16, 5)
    b = D.dprc_norm_hutch([(A, E, 4)], 16, 5)
    assert torch.equal(a, b)


# ---- clip factors, accumulation, noise --------------------------------------------------------

def test_clip_scale_edges(D):
    C = 2.0
    vals = [0.0, 4.0, 16.0, 1.0, math.inf, math.nan, -1.0, 1e30, 3.9999998]
    n2 = torch.tensor(vals, dtype=torch.float32, device="cuda")
    c = D.dprc_clip_scale(n2, C).cpu().numpy()
    ref = est.clip_scale(np.array(vals, dtype=np.float32).astype(np.float64), C)
    assert np.all(np.abs(c - ref) <= 1e-6 * np.maximum(ref, 1e-30))


@pytest.mark.parametrize("B,T,d,p,dtype", [
    (3, 150, 200, 260, "bf16"),     # ragged tiles; per-sample scaling inside a tile
    (2, 2000, 96, 72, "bf16"),      # few tiles -> split over samples and tokens
    (2, 64, 64, 48, "f32"),         # the tiny workload
    (2, 300, 500, 1000, "bf16"),    # 2 x 4 = 8 tiles: the XCD tile order (a multiple of 8 tiles), ragged
    (1, 260, 2000, 700, "bf16"),    # 8 x 3 = 24 tiles with d > p (the other walking order), ragged
])
def test_clip_accumulate_parity(D, B, T, d, p, dtype):
    A, E = _draw(B, T, d, p, dtype=dtype, layer=9)
    cvals = [0.25, 0.0, 0.8] if B == 3 else [0.37, 1.0][:B]
    c = torch.tensor(cvals, dtype=torch.float32, device="cuda")
    g = D.dprc_clip_accumulate(A, E, c)
    ref = est.clip_accumulate(_np(A), _np(E), np.array(cvals, dtype=np.float32).astype(np.float64))
    err = np.linalg.norm(g.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err < GRAD_RTOL
    # accumulate onto an existing gradient
    g0 = torch.full_like(g, 0.5)
    D.dprc_clip_accumulate(A, E, c, grad=g0, accumulate=True)
    err2 = np.linalg.norm(g0.cpu().numpy() - (ref + 0.5)) / np.linalg.norm(ref + 0.5)
    assert err2 < GRAD_RTOL


@pytest.mark.parametrize("aligned", [True, False])
def test_clip_accumulate_layers_parity(D, aligned):
    # several layers of one batch in one launch, no token splits: each layer's gradient against
    # the oracle and against a call of its own (which splits the small ones over tokens); 8 and
    # 15 tiles (the XCD ordering, ragged edges), T free per layer; with a 1001-wide layer the
    # launch takes element loads; then accumulation onto existing gradients
    B = 3
    shapes = [(150, 1024, 512), (100, 520, 1032), (64, 64, 48), (77, 256, 256), (150, 2048, 512)]
    if not aligned:
        shapes.append((90, 1001, 96))
    pairs = [(*_draw(B, T, d, p, layer=500 + j), j) for j, (T, d, p) in enumerate(shapes)]
    cvals = [0.25, 0.0, 0.8]
    c = torch.tensor(cvals, dtype=torch.float32, device="cuda")
    grads = D.dprc_clip_accumulate_layers(pairs, c)
    for (A, E, j), g in zip(pairs, grads):
        ref = est.clip_accumulate(_np(A), _np(E), np.array(cvals, dtype=np.float32).astype(np.float64))
        got = g.cpu().numpy()
        assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < GRAD_RTOL, j
        solo = D.dprc_clip_accumulate(A, E, c).cpu().numpy()
        assert np.linalg.norm(got - solo) / np.linalg.norm(solo) < 1e-5, j
    g0 = [torch.full_like(g, 0.5) for g in grads]
    D.dprc_clip_accumulate_layers(pairs, c, grads=g0, accumulate=True)
    for g, gacc in zip(grads, g0):
        assert torch.allclose(gacc, g + 0.5, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("d,p,pad", [
    (1025, 13200, 0),     # 260 tiles: a round of 256 whole ones, then four as quarters
    (1032, 13057, 1),     # the same with odd rows
    (520, 300, 0),        # six tiles, all as quarters, some of them past the edges
])
def test_clip_accumulate_quarter_tiles(D, d, p, pad):
    A, E = _draw(2, 70, d, p, layer=560, row_pad_a=pad, row_pad_e=pad)
    c = torch.tensor([0.25, 1.0], device="cuda")
    ref = est.clip_accumulate(_np(A), _np(E), c.cpu().numpy().astype(np.float64))
    g, = D.dprc_clip_accumulate_layers([(A, E)], c)
    assert np.linalg.norm(g.cpu().numpy() - ref) < 1e-5 * np.linalg.norm(ref)
    g = D.dprc_clip_accumulate(A, E, c, grad=torch.full((d, p), 0.5, device="cuda"), accumulate=True)
    assert np.linalg.norm(g.cpu().numpy() - ref - 0.5) < 1e-5 * np.linalg.norm(ref + 0.5)


def test_clip_accumulate_layers_two_launches(D):
    # 70 layers (64 per launch), gradients with row strides wider than p
    B, pairs, grads = 2, [], []
    for j in range(70):
        d, p = 40 + 8 * (j % 4), 24 + 8 * (j % 5)
        A, E = _draw(B, 30 + j, d, p, layer=600 + j)
        pairs.append((A, E, j))
        grads.append(torch.zeros(d, p + 8, device="cuda")[:, :p])
    c = torch.tensor([0.6, 1.0], device="cuda")
    D.dprc_clip_accumulate_layers(pairs, c, grads=grads)
    for (A, E, j), g in zip(pairs, grads):
        solo = D.dprc_clip_accumulate(A, E, c).cpu().numpy()
        assert np.linalg.norm(g.cpu().numpy() - solo) / np.linalg.norm(solo) < 1e-5, j


def test_clip_accumulate_layers_edges(D):
    # a layer with a whole round of tiles (a launch of its own) between small ones, a
    # one-token layer, and all-zero factors (nothing added, accumulation leaves the
    # gradients as they were)
    B = 2
    shapes = [(64, 40, 24), (64, 4096, 4096), (1, 8, 8), (33, 300, 72)]
    pairs = [(*_draw(B, T, d, p, layer=700 + j), j) for j, (T, d, p) in enumerate(shapes)]
    c = torch.tensor([0.3, 0.9], device="cuda")
    grads = D.dprc_clip_accumulate_layers(pairs, c)
    for (A, E, j), g in zip(pairs, grads):
        solo = D.dprc_clip_accumulate(A, E, c)
        assert ((g - solo).norm() / solo.norm()).item() < 1e-5, j
        rows = [0, A.shape[2] // 2, A.shape[2] - 1]
        ref = est.clip_accumulate_rows(_np(A), _np(E), np.array([0.3, 0.9], dtype=np.float32).astype(np.float64), rows)
        got = g[rows].cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < GRAD_RTOL, j
    zero = torch.zeros(B, device="cuda")
    fresh = D.dprc_clip_accumulate_layers(pairs, zero)
    assert all(torch.count_nonzero(g) == 0 for g in fresh)
    before = [g.clone() for g in grads]
    D.dprc_clip_accumulate_layers(pairs, zero, grads=grads, accumulate=True)
    assert all(torch.equal(g, b) for g, b in zip(grads, before))


def test_clip_accumulate_zero_factor_drops_nonfinite_sample(D):
    A, E = _draw(2, 100, 64, 64, layer=10)
    A[1, 3, 5] = float("nan")
    E[1, 7, 9] = float("inf")
    c = torch.tensor([0.5, 0.0], device="cuda")
    g = D.dprc_clip_accumulate(A, E, c).cpu().numpy()
    assert np.all(np.isfinite(g))
    ref = est.clip_accumulate(_np(A)[:1], _np(E)[:1], [0.5])
    assert np.linalg.norm(g - ref) / np.linalg.norm(ref) < GRAD_RTOL


def test_clip_accumulate_all_zero_factors(D):
    A, E = _draw(2, 70, 40, 30, layer=11)
    g = D.dprc_clip_accumulate(A, E, torch.zeros(2, device="cuda"))
    assert torch.count_nonzero(g) == 0


@pytest.mark.parametrize("numel,offset", [(1000, 0), (1023, 0), (7, 1)])
def test_add_noise_parity(D, numel, offset):
    sigma, C = 0.8, 1.0
    base = torch.randn(numel + offset, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    g = base[offset:].clone() if offset == 0 else base[offset:]
    g0 = g.clone().cpu().numpy().astype(np.float64)
    D.dprc_add_noise(g, sigma, C, 77, 5)
    ref = est.add_noise(g0, sigma, C, 77, 5)
    assert np.max(np.abs(g.cpu().numpy() - ref)) <= 1e-5 * sigma * C + 4e-7 * np.max(np.abs(ref))


def test_add_noise_moments(D):
    g = torch.zeros(1 << 22, device="cuda")
    D.dprc_add_noise(g, 1.0, 1.0, 3, 9)
    x = g.double()
    n = x.numel()
    assert abs(x.mean().item()) < 5 / math.sqrt(n)
    assert abs(x.var().item() - 1.0) < 5 * math.sqrt(2.0 / n)


# ---- private AdamW step (noise + 1/B + AdamW + transposed bf16 weights) ---------------------

@pytest.mark.parametrize("d,p,ld_pad,sigma,steps,wout", [
    (128, 256, 0, 0.7, 3, True),      # vector path, three steps
    (67, 130, 3, 0.5, 2, True),       # p not a multiple of 4, padded rows: element path, ragged tiles
    (64, 64, 4, 0.0, 1, False),       # no noise, no weight copy, padded rows
    (1, 5, 0, 1.0, 1, True),
    (3080, 3200, 0, 0.7, 1, True),    # more than 256 MB of arrays: non-temporal accesses, ragged tiles
])
def test_private_adamw_parity(D, d, p, ld_pad, sigma, steps, wout):
    r = np.random.default_rng(1000 * d + p)
    ld = p + ld_pad
    C, Bsz, lr, b1, b2, eps, wd, seed, tid = 1.5, 4, 1e-2, 0.9, 0.99, 1e-8, 0.05, 21, 5

    def dev(x):
        buf = torch.zeros(d, ld, dtype=torch.float32, device="cuda")
        buf[:, :p] = torch.tensor(x, dtype=torch.float32)
        return buf[:, :p]
    th0 = (r.standard_normal((d, p)) * 0.02).astype(np.float32)
    theta, m, v = dev(th0), dev(np.zeros((d, p))), dev(np.zeros((d, p)))
    w = torch.empty(p, d, dtype=torch.bfloat16, device="cuda") if wout else None
    th, mr, vr = th0.astype(np.float64), 0.0, 0.0
    firm = None
    for t in range(1, steps + 1):
        G = dev((r.standard_normal((d, p)) * 0.3).astype(np.float32))
        D.dprc_private_adamw(theta, m, v, G, sigma, C, seed, tid, 1.0 / Bsz, lr, b1, b2, eps, wd, t, w=w)
        G64 = est.as_f64(G.cpu())
        g = (est.add_noise(G64, sigma, C, seed, tid) if sigma > 0 else G64) / Bsz
        if firm is None:
            firm = np.abs(g) > 1e-4               # first update lr g/(|g|+eps) is steep near g = 0
        th, mr, vr = est.adamw(th, g, mr, vr, t, lr, b1, b2, eps, wd)
    torch.cuda.synchronize()
    got = theta.cpu().double().numpy()
    assert firm.mean() > 0.99
    assert np.max(np.abs(got - th)[firm]) <= 2e-6
    assert np.max(np.abs(got - th)) <= 2 * lr * steps
    assert np.allclose(m.cpu().double().numpy(), mr, rtol=1e-5, atol=1e-8)
    assert np.allclose(v.cpu().double().numpy(), vr, rtol=1e-5, atol=1e-10)
    if wout:
        assert torch.equal(w, theta.t().to(torch.bfloat16))
