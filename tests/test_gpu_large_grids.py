"""Calls whose launches hold 2^32 threads or more: a grid dimension takes fewer, so their
workgroups fill several rows of it.  Small operands in all but one direction."""

import numpy as np
import pytest
import torch

from oracle import accountant as ac

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_24879_amd import dprc
    dprc.lib()
    return dprc


@pytest.fixture(autouse=True)
def _free():
    yield
    torch.cuda.empty_cache()


def test_step_pld_grid(D):
    n, sigma, p = (1 << 26) + 3, 1.0, 0.25
    h = 20.0 / n
    q, qi = D.dprc_pld_step(sigma, p, h, n)
    for t in (-0.25, -0.1, 0.0, 0.5, 2.0):              # probability above a cut, against the survival function
        j = int(t / h) + n - 1
        cut = (j - n + 0.5) * h
        s = np.log(1.0 / p - (1.0 - p) / p * np.exp(-cut))
        al, _, _, beb = ac.mechanism_kernels(np.array([cut + s]), sigma)
        assert abs(q[j:].sum().item() + qi.item() - (p * beb + (1.0 - p) * al).item()) < 1e-11, t


def test_fp32_token_rows(D):
    T = (1 << 27) + 5
    A = torch.ones(1, T, 1, device="cuda")
    E = torch.full((1, T, 1), 2.0 ** -20, device="cuda")
    n2 = D.dprc_norm_hutch([(A, E, 0)], 1, 3)
    assert abs(n2.item() / (T * 2.0 ** -20) ** 2 - 1.0) < 1e-6


def test_fp32_reduced_width(D):
    d = (1 << 29) + 70
    A = torch.ones(1, 1, d, device="cuda")
    E = torch.full((1, 1, 1), 2.0 ** -14, device="cuda")
    n2 = D.dprc_norm_hutch([(A, E, 0)], 1, 3)
    assert n2.item() == np.float32(d * 2.0 ** -28)


def _halves(call, pairs):
    B = pairs[0][0].shape[0]
    parts = [[(A[b0:b1], E[b0:b1], j) for (A, E, j) in pairs] for b0, b1 in ((0, B // 2), (B // 2, B))]
    return torch.cat([call(q) for q in parts])


def test_wide_token_reduction(D):
    # 80 columns: one reduction of 129 pairs of tiles for each of 65535 samples
    B, d = 65535, 33000
    A = torch.randn(B, 1, 8, device="cuda").bfloat16().repeat(1, 1, d // 8)
    E = torch.randn(B, 1, 8, device="cuda").bfloat16()
    n2 = D.dprc_norm_hutch([(A, E, 0)], 80, 3)
    assert torch.equal(n2, _halves(lambda q: D.dprc_norm_hutch(q, 80, 3), [(A, E, 0)]))


def test_hutchpp_qr(D):
    # 258 blocks of 128 rows for each of 65535 samples
    B, p = 65535, 33000
    A = torch.randn(B, 1, 8, device="cuda").bfloat16()
    E = torch.randn(B, 1, 8, device="cuda").bfloat16().repeat(1, 1, p // 8)
    n2 = D.dprc_norm_hutchpp([(A, E, 0)], 1, 1, 3)
    assert torch.equal(n2, _halves(lambda q: D.dprc_norm_hutchpp(q, 1, 1, 3), [(A, E, 0)]))
