"""GPU privacy accounting against the oracle.

The chi-squared CDF and MiddleRegionCDF kernels (fp64) against the oracle's
scipy-based CDF and brute-force supremum, the paper's d = 3 counter-example
evaluated by the kernel, x_+ from the GPU binary search, and eps / noise
multipliers from the GPU accountant (torch fp64 PLD) against the oracle's
numpy accountant, without and with the Hutchinson envelope.
"""

import math

import numpy as np
import pytest
import torch

from oracle import accountant as ac

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_24879_amd import accountant, dprc
    dprc.lib()
    return dprc, accountant


def _t(x):
    return torch.tensor(np.asarray(x, dtype=np.float64), device="cuda")


@pytest.mark.parametrize("dof", [1, 3, 16, 100, 1000, 32768])
def test_chi2_cdf(mods, dof):
    D, _ = mods
    xs = np.concatenate([np.linspace(0.0, 3.0, 31) * dof, [1e-6 * dof, dof - math.sqrt(dof), dof + 0.5]])
    got = D.dprc_chi2_cdf(_t(xs), dof).cpu().numpy()
    ref = np.array([ac.chi2_cdf(x, dof) for x in xs])
    assert np.all(np.abs(got - ref) <= 1e-12 + 1e-9 * ref)


@pytest.mark.parametrize("k,d,nl,xs", [
    (4, 3, 11, [0.7, 1.0, 1.1, 1.3, 1.9]),
    (2, 5, 6, [0.95, 1.05, 1.2, 1.5]),
    (8, 4, 7, [1.02, 1.06]),
    (1, 2, 21, [0.4, 1.5, 3.0]),
])
def test_middle_region_matches_brute_force(mods, k, d, nl, xs):
    D, _ = mods
    best, arg = D.dprc_envelope_middle(_t(xs), k, d, nl)
    best, arg = best.cpu().numpy(), arg.cpu().numpy()
    lam = ac.lambda_grid(nl)
    for e, x in enumerate(xs):
        ref, rarg = ac.middle_region(x, k, d, nl)
        assert abs(best[e] - ref) < 1e-10, (x, best[e], ref)
        i, j, l = arg[e]
        assert 1 <= i and 1 <= j and i + j <= d and 0 <= l < nl
        assert abs(ac.two_level_cdf(x, int(i), int(j), float(lam[l]), k) - ref) < 1e-10


@pytest.mark.parametrize("k,d,nx", [(1, 2, 1), (4, 17, 60), (32, 60, 7)])
def test_middle_region_of_single_terms(mods, k, d, nx):
    # n_lambda = 1: lam = 0 only, one incomplete gamma per form
    D, _ = mods
    from scipy import special
    xs = np.concatenate([[-1.0, 0.0], np.linspace(0.3, 2.5, nx)])
    best, arg = D.dprc_envelope_middle(_t(xs), k, d, 1)
    n2 = k * np.arange(1, d)
    ref = special.gammainc(n2 / 2, np.maximum(xs, 0.0)[:, None] * n2 / 2)
    assert np.max(np.abs(best.cpu().numpy() - ref.max(axis=1))) < 1e-12
    i, j, l = arg.cpu().numpy().T
    assert np.all(l == 0) and np.all(i >= 1) and np.all(i + j <= d)
    assert np.max(np.abs(ref[np.arange(len(xs)), j - 1] - ref.max(axis=1))) < 1e-12


def test_szekely_counterexample_on_gpu(mods):
    # d = 3, k = 1 at x = 1.5: the best two-level form puts 0.7 on one coordinate and 0.15 on each
    # of the others, above the uniform form 0.7877 and every rank-2 form (0.7872)
    D, _ = mods
    best, arg = D.dprc_envelope_middle(_t([1.5]), 1, 3, 51)
    assert abs(best.item() - 0.79519) < 1e-5
    assert best.item() > ac.chi2_cdf(4.5, 3) > 0.7872
    i, j, l = arg[0].tolist()
    assert (i, j, l) == (2, 1, 30)          # lam = 0.3 on the pair: 0.15 + 0.15, 0.7 on the single one


def test_x_plus(mods):
    _, A = mods
    for k, d in [(4, 3), (16, 2)]:
        assert abs(A.x_plus(k, d, tol=1e-7, n_lambda=11) - ac.x_plus(k, d, tol=1e-7, n_lambda=11)) < 3e-7


def test_epsilon_plain_matches_oracle(mods):
    _, A = mods
    for (sigma, N, B, E, delta) in [(1.1, 1000, 50, 2, 1e-5), (0.9, 600, 64, 3, 1e-6), (2.0, 40, 40, 9, 1e-5)]:
        got = A.epsilon(sigma, N, B, E, delta)
        ref = ac.epsilon(sigma, N, B, E, delta)
        assert abs(got - ref) <= 1e-6 * ref, (got, ref)


def test_epsilon_with_envelope_matches_oracle(mods):
    _, A = mods
    k, d, nl, nb = 8, 4, 7, 600
    y, w = A.envelope_law(k, d, n_bins=nb, n_lambda=nl)
    xp = ac.x_plus(k, d, tol=1e-6, n_lambda=nl)
    y_max = 1.0 + 12.0 * math.sqrt(2.0 / k)
    yr, wr = ac.envelope_bins(lambda v: ac.envelope_cdf([v], k, d, xp, nl)[0], 0.0, y_max, nb)
    assert np.allclose(y.cpu().numpy(), yr, rtol=0, atol=1e-12)
    assert np.max(np.abs(w.cpu().numpy() - wr)) < 1e-8
    got = A.epsilon(1.0, 1000, 50, 2, 1e-5, envelope=(y, w))
    ref = ac.epsilon(1.0, 1000, 50, 2, 1e-5, y=yr, w=wr)
    assert abs(got - ref) <= 1e-5 * ref
    # randomized clipping costs privacy: more eps than deterministic clipping at the same sigma
    assert got > A.epsilon(1.0, 1000, 50, 2, 1e-5)


def test_noise_multiplier_brackets_the_target(mods):
    _, A = mods
    s = A.noise_multiplier(2.0, 1000, 50, 2, 1e-5, tol=1e-3)
    assert A.epsilon(s, 1000, 50, 2, 1e-5) <= 2.0 < A.epsilon(s - 2e-3, 1000, 50, 2, 1e-5)


def test_envelope_bins_kernel_matches_oracle(mods):
    # the binning kernel on a smooth CDF (chi^2(k)/k), a step CDF and a CDF with a dip
    D, _ = mods
    k, y_max = 32, 1.0 + 12.0 * math.sqrt(2.0 / 32)
    for n in (7, 1000, 4000, 70000):
        ys = np.linspace(0.0, y_max, n + 1)
        F = np.array([ac.vertex_cdf(y, k) for y in ys])
        ybar, w = D.dprc_envelope_bins(_t(F), 0.0, y_max)
        yr, wr = ac.envelope_bins(lambda v: ac.vertex_cdf(v, k), 0.0, y_max, n)
        assert np.allclose(ybar.cpu().numpy(), yr, rtol=0, atol=1e-13), n
        assert np.max(np.abs(w.cpu().numpy() - wr)) < 1e-14, n
    vals = np.array([0.0, 0.4, 0.39, 0.4, 1.0])
    ybar, w = D.dprc_envelope_bins(_t(vals), 0.0, 4.0)
    assert np.allclose(w.cpu().numpy(), [0.4, 0.0, 0.0, 0.6], atol=1e-15)
    step = (np.linspace(0.0, 3.0, 301) >= 0.3141).astype(np.float64)
    _, w = D.dprc_envelope_bins(_t(step), 0.0, 3.0)
    w = w.cpu().numpy()
    assert w[31] == 1.0 and np.count_nonzero(w) == 1


@pytest.mark.parametrize("sigma,p,envelope", [(0.8, 0.25, False), (1.1, 0.05, True), (2.0, 1.0, False),
                                              (0.9, 1.0, True)])
def test_step_pld_kernel_matches_oracle(mods, sigma, p, envelope):
    D, A = mods
    h, t_max = 1e-3, 20.0
    y = w = None
    if envelope:
        y, w = A.envelope_law(8, 4, n_bins=300, n_lambda=7)
    q, qi = D.dprc_pld_step(sigma, p, h, int(round(t_max / h)), y, w)
    grid, qr, qir = ac.single_step_pld(sigma, p, h, t_max, None if y is None else y.cpu().numpy(),
                                       None if w is None else w.cpu().numpy())
    got = q.cpu().numpy()
    assert got.shape == qr.shape
    assert np.max(np.abs(got - qr)) < 1e-13
    assert abs(qi.item() - qir) < 1e-13
    assert abs(got.sum() + qi.item() - 1.0) < 1e-12


def test_pld_fold_and_delta_kernels_match_oracle(mods):
    # one composition and delta(eps) at a batch of eps values against the oracle's numpy steps
    D, A = mods
    h, t_max = 1e-3, 8.0
    q, qi = D.dprc_pld_step(0.7, 0.3, h, int(round(t_max / h)))
    grid, qr, qir = ac.single_step_pld(0.7, 0.3, h, t_max)
    q2, qi2 = A._compose2(q, qi, q, qi)
    r2, ri2 = ac._conv_truncated(qr, qir, qr, qir)
    assert np.max(np.abs(q2.cpu().numpy() - r2)) < 1e-12
    assert abs(qi2.item() - ri2) < 1e-12
    eps = np.array([0.0, 0.1, 0.5, 1.0, 2.5, 7.9995, 8.5])
    got = D.dprc_pld_delta(q2, h, qi2, _t(eps)).cpu().numpy()
    ref = np.array([ac.delta_of_eps(grid, r2, ri2, e) for e in eps])
    assert np.max(np.abs(got - ref)) < 1e-12


@pytest.mark.parametrize("k,d,i,j,lam", [
    (1, 3, 1, 2, 0.5), (1, 64, 63, 1, 0.01), (2, 5, 2, 1, 0.35), (32, 64, 1, 63, 0.5), (32, 64, 40, 3, 0.02),
    (64, 200, 1, 199, 0.5),                  # the second term is narrow: more than 16 panels
])
def test_middle_region_single_forms(mods, k, d, i, j, lam):
    # MiddleRegionCDF is the largest form; each form's own CDF is checked through d = i + j with
    # the grid holding lam, against fine quadrature (400 panels of 32 nodes, scipy's gammainc)
    D, _ = mods
    from scipy import special
    nodes, w = np.polynomial.legendre.leggauss(32)

    def form(x, i, j, lam):
        n1, n2 = i * k, j * k
        a, b = lam / n1, (1 - lam) / n2
        smax, c = math.sqrt(x / a), math.sqrt(n1)
        lo, hi = max(0.0, c - 10), min(smax, c + 10)
        if hi <= lo:
            return 0.0
        edge = hi >= smax
        t = np.linspace(0 if edge else lo, math.sqrt(smax - lo) if edge else hi, 401)
        h = (t[1:] - t[:-1]) / 2
        tt = (t[:-1] + h)[:, None] + h[:, None] * nodes
        s = smax - tt * tt if edge else tt
        rest = a * tt * tt * (2 * smax - tt * tt) if edge else x - a * s * s
        ok = (s > 0) & (rest > 0)
        f = np.exp((1 - n1 / 2) * math.log(2) - special.gammaln(n1 / 2) + (n1 - 1) * np.log(np.where(ok, s, 1)) - s * s / 2)
        f = np.where(ok, f * (2 * tt if edge else 1), 0) * special.gammainc(n2 / 2, np.where(ok, rest, 0) / (2 * b))
        return float((h * (f @ w)).sum())

    for x in (0.8, 1.001, 1.3):
        best, arg = D.dprc_envelope_middle(_t([x]), k, d, 51)
        bi, bj, bl = arg[0].tolist()
        blam = bl / 100.0
        ref = form(x, bi, bj, blam) if bl else special.gammainc(bj * k / 2, x * bj * k / 2)
        assert abs(best.item() - ref) < 1e-11            # the maximiser's value
        assert best.item() > form(x, i, j, lam) - 1e-11  # and no other form exceeds it


@pytest.mark.parametrize("n_half,n_bins", [(1, 0), (33, 1), (100, 65), (383, 513), (385, 4), (700, 513)])
def test_pld_small_grids(mods, n_half, n_bins):
    # grids shorter than a workgroup, bins that do not fill a wave's table
    D, A = mods
    h, sigma, p = 0.05, 0.9, 0.3
    y = w = None
    if n_bins:
        y = np.linspace(0.3, 2.0, n_bins)
        w = np.full(n_bins, 1.0 / n_bins)
        w[n_bins // 2] = 0.0
        w /= max(w.sum(), 1e-300) if w.sum() > 0 else 1.0
        if w.sum() == 0:
            w[:] = 1.0
    q, qi = D.dprc_pld_step(sigma, p, h, n_half, _t(y) if n_bins else None, _t(w) if n_bins else None)
    grid, qr, qir = ac.single_step_pld(sigma, p, h, n_half * h, y, w)
    assert np.max(np.abs(q.cpu().numpy() - qr)) < 1e-13 and abs(qi.item() - qir) < 1e-13
    r = _t(np.convolve(qr, qr))
    q2, qi2 = D.dprc_pld_fold(r, len(qr), qi, qi)
    r2, ri2 = ac._conv_truncated(qr, qir, qr, qir)
    assert np.max(np.abs(q2.cpu().numpy() - r2)) < 1e-13 and abs(qi2.item() - ri2) < 1e-13


@pytest.mark.parametrize("sigma", [0.02, 0.5])
def test_step_pld_beyond_the_range_of_exp(mods, sigma):
    # losses past 709, where e^u is not a double: at sigma = 0.02 probability is left there
    D, _ = mods
    h, t_max, p, k, nb = 0.25, 1000.0, 0.0256, 32, 400
    y, w = ac.envelope_bins(lambda v: ac.vertex_cdf(v, k), 0.0, 1.0 + 12.0 * math.sqrt(2.0 / k), nb)
    q, qi = D.dprc_pld_step(sigma, p, h, int(round(t_max / h)), _t(y), _t(w))
    grid, qr, qir = ac.single_step_pld(sigma, p, h, t_max, y, w)
    assert np.max(np.abs(q.cpu().numpy() - qr)) < 1e-13 and abs(qi.item() - qir) < 1e-13
    eps = [0.0, 299.75, 500.0, 720.25, 990.0]
    got = D.dprc_pld_delta(q, h, qi, _t(eps)).cpu().numpy()
    assert np.max(np.abs(got - [ac.delta_of_eps(grid, qr, qir, e) for e in eps])) < 1e-12


def test_step_pld_ignores_bins_without_weight(mods):
    # padding bins of weight zero, whatever their points hold, change nothing
    D, _ = mods
    y, w = np.linspace(0.4, 1.8, 70), np.linspace(1.0, 2.0, 70)
    w /= w.sum()
    pad = np.array([np.nan, -1.0, 0.0, np.inf] * 10)
    q, qi = D.dprc_pld_step(0.9, 0.2, 0.01, 700, _t(np.concatenate([pad, y, pad])),
                            _t(np.concatenate([0 * w[:40], w, 0 * w[:40]])))
    grid, qr, qir = ac.single_step_pld(0.9, 0.2, 0.01, 7.0, y, w)
    assert np.max(np.abs(q.cpu().numpy() - qr)) < 1e-13 and abs(qi.item() - qir) < 1e-13


@pytest.mark.parametrize("h", [1e-3, 100.0, 400.0])
def test_pld_delta_at_any_cell_width(mods, h):
    # cells so wide that e^(2h) is not a double; eps below, at, between and beyond the cells
    D, _ = mods
    L = 3001
    q = np.random.default_rng(3).random(L)
    q /= 1.01 * q.sum()
    qi = 1.0 - q.sum()
    grid = (np.arange(L) - (L - 1) // 2) * h
    eps = np.array([-1e308, -1000 * h, -h, 0.0, 0.5 * h, 700 * h, 1e308])
    got = D.dprc_pld_delta(_t(q), h, _t([qi]), _t(eps)).cpu().numpy()
    assert np.max(np.abs(got - [ac.delta_of_eps(grid, q, qi, e) for e in eps])) < 1e-12
    assert D.dprc_pld_delta(_t(q), h, _t([qi]), _t([np.nan])).item() == qi


@pytest.mark.parametrize("L", [1, 501, 14999, 15001])
def test_pld_fold_with_the_atom_in_place(mods, L):
    # q_inf may be one of the atoms that the call reads, or both
    D, _ = mods
    rng = np.random.default_rng(L)
    r = _t(rng.random(2 * L - 1) / L)
    ainf, binf = _t([0.125]), _t([0.25])
    q, qi = D.dprc_pld_fold(r, L, ainf, binf)
    out = torch.empty_like(q)
    for a, b in ((ainf, binf), (binf, _t([0.125]))):
        atom = a.clone()
        pair = (atom, b) if a is ainf else (b, atom)
        assert D.lib().dprc_pld_fold(r.data_ptr(), L, pair[0].data_ptr(), pair[1].data_ptr(), out.data_ptr(),
                                     atom.data_ptr(), D._stream(r.device)) == D.SUCCESS
        assert torch.equal(out, q) and torch.equal(atom, qi)
    half = D.dprc_pld_fold(r, L, ainf, ainf)
    both = ainf.clone()
    assert D.lib().dprc_pld_fold(r.data_ptr(), L, both.data_ptr(), both.data_ptr(), out.data_ptr(), both.data_ptr(),
                                 D._stream(r.device)) == D.SUCCESS
    assert torch.equal(out, half[0]) and torch.equal(both, half[1])


@pytest.mark.parametrize("L,n_eps", [(1, 1), (255, 512), (1023, 513), (4097, 700), (16385, 600), (20001, 3)])
def test_pld_delta_of_few_and_many_eps(mods, L, n_eps):
    # workgroups of 1024 and 256 threads, runs of 16 cells per thread that end inside the grid
    D, _ = mods
    q = np.random.default_rng(L).random(L)
    q /= 1.25 * q.sum()
    qi, h = 1.0 - q.sum(), 7.0 / L
    grid = (np.arange(L) - (L - 1) // 2) * h
    eps = np.linspace(-3.6, 3.6, n_eps)
    got = D.dprc_pld_delta(_t(q), h, _t([qi]), _t(eps)).cpu().numpy()
    assert np.max(np.abs(got - [ac.delta_of_eps(grid, q, qi, e) for e in eps])) < 1e-12


@pytest.mark.parametrize("L", [1, 191, 193, 14999, 15001, 40001])
def test_pld_fold_on_either_side_of_one_workgroup(mods, L):
    D, _ = mods
    r = np.random.default_rng(L).standard_normal(2 * L - 1)          # negatives are clipped
    q, qi = D.dprc_pld_fold(_t(r), L, _t([0.1]), _t([0.2]))
    v, c = np.maximum(r, 0.0), (L - 1) // 2
    ref = v[c:c + L].copy()
    ref[0] += v[:c].sum()
    inf0 = 1.0 - 0.9 * 0.8
    scale = (1.0 - inf0) / v.sum() if v.sum() > 0 else 0.0
    assert np.max(np.abs(q.cpu().numpy() - ref * scale)) < 1e-13
    assert abs(qi.item() - (inf0 + v[c + L:].sum() * scale)) < 1e-13
