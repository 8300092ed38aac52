"""Kernel variants at the sizes where their blocks begin and end, against the
CPU oracle.  Tolerances are those of test_gpu_parity.py: l relative 1e-10 and
the score 1e-8 of each component plus its rounding floor."""
import numpy as np
import pytest

import inputgen
from scorecheck import assert_score_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


@pytest.fixture(scope="module")
def exa():
    import paper_1908_06936_amd as exa

    return exa


# the 128 x 128 factor works in 16-wide steps: below, at and above one step,
# the last step, a whole block and the first rows of the next block
@pytest.mark.parametrize("n", [2, 15, 16, 17, 33, 112, 113, 127, 128, 129, 145])
def test_block_factor_step_edges(orc, exa, n):
    ctx = exa.Context(ts=128)
    x, y = inputgen.uniform(n, seed=100 + n)
    th = [1.2, 0.1, 0.9]
    z = orc.simulate(x, y, th, inputgen.normals(n, seed=n))
    ll_ref, g_ref = orc.loglik_grad(x, y, z, th)
    ll, g = ctx.loglik_grad(dev(x), dev(y), dev(z), th)
    assert ll == pytest.approx(ll_ref, rel=1e-10)
    assert_score_close(g, g_ref, n, th)


@pytest.mark.parametrize("pos", [1, 15, 16, 40, 112, 127, 128, 140])
def test_block_factor_reports_the_first_failed_pivot(exa, pos):
    # points on a line far apart (the covariance underflows to the identity
    # times sigma^2 = 4) except for two that coincide, so the second of the two
    # is the one failing pivot (4 - (4 / 2)^2 = 0 exactly), in Z-order column pos
    n = 150
    x = np.arange(n, dtype=np.float64) * 1000.0
    x[pos] = x[pos - 1]
    ctx = exa.Context(ts=256)
    st, ll, info = ctx.loglik_status(dev(x), dev(np.zeros(n)), dev(np.ones(n)), [4.0, 0.1, 0.5])
    assert st == exa.ENOTPD and ll == -np.inf and info == pos + 1


# n and tile sizes at which the launches of one call take 32-, 64- and 128-wide
# output blocks (chosen by the number of blocks), with ragged last tiles
@pytest.mark.parametrize("n,ts", [(640, 640), (900, 384), (1300, 128), (1409, 256), (2000, 128)])
def test_block_widths(orc, exa, n, ts):
    ctx = exa.Context(ts=ts)
    x, y = inputgen.uniform(n, seed=200 + n)
    th = [0.9, 0.12, 0.7]
    z = orc.simulate(x, y, th, inputgen.normals(n, seed=n))
    ll_ref, g_ref = orc.loglik_grad(x, y, z, th)
    ll, g = ctx.loglik_grad(dev(x), dev(y), dev(z), th)
    assert ll == pytest.approx(ll_ref, rel=1e-10)
    assert_score_close(g, g_ref, n, th)


# kriging and the Fisher information on the narrow blocks: few and many new
# points (blocks of 128 columns, ragged), one tile and several, padded last rows
@pytest.mark.parametrize("n,ts,m", [(130, 128, 1), (300, 512, 130), (900, 256, 700), (1100, 128, 1500)])
def test_kriging_block_widths(orc, exa, n, ts, m):
    ctx = exa.Context(ts=ts)
    x, y = inputgen.uniform(n, seed=300 + n)
    xn, yn = inputgen.uniform(m, seed=400 + m)
    th = [1.1, 0.1, 0.8]
    z = orc.simulate(x, y, th, inputgen.normals(n, seed=n))
    mean, mse = ctx.predict(dev(x), dev(y), dev(z), th, dev(xn), dev(yn))
    mean_ref, mse_ref = orc.predict(x, y, z, th, xn, yn)
    np.testing.assert_allclose(mean.cpu().numpy(), mean_ref, rtol=0, atol=1e-9 * np.abs(mean_ref).max())
    np.testing.assert_allclose(mse.cpu().numpy(), mse_ref, rtol=0, atol=1e-9 * th[0])


@pytest.mark.parametrize("n,ts,nugget", [(129, 128, 0.0), (400, 512, 0.0), (700, 128, 0.1), (900, 384, 0.0)])
def test_fisher_block_widths(orc, exa, n, ts, nugget):
    ctx = exa.Context(ts=ts)
    ctx.set_nugget(nugget)
    x, y = inputgen.uniform(n, seed=500 + n)
    th = [1.3, 0.1, 0.6]
    ref = orc.fisher(x, y, th, nugget)
    got = ctx.fisher(dev(x), dev(y), th)
    d = np.sqrt(np.diag(ref))
    assert np.max(np.abs(got - ref) / np.outer(d, d)) <= 1e-9


# the order of the locations by counting (up to 16,384 points) and by the
# bitonic network above: the sorted problem, and so every bit of l, does not
# depend on the caller's order
@pytest.mark.parametrize("n", [1, 255, 257, 511, 513, 2049, 16384, 16385])
def test_order_does_not_depend_on_the_callers(exa, n):
    ctx = exa.Context(ts=1024)
    ctx.set_dst_band(2)  # zeroes tiles by the order, and keeps the large ones cheap
    x, y = inputgen.uniform(n, seed=600 + n)
    z = inputgen.smooth_field(x, y, seed=n)
    th = [1.0, 0.002, 0.5]
    a = ctx.loglik(dev(x), dev(y), dev(z), th)
    p = inputgen.shuffled(n, seed=n)
    b = ctx.loglik(dev(x[p]), dev(y[p]), dev(z[p]), th)
    assert np.isfinite(a) and a == b


# DST likelihoods after other work has filled the workspace: the tiles outside
# the band are neither read nor written
@pytest.mark.parametrize("n,band", [(700, 1), (900, 2), (1000, 3)])
def test_dst_ignores_what_lies_outside_the_band(orc, exa, n, band):
    ctx = exa.Context(ts=128)
    x, y = inputgen.jittered_grid(32, seed=n)
    x, y = x[:n], y[:n]
    th = [1.0, 0.01, 0.5]
    z = inputgen.smooth_field(x, y, seed=n)
    X, Y, Z = dev(x), dev(y), dev(z)
    ctx.loglik_grad(X, Y, Z, [1.0, 0.1, 1.0])
    ctx.set_dst_band(band)
    ref = orc.loglik_dst(x, y, z, th, 128, band)
    assert ctx.loglik(X, Y, Z, th) == pytest.approx(ref, rel=1e-10)
    ll, g = ctx.loglik_grad(X, Y, Z, th)
    ll_ref, g_ref = orc.loglik_grad_dst(x, y, z, th, 128, band)
    assert ll == pytest.approx(ll_ref, rel=1e-10)
    assert_score_close(g, g_ref, n, th)


# block orders over the XCDs: below, at and past the size from which a tile's
# (or a tile row's) blocks go to one XCD together, against tiles of one block,
# which are always in dispatch order
@pytest.mark.parametrize("n,ts", [(11264, 256), (11265, 256), (12000, 512)])
def test_block_orders_over_the_xcds(exa, n, ts):
    x, y = inputgen.uniform(n, seed=700 + ts)
    z = inputgen.smooth_field(x, y, seed=n)
    th = [1.0, 0.02, 0.5]
    X, Y, Z = dev(x), dev(y), dev(z)
    ll, g = exa.Context(ts=ts).loglik_grad(X, Y, Z, th)
    ll_ref, g_ref = exa.Context(ts=128).loglik_grad(X, Y, Z, th)
    assert ll == pytest.approx(ll_ref, rel=1e-10)
    assert_score_close(g, g_ref, n, th)


# the same at sizes from which the trailing update, the inverse's update and the
# mixed inverse's update take whole tiles (ts = 256 and 768) and, at ts = 768 and in
# the contraction there, rows of a tile as chunks; the mixed score against FP64 at
# the 1e-6 that the default map is held to
@pytest.mark.parametrize("n,ts", [(17001, 256), (18601, 768)])
def test_block_orders_of_every_chunked_launch(exa, n, ts):
    x, y = inputgen.uniform(n, seed=900 + ts)
    z = inputgen.smooth_field(x, y, seed=n)
    th = [1.0, 0.02, 0.5]
    X, Y, Z = dev(x), dev(y), dev(z)
    ctx = exa.Context(ts=ts)
    ll, g = ctx.loglik_grad(X, Y, Z, th)
    ll_ref, g_ref = exa.Context(ts=128).loglik_grad(X, Y, Z, th)
    assert ll == pytest.approx(ll_ref, rel=1e-10)
    assert_score_close(g, g_ref, n, th)
    lm, gm = ctx.loglik_grad(X, Y, Z, th, "mixed")
    assert lm == pytest.approx(ll_ref, rel=1e-6)
    assert np.abs(np.subtract(gm, g_ref)).max() <= 1e-6 * np.abs(g_ref).max()


# entries at the ends of the table and of the fast forms: distances below and
# above e^-23 beta and 700 beta, zero, squares that overflow and nearly vanish,
# and ranges outside the short division, against the closed forms of nu = 1/2
# and 3/2 in extended precision
@pytest.mark.parametrize("beta", [1.0, 0.3, 3.0, 1e-120, 1e120])
@pytest.mark.parametrize("nu", [0.5, 1.5])
def test_matern_entries_at_the_ends(exa, nu, beta):
    ld = np.longdouble
    x = np.concatenate([
        np.exp(-23.0) * np.array([1e-3, 0.5, 1.0 - 1e-9, 1.0, 1.0 + 1e-9, 2.0]),
        np.array([1e-6, 1e-3, 0.25, np.sqrt(0.5), 1.0, np.sqrt(2.0), 2.0, 9.0, 100.0, 699.0, 699.999]),
        np.exp(-23.0 + 0.25 * np.array([1, 17, 60, 92, 93, 118])) * (1 + 1e-13)])
    r = np.concatenate([[0.0], x * beta, [701.0 * beta, 1e8 * beta]])
    if beta == 1.0:
        r = np.concatenate([r, [1e160]])
    cov = exa.Context(ts=128).matern_cov(dev(r), dev(np.zeros_like(r)), [1.7, beta, nu]).cpu().numpy()
    got = cov[0]
    q = r.astype(ld) / ld(beta)
    ref = ld(1.7) * np.exp(-q) * (1 if nu == 0.5 else 1 + q)
    ref[q > 700] = 0
    assert got[0] == 1.7 and np.all(got[q > 700] == 0)
    assert np.all(np.abs(got - ref) <= 1e-14 * ref)
    np.testing.assert_array_equal(cov, cov.T)


# z = L e by row blocks and shares of the tile columns: one tile, as many tiles as
# shares, more tiles than shares and a last block with one row
@pytest.mark.parametrize("n,ts", [(1, 128), (100, 256), (700, 128), (1025, 128), (4225, 128), (2049, 1024)])
def test_simulate_shares(orc, exa, n, ts):
    x, y = inputgen.uniform(n, seed=800 + n)
    th = [1.2, 0.05, 0.5]
    e = inputgen.normals(n, seed=n)
    z = exa.Context(ts=ts).simulate(dev(x), dev(y), th, dev(e)).cpu().numpy()
    # L is the factor in the library's order of the locations: z^T Sigma^-1 z =
    # e^T e whatever that order is, and every tile size has the same one
    assert z @ np.linalg.solve(orc.matern_cov(x, y, th), z) == pytest.approx(e @ e, rel=1e-9)
    other = exa.Context(ts=384).simulate(dev(x), dev(y), th, dev(e)).cpu().numpy()
    np.testing.assert_allclose(z, other, rtol=0, atol=1e-9 * np.abs(e).max())


# sigma2 and beta by powers of two: entries (exactly) and score scale with them, also
# where sigma2 (or sigma2 / beta) times the table's largest factor, x^nu e^x
# K_nu(x) near x = 700, would overflow
@pytest.mark.parametrize("ks,kb", [(950, 0), (-950, 0), (500, -500)])
@pytest.mark.parametrize("nu", [0.5, 2.0, 14.5])
def test_entries_and_score_scale_by_powers_of_two(exa, nu, ks, kb):
    ctx = exa.Context(ts=128)
    x = np.array([0.0, 0.25, 1.0, 3.0, 10.0, 40.0, 400.0, 640.0, 690.0, 699.0])
    y, th, big = np.zeros_like(x), [1.0, 1.0, nu], [2.0 ** ks, 2.0 ** kb, nu]
    X = dev(np.ldexp(x, kb))
    if kb == 0:
        a = ctx.matern_cov(dev(x), dev(y), th).cpu().numpy()
        b = ctx.matern_cov(X, dev(y), big).cpu().numpy()
        np.testing.assert_array_equal(b, np.ldexp(a, ks))
    ctx.set_nugget(0.1)
    z = np.cos(np.arange(x.size))
    l0, g0 = ctx.loglik_grad(dev(x), dev(y), dev(z), th)
    ctx.set_nugget(0.1 * 2.0 ** ks)
    l1, g1 = ctx.loglik_grad(X, dev(y), dev(np.ldexp(z, ks // 2)), big)
    assert l1 == pytest.approx(l0 - 0.5 * x.size * ks * np.log(2.0), rel=1e-13)
    assert_score_close([g1[0] * 2.0 ** ks, g1[1] * 2.0 ** kb, g1[2]], g0, x.size, th)
