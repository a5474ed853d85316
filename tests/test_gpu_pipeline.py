"""Filtered-DNS pipeline kernels at the sizes where their tiles end: filter
segments and row groups, sample tiles; against the FP64 oracle.

Tolerances: the filter's outputs are sums of at most 255 x 255 FP64 products with
positive weights of sum 1, so both sides lie within about 2 * 255 * 2^-53 = 6e-14 of
the exact value relative to the largest output; inputs and targets as in the
other sample test (one FP32 rounding).
"""

import numpy as np
import pytest

from oracle import learned as L

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1705_09807_amd import learned
    return learned


def _fields(nx, ny, seed):
    r = np.random.default_rng(seed)
    m = 0.05 * r.standard_normal((5, ny, nx))
    m[0] += 1.0
    return m


@pytest.mark.parametrize("nx,ny,factor,delta", [
    (4, 4, 1, 0.7), (16, 16, 16, 3.0), (127, 9, 1, 3.0), (129, 140, 1, 80.0), (254, 12, 2, 5.0), (258, 34, 2, 9.0),
    (508, 28, 4, 2.0), (516, 60, 4, 16.0), (512, 136, 4, 87.0), (520, 48, 8, 24.0), (1040, 272, 16, 64.0),
    (48, 160, 16, 7.0),
    # several rows per workgroup, the last one's fewer; both sides of 2 R = 6 P
    (64, 3076, 4, 16.0), (64, 3076, 4, 17.0), (96, 3100, 2, 6.0), (96, 3080, 8, 24.0), (256, 3088, 16, 48.0)])
def test_filter_segments(nx, ny, factor, delta):
    G = _gpu()
    print("filter", nx, ny, factor, delta, flush=True)
    m = _fields(nx, ny, nx + ny)
    out = G.filter_subsample(torch.from_numpy(m).cuda(), factor, delta).cpu().numpy()
    want = L.filtered_fields(*m, factor, delta)
    for k in range(12):
        assert np.abs(out[k] - want[k]).max() <= 1e-13 * np.abs(want[k]).max(), k


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_filter_keeps_a_bad_cell_within_its_radius(bad):
    G = _gpu()
    nx, ny, factor, delta = 320, 96, 4, 8.0
    m = _fields(nx, ny, 3)
    x, y, R = 201, 50, 12  # R = ceil(5 * 8 / sqrt(12))
    m[1, y, x] = bad
    out = G.filter_subsample(torch.from_numpy(m).cuda(), factor, delta).cpu().numpy()
    X, Y = np.arange(nx // factor) * factor, np.arange(ny // factor) * factor
    hit = (np.abs(Y - y) <= R)[:, None] & (np.abs(X - x) <= R)[None, :]
    for k in (1, 5, 6, 11):  # m_x, m_x m_x / rho, m_x m_y / rho, (m_x B_y - m_y B_x) / rho
        assert np.array_equal(~np.isfinite(out[k]), hit), k
    for k in (0, 2, 3, 4, 7, 8, 9, 10):
        assert np.isfinite(out[k]).all(), k


@pytest.mark.parametrize("stencil", ["iso9", "central5"])
@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 7), (31, 8), (32, 9), (33, 17), (66, 33)])
def test_sample_tiles(nx, ny, stencil):
    G = _gpu()
    print("samples", nx, ny, stencil, flush=True)
    r = np.random.default_rng(nx * 100 + ny)
    c = 0.05 * r.standard_normal((12, ny, nx))
    c[0] += 1.0
    X, T = G.closure_samples(torch.from_numpy(c).cuda(), 4.0, stencil)
    X, T = X.cpu().numpy(), T.cpu().numpy()
    Xo = L.closure_features(c[0], c[1], c[2], c[3], c[4])
    To = (L.exact_subgrid(c) - L.analytic_subgrid(c[0], c[1], c[2], c[3], c[4], 4.0, stencil)).reshape(4, -1).T
    assert np.all(np.abs(X - Xo) <= 1.2e-7 * np.abs(Xo) + 1e-12)
    assert np.all(X[:, 63] == 0.0)
    assert np.all(np.abs(T - To).max(axis=0) <= 1e-6 * np.abs(To).max(axis=0))


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512, 1024, 2048])
def test_spectra_of_every_length(n):
    """Every transform length up to 2048 (4096 and beyond have closed forms in the
    other spectra test): white fields, so every bin holds energy.  FP64 on both
    sides: within 1e-13 of the total, as there, and equal when repeated."""
    from oracle import spectra as S
    G = _gpu()
    m = _fields(n, n, n)
    d = torch.from_numpy(m).cuda()
    got = G.spectra(d)
    want = (*S.energy_spectra(*m), S.x_spectrum(m[1] / m[0], m[2] / m[0]))
    for g, w in zip(got, want):
        assert np.abs(g.cpu().numpy() - w).max() <= 1e-13 * w.sum()
    for g, h in zip(got, G.spectra(d)):
        assert torch.equal(g, h)


@pytest.mark.parametrize("schedule,mag", [("fused", "d2q5"), ("fused", "d2q9"), ("aa", "d2q5")])
@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 4), (62, 9), (63, 64), (254, 7), (255, 33), (600, 19)])
def test_diagnostics_strips(nx, ny, schedule, mag):
    """Strip and segment edges of the diagnostics at both time parities: sums of the
    moments the library returns, in FP64 (about 30 roundings per term: 1e-13)."""
    _gpu()
    from paper_1705_09807_amd import Sim
    s = Sim(nx=nx, ny=ny, nu=1e-2, eta=1e-2, dtype="fp64", schedule=schedule, mag_lattice=mag)
    s.init_from_moments(torch.from_numpy(_fields(nx, ny, nx + ny)))
    for _ in range(2):
        s.step(1)
        d = s.diagnostics()
        rho, mx, my, bx, by = s.moments().cpu().numpy()
        ux, uy = mx / rho, my / rho
        ddx = lambda a: (np.roll(a, -1, 1) - np.roll(a, 1, 1)) / 2  # noqa: E731
        ddy = lambda a: (np.roll(a, -1, 0) - np.roll(a, 1, 0)) / 2  # noqa: E731
        w, jz, dv = ddx(uy) - ddy(ux), ddx(by) - ddy(bx), ddx(bx) + ddy(by)
        want = dict(mass=rho.sum(), e_kin=((mx ** 2 + my ** 2) / rho / 2).mean(), e_mag=((bx ** 2 + by ** 2) / 2).mean(),
                    enstrophy=(w ** 2 / 2).mean(), j2=(jz ** 2).mean(), divb_max=np.abs(dv).max(),
                    divb_rms=np.sqrt((dv ** 2).mean()))
        for k, v in want.items():
            assert abs(d[k] - v) <= 1e-13 * abs(v) + 1e-18, k
        for k, a in (("mom_x", mx), ("mom_y", my), ("bsum_x", bx), ("bsum_y", by)):
            assert abs(d[k] - a.sum()) <= 1e-13 * np.abs(a).sum(), k
        assert d["nonfinite"] == 0


@pytest.mark.parametrize("x,y", [(0, 0), (253, 3), (254, 8), (299, 40)])
def test_diagnostics_counts_a_bad_cell(x, y):
    _gpu()
    from paper_1705_09807_amd import Sim
    nx, ny = 300, 41
    s = Sim(nx=nx, ny=ny, nu=1e-2, eta=1e-2, dtype="fp64")
    s.init_from_moments(torch.from_numpy(_fields(nx, ny, 5)))
    st = s.get_state()
    st[11, y, x] = float("inf")
    s.set_state(st)
    d = s.diagnostics()
    assert d["nonfinite"] == 1 and np.isnan(d["mass"])


@pytest.mark.parametrize("n", [2, 255, 257, 1000, 65535, 65537, 200003])
def test_feature_stats_rows(n):
    """Row counts around the thread, workgroup and grid sizes, with columns whose mean
    is 1e4 spreads, whose first row is an outlier, and that are constant.  FP64
    statistics rounded to FP32: two FP32 roundings (2.4e-7) against numpy's."""
    G = _gpu()
    r = np.random.default_rng(n)
    X = r.standard_normal((n, 64)).astype(np.float32)
    X[:, 4] = (1.0 + 1e-4 * X[:, 4]).astype(np.float32)
    X[0, 13] = 3e4
    X[:, 22] = 0.1
    X[:, 63] = 0
    T = (1e-6 * r.standard_normal((n, 4))).astype(np.float32)
    T[:, 3] = 0
    m = G.Mlp(G.glorot_params(1))
    m.fit_norm(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda())
    nm = m.norm.cpu().numpy()
    c = X[:, 4:63:9].astype(np.float64)
    mean, sd = c.mean(0), c.std(0)
    assert np.all(np.abs(nm[:7] - mean) <= 2.4e-7 * np.abs(mean) + 1e-12)
    for f in (0, 1, 3, 4, 5, 6):
        assert abs(nm[8 + f] * sd[f] - 1) <= 2.4e-7, f
    assert nm[10] == 1.0 and nm[15] == 1.0
    rms = np.sqrt((T.astype(np.float64) ** 2).mean(0))
    assert np.all(np.abs(nm[16:19] - rms[:3]) <= 2.4e-7 * rms[:3]) and nm[19] == 1.0


def test_feature_stats_of_an_infinite_column():
    G = _gpu()
    X = np.random.default_rng(1).standard_normal((3000, 64)).astype(np.float32)
    X[0, 31] = np.inf
    m = G.Mlp(G.glorot_params(1))
    m.fit_norm(torch.from_numpy(X).cuda(), torch.zeros(3000, 4, device="cuda"))
    nm = m.norm.cpu().numpy()
    assert nm[3] == np.inf and nm[11] == 1.0
    assert np.isfinite(np.delete(nm[:20], 3)).all()
