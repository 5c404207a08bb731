"""The one-wave filter and sampler bodies (widths 16 and 32) at the edges of
their tiles: d and d_y on either side of a tile, blocks of one step, a single
time step.  Compared with the FP64 oracle; models are well conditioned (cond
below 1e3), so 64-bit recursions agree to 1e-9 (the bound of the parity tests).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_00301_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-9


@pytest.fixture(scope="module")
def S():
    from paper_2303_00301_amd import sampler
    return sampler


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def N_(t):
    return t.detach().cpu().numpy()


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def _model(rng, d):
    A = rng.standard_normal((d, d))
    return (rng.standard_normal(d), np.eye(d) + 0.1 * np.ones((d, d)),
            W.random_stable_F(rng, d, 0.9), 0.1 * rng.standard_normal(d),
            A @ A.T / d + 0.2 * np.eye(d))


@pytest.mark.parametrize("d", [1, 15, 16, 17, 31, 32])
@pytest.mark.parametrize("N,block", [(1, 0), (6, 1), (29, 4)])
def test_filter_and_sampler(S, d, N, block):
    rng = np.random.default_rng(100 * d + N)
    m0, P0, F, b, Q = _model(rng, d)
    om, Om = rng.standard_normal((N, d)), rng.uniform(0.1, 2.0, size=(N, d))
    xi = rng.standard_normal((N, d))
    ref = oracle.kf(m0, P0, F, Q, np.eye(d), np.stack([np.diag(o) for o in Om]), om, b=b,
                    R_per_t=True)
    x_ref, rc = oracle.rts_sample(F, ref["mf"], ref["Pf"], ref["mp"], ref["Pp"], xi)
    assert ref["rc"] == 0 and rc == 0
    M = S.DeviceModel.from_arrays(N, m0, P0, F, Q, 1, b=b)
    mf, Pf, ell, st = S.aux_filter(M, T(om), T(Om), block=block)
    x, st2 = S.rts_sample(M, mf, Pf, T(xi), block=block)
    assert int(st[0]) == 0 and int(st2[0]) == 0
    for got, want in ((mf, ref["mf"]), (Pf, ref["Pf"]), (ell, ref["ell"]), (x, x_ref)):
        assert _rel(N_(got), want) < TOL


@pytest.mark.parametrize("d,dy", [(16, 3), (17, 17), (32, 5)])
def test_dense_gaussian_step(S, d, dy):
    """Order 2 with Gaussian emissions: the dense constant Omega."""
    rng = np.random.default_rng(d + dy)
    N = 21
    m0, P0, F, b, Q = _model(rng, d)
    H, R = rng.standard_normal((dy, d)) / np.sqrt(d), 0.5 * np.eye(dy) + 0.1 * np.ones((dy, dy))
    y, x = rng.standard_normal((N, dy)), rng.standard_normal((N, d))
    xi = rng.standard_normal((2, N, d))
    kw = dict(m0=m0, P0=P0, F=F, Q=Q, b=b, H=H, R=R)
    r = oracle.mh_step(oracle.Model(emit=W.EMIT_GAUSSIAN, **kw), y, x, 0.5, 2, xi[0], xi[1], 0.4)
    M = S.DeviceModel.from_arrays(N, emit=S.EMIT_GAUSSIAN, **kw)
    out = S.mh_step(M, T(y), T(x), 0.5, 2, T(xi), T([0.4]), block=4)
    assert int(out["status"][0]) == 0 and int(out["accepted"][0]) == 1
    assert _rel(N_(out["logZ_fwd"])[0], r["logZ_fwd"]) < TOL
    assert _rel(N_(out["logZ_rev"])[0], r["logZ_rev"]) < TOL
    assert _rel(N_(out["x_out"]), r["x_out"]) < TOL


@pytest.mark.parametrize("dx,dy", [(16, 16), (17, 16), (16, 17), (5, 32), (32, 1), (32, 17)])
@pytest.mark.parametrize("N,block", [(1, 0), (23, 4)])
def test_general_observations(S, dx, dy, N, block):
    """Log-likelihood and gradient (general H, R) on either side of one tile of
    observations; the gradient within the adjoint tests' bound."""
    pw = W.lgssm_params(N=N, dx=dx, dy=dy, seed=dx + dy)
    t = pw.theta0
    ref = oracle.kf(pw.m0, pw.P0, t.F, np.diag(np.exp(t.logq)), t.H, np.diag(np.exp(t.logr)), pw.y)
    model = S.LGSSM(pw.m0, pw.P0, pw.y)
    th = (T(t.F), T(t.logq), T(t.H), T(t.logr))
    ll, ell, st, ws = S.lgssm_loglik(model, *th, block=block, ell=True)
    g = S.lgssm_loglik_grad(model, *th, ws, block=block)
    assert int(st[0]) == 0 and int(g[4][0]) == 0
    _, *g_ref = oracle.fisher_score(pw.m0, pw.P0, t.F, t.logq, t.H, t.logr, pw.y)
    for got, want in zip(g[:4], g_ref):
        assert np.linalg.norm(N_(got) - want) < 1e-8 * max(1.0, np.linalg.norm(want))
    assert _rel(N_(ell), ref["ell"]) < TOL
    assert abs(float(ll[0]) - ref["ell"].sum()) < TOL * max(1.0, abs(ref["ell"].sum()))


@pytest.mark.parametrize("N,d,block", [(17, 4, 1), (300, 3, 1), (260, 17, 1), (4200, 2, 1)])
def test_path_scan_levels(S, N, d, block):
    """Path sampler with one, two and three levels over the block aggregates."""
    rng = np.random.default_rng(N + d)
    m0, P0, F, b, Q = _model(rng, d)
    om, Om = rng.standard_normal((N, d)), rng.uniform(0.1, 2.0, size=(N, d))
    xi = rng.standard_normal((N, d))
    ref = oracle.kf(m0, P0, F, Q, np.eye(d), np.stack([np.diag(o) for o in Om]), om, b=b,
                    R_per_t=True)
    x_ref, rc = oracle.rts_sample(F, ref["mf"], ref["Pf"], ref["mp"], ref["Pp"], xi)
    M = S.DeviceModel.from_arrays(N, m0, P0, F, Q, 1, b=b)
    x, st = S.rts_sample(M, T(ref["mf"]), T(ref["Pf"]), T(xi), block=block)
    assert rc == 0 and int(st[0]) == 0
    assert _rel(N_(x), x_ref) < TOL


@pytest.mark.parametrize("N,d,dy", [(1, 5, 3), (17, 64, 64), (9, 20, 33), (40, 64, 17)])
@pytest.mark.parametrize("repeat", [False, True])
def test_multivariate_t_sites(S, N, d, dy, repeat):
    """Multivariate-t linearisation with time steps, sites and coordinates short of
    a tile, and with coordinates observed by several sites (dy > d needs them)."""
    rng = np.random.default_rng(N + d + dy)
    site = rng.integers(0, d, size=dy) if repeat or dy > d else rng.permutation(d)[:dy]
    A = rng.standard_normal((dy, dy))
    m0, P0, F, b, Q = _model(rng, d)
    kw = dict(m0=m0, P0=P0, F=F, Q=Q, b=b, R=A @ A.T / dy + np.eye(dy),
              site=site.astype(np.int32), nu=2.0)
    y, x = rng.standard_normal((N, dy)), rng.standard_normal((N, d))
    xi = rng.standard_normal((2, N, d))
    r = oracle.mh_step(oracle.Model(emit=W.EMIT_MVT, **kw), y, x, 0.05, 1, xi[0], xi[1], 1e-9)
    M = S.DeviceModel.from_arrays(N, emit=S.EMIT_MVT, **kw)
    out = S.mh_step(M, T(y), T(x), 0.05, 1, T(xi), T([1e-9]))
    assert int(out["status"][0]) == r["status"] and int(out["accepted"][0]) == r["accepted"]
    for k in ("logZ_fwd", "logZ_rev", "log_ratio"):
        assert abs(float(out[k][0]) - r[k]) < 1e-9 * N * d * max(1.0, abs(r["logZ_fwd"]))
    assert _rel(N_(out["x_out"]), r["x_out"]) < TOL


# width 64: factorisations by 2 x 2 blocks of 32, at the edges of the second
# block and of its tiles
@pytest.mark.parametrize("d", [33, 48, 49, 63, 64])
@pytest.mark.parametrize("N,block", [(1, 0), (29, 4)])
def test_width_64(S, d, N, block):
    test_filter_and_sampler(S, d, N, block)


# width 64, more steps than compute units: the sampler's elements are built by
# one wave per step
@pytest.mark.parametrize("d,N", [(33, 515), (49, 600), (64, 1025)])
def test_width_64_one_wave_build(S, d, N):
    test_filter_and_sampler(S, d, N, 0)


# Gaussian linearisation: columns in registers at the widths of the two register
# forms and past them, one step, a partial workgroup, more steps than waves
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("N,d,dy", [(1, 1, 1), (3, 16, 16), (5, 5, 17), (6, 32, 32), (5, 33, 4),
                                    (5, 4, 40), (4099, 2, 1)])
def test_gaussian_linearisation(S, N, d, dy, order):
    rng = np.random.default_rng(N + 10 * d + dy)
    m0, P0, F, b, Q = _model(rng, d)
    H, R = rng.standard_normal((dy, d)) / np.sqrt(d), 0.5 * np.eye(dy) + 0.1 * np.ones((dy, dy))
    y, x = rng.standard_normal((N, dy)), rng.standard_normal((N, d))
    xi = rng.standard_normal((2, N, d))
    kw = dict(m0=m0, P0=P0, F=F, Q=Q, b=b, H=H, R=R)
    r = oracle.mh_step(oracle.Model(emit=W.EMIT_GAUSSIAN, **kw), y, x, 0.5, order, xi[0], xi[1],
                       1e-300)
    M = S.DeviceModel.from_arrays(N, emit=S.EMIT_GAUSSIAN, **kw)
    out = S.mh_step(M, T(y), T(x), 0.5, order, T(xi), T([1e-300]))
    assert int(out["status"][0]) == 0 and int(out["accepted"][0]) == r["accepted"]
    assert _rel(N_(out["logZ_fwd"])[0], r["logZ_fwd"]) < TOL
    assert _rel(N_(out["logZ_rev"])[0], r["logZ_rev"]) < TOL
    assert _rel(N_(out["x_out"]), r["x_out"]) < TOL


# width 32: groups of eight blocks, and a last level of at most sixteen nodes
# that is chained instead of scanned
@pytest.mark.parametrize("N", [8, 16, 17, 128, 129])
def test_path_scan_levels_32(S, N):
    test_path_scan_levels(S, N, 17, 1)


def test_noalloc_default_blocks_at_the_scratch_limit(S):
    """d = 64, N = 300: the default's blocks of two steps need more than the fixed
    scratch array, blocks of four fit it and are taken."""
    w = W.latent_field(N=300, d=64, n_sites=32)
    M = S.DeviceModel.from_workload(w)
    args = (M, T(w.y), T(w.x_true), w.delta, w.order, T(w.normals(1)[0]), T(w.uniforms(1)[:1]))
    ref = S.mh_step(*args, block=4)
    f, i = dict(dtype=torch.float64, device="cuda"), dict(dtype=torch.int32, device="cuda")
    new = lambda: (torch.empty_like(args[2]), torch.empty(1, **f), torch.empty(1, **i),
                   torch.empty(1, **f), torch.empty(1, **f), torch.empty(1, **i))
    out = new()
    S.mh_step_noalloc(*args, *out)
    torch.cuda.synchronize()
    assert int(out[5][0]) == 0 and int(out[2][0]) == int(ref["accepted"][0])
    assert _rel(N_(out[0]), N_(ref["x_out"])) < 1e-12
    assert _rel(N_(out[3]), N_(ref["logZ_fwd"])) < 1e-12
    with pytest.raises(RuntimeError):
        S.mh_step_noalloc(*args, *new(), block=2)
