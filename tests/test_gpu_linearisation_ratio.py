"""The log acceptance ratio of the rewritten linearisation kernels: every term of
the reverse pass reaches it and nothing else, so each quantity is held by its own
size (the parity suite's bounds: 1e-9 per time step and coordinate on the ratio,
1e-8 relative on the log marginal likelihoods)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_00301_amd import workloads as W
from tests.test_gpu_one_wave import _model
from tests.test_gpu_parity import S, _compare_step  # noqa: F401

pytestmark = pytest.mark.gpu


def _gaussian(rng, d, dy):
    m0, P0, F, b, Q = _model(rng, d)
    return dict(m0=m0, P0=P0, F=F, Q=Q, b=b, H=rng.standard_normal((dy, d)) / np.sqrt(d),
                R=0.5 * np.eye(dy) + 0.1 * np.ones((dy, dy)))


# the register forms for d, d_y <= 16 and <= 32 and the form past them; order 2's
# proposal is exact, so its ratio is zero by the cancellation of every term
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("N,d,dy", [(1, 1, 1), (7, 2, 1), (3, 16, 16), (21, 16, 3), (5, 17, 2),
                                    (5, 5, 17), (21, 20, 20), (6, 32, 32), (6, 31, 9), (5, 33, 4),
                                    (5, 4, 40), (4099, 2, 1)])
def test_gaussian(S, N, d, dy, order):  # noqa: F811
    rng = np.random.default_rng(N + 100 * d + dy)
    kw = _gaussian(rng, d, dy)
    M = S.DeviceModel.from_arrays(N, emit=S.EMIT_GAUSSIAN, **kw)
    r = _compare_step(S, oracle.Model(emit=W.EMIT_GAUSSIAN, **kw), M, rng.standard_normal((N, dy)),
                      rng.standard_normal((N, d)), 0.5, order, rng.standard_normal((2, N, d)), 1e-300)
    assert r["status"] == 0
    assert order == 1 or abs(r["log_ratio"]) < 1e-9 * N * d + 1e-9


@pytest.mark.parametrize("N,d,dy", [(1, 5, 3), (17, 64, 64), (9, 20, 33), (40, 64, 17)])
@pytest.mark.parametrize("repeat", [False, True])
def test_multivariate_t(S, N, d, dy, repeat):  # noqa: F811
    rng = np.random.default_rng(N + d + dy)
    site = rng.integers(0, d, size=dy) if repeat or dy > d else rng.permutation(d)[:dy]
    A = rng.standard_normal((dy, dy))
    m0, P0, F, b, Q = _model(rng, d)
    kw = dict(m0=m0, P0=P0, F=F, Q=Q, b=b, R=A @ A.T / dy + np.eye(dy),
              site=site.astype(np.int32), nu=2.0)
    M = S.DeviceModel.from_arrays(N, emit=S.EMIT_MVT, **kw)
    r = _compare_step(S, oracle.Model(emit=W.EMIT_MVT, **kw), M, rng.standard_normal((N, dy)),
                      rng.standard_normal((N, d)), 0.05, 1, rng.standard_normal((2, N, d)), 1e-9)
    assert r["status"] == 0
    torch.cuda.synchronize()
