"""The no-allocation step's scan block at the limit of its scratch array."""
import numpy as np
import pytest
import torch

from paper_2303_00301_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2303_00301_amd import sampler
    return sampler


@pytest.mark.parametrize("N", [96, 300])  # blocks of two fit; only blocks of four do
def test_negative_block_is_refused(S, N):
    w = W.latent_field(N=N, d=64, n_sites=32)
    M = S.DeviceModel.from_workload(w)
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    f, i = dict(dtype=torch.float64, device="cuda"), dict(dtype=torch.int32, device="cuda")
    y, x = T(w.y), T(w.x_true)
    out = (torch.zeros_like(x), torch.empty(1, **f), torch.empty(1, **i), torch.empty(1, **f),
           torch.empty(1, **f), torch.empty(1, **i))
    with pytest.raises(RuntimeError, match="block must be >= 0"):
        S.mh_step_noalloc(M, y, x, w.delta, w.order, T(w.normals(1)[0]), T(w.uniforms(1)[:1]), *out,
                          block=-1)
    torch.cuda.synchronize()
    assert not out[0].any()
