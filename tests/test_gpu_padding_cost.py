"""Work that a small problem need not pay for: what padding is left out, is left
out of the time too, and the results at the edges of what is left out are the
oracle's.  Times are minima over bursts, compared within one process.
"""
import numpy as np
import pytest
import torch

from tests.test_gpu_sqrt import _check, _model

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2303_00301_amd import sampler
    return sampler


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _us(f, n=10):
    """Time of f from replays of a graph of n calls: the host is not in it."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        f()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(n):
            f()
    graph.replay()
    best = float("inf")
    for _ in range(8):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        graph.replay()
        e[1].record()
        e[1].synchronize()
        best = min(best, e[0].elapsed_time(e[1]) / n * 1e3)
    return best


# one to three columns in all, groups of four columns filled and not, the same in
# a second panel
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("N,d,block", [(40, 1, 0), (40, 2, 0), (9, 3, 1), (40, 4, 0), (9, 6, 2),
                                       (40, 8, 0), (23, 10, 4), (23, 21, 4)])
def test_square_root_columns(S, dtype, N, d, block):
    rng = np.random.default_rng(4000 + 11 * N + d)
    m0, P0, F, b, Q = _model(rng, d, 1e2)
    _check(S, m0, P0, F, b, Q, 0.5 * rng.standard_normal((N, d)), rng.uniform(0.05, 1.0, (N, d)),
           rng.standard_normal((N, d)), dtype, block)


def test_square_root_cost_of_one_coordinate(S):
    """Two columns to triangularise take well below the time of sixteen (117 us
    against 184 at T = 20; 183 against 199 with the padded columns eliminated)."""
    def run(d, N=20):
        rng = np.random.default_rng(d)
        m0, P0, F, b, Q = _model(rng, d, 1e1)
        M = S.DeviceModel.from_arrays(N, m0, P0, F, Q, 1, b=b)
        om, Om, xi = (T(a) for a in (rng.standard_normal((N, d)), rng.uniform(0.1, 1.0, (N, d)),
                                     rng.standard_normal((N, d))))
        return _us(lambda: S.sqrt_filter_sample(M, om, Om, xi))
    one, eight = run(1), run(8)
    print(one, eight)
    assert one < 0.8 * eight, (one, eight)


def test_sampler_build_while_every_step_has_a_cu(S):
    """Width 64, as many transitions as compute units (the last step has none):
    one team per CU, not the slower wave per step (150 us against 171)."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count

    def run(N, d=64):
        rng = np.random.default_rng(N)
        m0, P0, F, b, Q = _model(rng, d, 1e1)
        M = S.DeviceModel.from_arrays(N, m0, P0, F, Q, 1, b=b)
        om, Om = T(rng.standard_normal((N, d))), T(rng.uniform(0.1, 1.0, (N, d)))
        mf, Pf, _, _ = S.aux_filter(M, om, Om)
        xi = T(rng.standard_normal((N, d)))
        return _us(lambda: S.rts_sample(M, mf, Pf, xi))
    fits, more = run(n_cu + 1), run(n_cu + 44)
    print(fits, more)
    assert fits < 0.94 * more, (fits, more)
