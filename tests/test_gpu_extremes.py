"""Filters at the ends of the exponent range, where an intermediate result can
overflow though the value asked for does not.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2303_00301_amd import sampler
    return sampler


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("d", [2, 4, 16, 20, 33, 64])
def test_log_det_of_pivots_far_apart(S, d):
    """One step with S = P0 + Omega = Omega to the last bit: log det S is a sum of
    logarithms between 1e-150 and 1e155.  The last two of every four pivots
    multiply to 1e310; all four multiply to 1e10."""
    Om = np.resize([1e-150, 1e-150, 1e155, 1e155], d)
    M = S.DeviceModel.from_arrays(1, np.zeros(d), 1e-200 * np.eye(d), 0.5 * np.eye(d), np.eye(d), 1)
    _, _, ell, st = S.aux_filter(M, T(np.zeros((1, d))), T(Om[None]))
    terms = np.log(2.0 * np.pi) + np.log(Om)
    assert int(st[0]) == 0
    # a sum of d terms: half an ulp of its largest partial sum for each
    assert abs(float(ell[0]) + 0.5 * terms.sum()) < d * 2.0 ** -52 * np.abs(terms).sum()
