"""The square root and the reciprocal of a triangularisation's pivot are correctly
rounded.  One step of a diagonal model in FP64 is, per coordinate, with u = sqrt(P0)
and s = sqrt(Omega),
    g = fma(u, u, s s),  l = u^2 (1 / sqrt(g)),  U = sqrt(fma(-l, l, u^2)),
(zero for a pivot <= 0), so that the updated factor U tells every bit of both."""
import math
from fractions import Fraction

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
D = 32


@pytest.fixture(scope="module")
def S():
    from paper_2303_00301_amd import sampler
    return sampler


def _expected(P0, Om):
    u, s = math.sqrt(P0), math.sqrt(Om)
    g = float(Fraction(u) ** 2 + Fraction(s * s))
    l = (u * u) * (1.0 / math.sqrt(g))
    p = float(Fraction(u * u) - Fraction(l) ** 2)
    return math.sqrt(p) if p > 0.0 else 0.0


# mantissas next to powers of two and anywhere, exponents of both parities; Omega
# from far below P0 (the second pivot is rounding, or not positive) to far above
@pytest.mark.parametrize("mantissa", ["one", "above one", "below two", "any"])
def test_pivots_are_correctly_rounded(S, mantissa):
    rng = np.random.default_rng(len(mantissa))
    zeros = n = 0
    for call in range(16):
        e = rng.integers(-400, 400, D)
        m = {"one": np.ones(D), "above one": 1.0 + rng.integers(0, 4, D) * 2.0 ** -52,
             "below two": 2.0 - rng.integers(1, 5, D) * 2.0 ** -52,
             "any": rng.uniform(1.0, 2.0, D)}[mantissa]
        P0 = np.ldexp(m, e)
        Om = np.ldexp(rng.uniform(1.0, 2.0, D), e + rng.integers(-56, 20, D))
        T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
        M = S.DeviceModel.from_arrays(1, np.zeros(D), np.diag(P0), 0.5 * np.eye(D), np.eye(D), 1)
        o = S.sqrt_filter_sample(M, T(np.zeros((1, D))), T(Om[None]), dtype="f64")
        got = o["Uf"].cpu().numpy()[0]
        want = np.array([_expected(*c) for c in zip(P0.tolist(), Om.tolist())])
        assert np.array_equal(got, np.diag(want)), np.flatnonzero(np.diag(got) != want)
        zeros += int((want == 0.0).sum())
        n += D
    assert 0 < zeros < n // 2  # pivots <= 0 are among them
