"""The standardized form's results are the same bits on every call for the same
points, from arrays whose dense prior takes one wave a problem to those of four
(65 pulsars on), with enough problems that workgroups start on every SIMD; and a
chain's bits are those of a call with that chain alone."""
import numpy as np
import pytest

from oracle import std
from test_gpu_std import api, make, points, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chains", [(33, 40), (67, 64), (81, 40), (113, 40)])
def test_repeated_calls_are_bit_identical(api, n, chains):  # noqa: F811
    ds = make(800 + n, [90] * n, (14, 14, 0))
    X = points(ds, std.StdPrepared(ds), chains, 9)
    first = run(api, ds, X)
    assert np.all(first[2] == 0)
    for _ in range(6):
        for a, b in zip(first, run(api, ds, X)):
            np.testing.assert_array_equal(a, b)
    for c in (0, chains - 1):
        for a, b in zip(first, run(api, ds, X[[c]])):
            np.testing.assert_array_equal(a[[c]], b)
