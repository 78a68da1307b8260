"""GPU parity of the standardized form's factorisations at the edges of their
tiles: the pulsar matrices (P rows) and the per-frequency matrices (n pulsars)
each at a full tile, at one row more and at one tile's remainder, from one tile
to eight, so that every number of waves and of tiles a wave holds is met, with
the shared form (k_std_fwd, k_std_prior_dense, k_std_bwd) and with split
coefficients (k_split_fac, k_split_bwd, k_split_bwd_c).  Bars as in
test_gpu_std."""
import numpy as np
import pytest

from oracle import std
from test_gpu_std import api, check, make, points, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu

COEFS = [(1, 1, 0), (12, 9, 4), (13, 5, 4), (20, 16, 4), (25, 2, 0), (30, 30, 2), (30, 3, 3), (20, 10, 20),
         (30, 4, 11), (30, 2, 18), (30, 2, 19), (30, 2, 26), (30, 2, 27)]   # P = 2, 32, 34, 48, 50, ... 112, 114


def _case(api, n, nf, split):  # noqa: F811
    ds = make(700 + n, [130] * n, nf)
    ds["split"] = split
    prep = std.StdPrepared(ds)
    X = points(ds, prep, 2, 71 + n)
    beta = np.array([1.0, 0.4])
    check(prep, X, run(api, ds, X, beta), beta=beta)


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("nf", COEFS)
def test_elimination_coefficient_tiles(api, nf, split):  # noqa: F811
    _case(api, 2, nf, split)


@pytest.mark.parametrize("n", [15, 32, 48, 49, 64, 80, 81, 96, 97, 112, 113])
def test_elimination_pulsar_tiles(api, n):  # noqa: F811
    _case(api, n, (2, 2, 0), 0)
