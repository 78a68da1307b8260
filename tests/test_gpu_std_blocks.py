"""GPU parity of the standardized form's kernels that take 16 chains as the
columns of matrix products (k_std_cw_fwd, k_std_cw_bwd, k_split_comb): bases of
2 K_D coefficients and 2 K_D + 1 sample times at a full 16-row tile, one row
more and a remainder of four, coefficient counts likewise, and one chain, a
full block of chains and one chain more.  Every chain's bits are those of a
call with that chain alone.  Bars as in test_gpu_std."""
import numpy as np
import pytest

from oracle import std
from test_gpu_std import api, check, make, points, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu

# (chains, coefficients (nf_rn, nf_gw, nf_dm), K_D or None): P = 2, 16, 18, 32, 34, 112, 114, 120
BLOCKS = [(1, (1, 1, 0), 1), (16, (8, 8, 0), 8), (17, (8, 8, 1), 9), (2, (16, 5, 0), 32), (17, (4, 4, 2), 33),
          (3, (30, 2, 26), 63), (2, (30, 2, 27), 64), (17, (30, 2, 30), 2)]


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("n,nf,kd", BLOCKS)
def test_chain_blocks(api, n, nf, kd, split):  # noqa: F811
    ds = make(610 + n, [140, 150], nf, cw=(kd, 2.0))
    ds["split"] = split
    prep = std.StdPrepared(ds)
    X = points(ds, prep, n, 63)
    beta = np.linspace(1.0, 0.3, n)
    got = run(api, ds, X, beta)
    pick = sorted({0, n // 2, n - 1})
    check(prep, X[pick], tuple(g[pick] for g in got), beta=beta[pick])
    one = run(api, ds, X[[n - 1]], beta[[n - 1]])
    for a, b in zip(got, one):
        np.testing.assert_array_equal(a[[n - 1]], b)
