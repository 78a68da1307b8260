"""GPU parity of the per-frequency kernels of 81 to 128 pulsars where the
diagonal-frequency workgroups come before the dense problems (more than two of
those per compute unit) and where they come after (fewer), on both sides of that
line, with diagonal red noise, DM and chains outside the prior box.  Every chain's
bits are those of a call with that chain alone.  Bars as in test_gpu_parity."""
import numpy as np
import pytest

from test_gpu_cholw import array
from test_gpu_parity import api, check, near, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nf,chains", [(82, (5, 4, 3), 128), (82, (5, 4, 3), 127), (97, (7, 2, 9), 257),
                                         (97, (7, 2, 0), 255), (113, (3, 30, 5), 17), (113, (9, 8, 2), 64)])
def test_diagonal_work_first_and_last(api, n, nf, chains):  # noqa: F811
    ds = array(n, nf, 930 + n)
    X = near(ds, chains, 13)
    X[3, 0] = ds["prior_hi"][0] + 1.0
    got = run(api, ds, X)
    pick = [0, 3, chains // 2, chains - 1]
    check(ds, X[pick], tuple(g[pick] for g in got))
    for c in (0, chains - 1):
        for a, b in zip(got, run(api, ds, X[[c]])):
            np.testing.assert_array_equal(a[[c]], b)
