"""GPU parity of the continuous wave where the caller's prior box lets its phase
grow without bound: Phi0 from the usual turn to the largest doubles, in the
per-TOA form (batched and plain) and in the standardized form's own basis.  Bars as in
test_gpu_parity and test_gpu_std."""
import numpy as np
import pytest

import synth
import test_gpu_std as ts
from oracle import std
from test_gpu_parity import api, check, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu

# beyond 2^60 the sum Phi0 + E / (32 X) is Phi0 in any order of rounding
PHI0 = np.array([1.0, -2.5, 3.0e6, 2.0 ** 61 + 4096.0, -1.0e19, 1.0e22, -3.7e40, 6381956970095103.0 * 2.0 ** 796,
                 1.1e150, -2.2e250, 1.7e300])


def box(ds, cw):
    ds["prior_lo"], ds["prior_hi"] = ds["prior_lo"].copy(), ds["prior_hi"].copy()
    ds["prior_lo"][cw + 4], ds["prior_hi"][cw + 4] = -2.0e300, 2.0e300


@pytest.mark.parametrize("tuning", [None, (16, 1, 1), (5, 2, 0), (33, 4, 1)])
@pytest.mark.parametrize("nf", [(6, 5, 0), (30, 14, 30)])
def test_phase_of_any_size(api, nf, tuning):  # noqa: F811
    ds = synth.make_array(990, 3, [300, 257, 513], 9 * synth.YEAR_S, backends_per_psr=[1, 2, 3], nu_range=(0.4e9, 2e9),
                          nf_rn=nf[0], nf_gw=nf[1], nf_dm=nf[2], has_cw=True)
    th = synth.injected_theta(ds, 5, rn=(-14.0, 3.5), dm=(-14.0, 3.5), cw=(0.3, 1.0, 8.7, -8.2, 0.5, 0.6, 0.9, -13.5))
    X = synth.random_points(ds, PHI0.size, 6, theta=th, theta_jitter=0.1)
    cw = ds["prior_lo"].size - 8
    box(ds, cw)
    X[:, cw + 4] = PHI0
    ref = check(ds, X, run(api, ds, X, tuning=tuning))
    if tuning is None:
        check(ds, X, run(api, ds, X, plain=True), ref=ref)


def test_phase_of_any_size_std(api):  # noqa: F811
    ds = ts.make(991, [140, 150], (8, 8, 1), cw=(9, 2.0))
    prep = std.StdPrepared(ds)
    X = ts.points(ds, prep, PHI0.size, 63, jitter=0.1)
    cw = prep.lay.cw
    box(ds, cw)
    X[:, cw + 4] = PHI0
    prep = std.StdPrepared(ds)
    ts.check(prep, X, ts.run(api, ds, X))
