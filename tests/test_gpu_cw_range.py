"""GPU parity of the continuous wave where the caller's prior box lets its phase
grow without bound: Phi0 from the usual turn to the largest doubles, in the
per-TOA form (batched and plain) and in the standardized form's own basis; and of
evolutions back in time beyond the range of 32 bits.  Bars as in test_gpu_parity
and test_gpu_std."""
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
    assert np.all(ref["status"] == 0)
    if tuning is None:
        check(ds, X, run(api, ds, X, plain=True), ref=ref)


@pytest.mark.parametrize("mass", [9.5, 20.0, 33.0, 36.0, 60.0, 110.0])
def test_evolution_back_in_time(api, mass):  # noqa: F811
    """Times up to zero: 1 - y from about 1 to 1e164 at the first TOA (at the chirp
    masses whose y is beyond 2^126 the 32-bit estimate of (1 - y)^(1/8) is infinite)."""
    ds = synth.make_array(992, 3, [300, 257, 513], 9 * synth.YEAR_S, backends_per_psr=[1, 2, 3], nu_range=(0.4e9, 2e9),
                          nf_rn=6, nf_gw=5, nf_dm=0, has_cw=True)
    ds["t"] = ds["t"] - ds["t"].max()
    th = synth.injected_theta(ds, 5, rn=(-14.0, 3.5), cw=(0.3, 1.0, 8.7, -8.2, 0.5, 0.6, 0.9, -13.5))
    X = synth.random_points(ds, 17, 6, theta=th, theta_jitter=0.1)
    cw = ds["prior_lo"].size - 8
    ds["prior_lo"], ds["prior_hi"] = ds["prior_lo"].copy(), ds["prior_hi"].copy()
    ds["prior_hi"][cw + 2], ds["prior_lo"][cw + 7] = 120.0, -60.0
    X[:, cw + 2] = mass + np.linspace(0.0, 0.5, 17)
    y = 51.2 * (10.0 ** X[:, cw + 2] * 4.925490947641e-6 * np.pi * 10.0 ** X[:, cw + 3]) ** (5.0 / 3.0) * \
        np.pi * 10.0 ** X[:, cw + 3] * -ds["t"].min()
    X[:, cw + 7] -= np.log10(1.0 + y) / 8.0         # the amplitude grows as (1 - y)^(1/8)
    ref = check(ds, X, run(api, ds, X))
    assert np.all(ref["status"] == 0)
    check(ds, X, run(api, ds, X, tuning=(16, 1, 1)), ref=ref)
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
