"""GPU parity of the TOA pass where a data set has fewer chunks than the device
has compute units, so that a chunk is split over two, four or eight waves: full
tiles, remainders, chunks shorter than the waves, single TOAs; and of the
continuous wave's delay from phases of nothing to evolution up to the
coalescence.  Bars as in test_gpu_parity."""
import numpy as np
import pytest

import synth
from oracle import cw as ocw
from test_gpu_parity import api, check, near, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cw", [False, True])
@pytest.mark.parametrize("nf", [(6, 5, 0), (3, 9, 4), (17, 6, 12), (30, 30, 30)])
def test_wave_remainders(api, nf, cw):  # noqa: F811
    """Chunks of 1, 2, 3, 7, 8, 15 and 16 tiles, each with a last tile of 1, 15
    or 16 TOAs, at the default tuning and at two that cut them."""
    counts = [1, 16, 31, 33, 112, 113, 128, 129, 240, 255, 256, 257, 512]
    ds = synth.make_array(970, len(counts), counts, 9 * synth.YEAR_S, backends_per_psr=[1 + i % 3 for i in range(13)],
                          nu_range=(0.4e9, 2e9), nf_rn=nf[0], nf_gw=nf[1], nf_dm=nf[2], has_cw=cw)
    th = synth.injected_theta(ds, 5, rn=(-14.0, 3.5), dm=(-14.0, 3.5),
                              cw=(0.3, 1.0, 8.7, -8.2, 0.5, 0.6, 0.9, -14.0) if cw else None)
    X = synth.random_points(ds, 18, 6, theta=th, theta_jitter=0.1)
    ref = check(ds, X, run(api, ds, X))
    for tuning in ((9, 1, 1), (5, 2, 0)):
        check(ds, X, run(api, ds, X, tuning=tuning), ref=ref)


@pytest.mark.parametrize("y_max", [1e-9, 1e-4, 0.3, 0.9, 0.9999])
def test_cw_evolution(api, monkeypatch, y_max):  # noqa: F811
    """One chirp mass per evolution: the frequency is set so that the evolution
    variable reaches y_max at the last TOA.  The oracle forms y dE/dy - E as a
    difference, which loses the digits of 1 / y: its delay is taken in 80 bits
    here."""
    delay = ocw.delay

    def wide(t, pos, theta, want_grad=True):
        L = np.longdouble
        h, g = delay(np.asarray(t, L), np.asarray(pos, L), np.asarray(theta, L), want_grad)
        return np.asarray(h, np.float64), None if g is None else np.asarray(g, np.float64)

    monkeypatch.setattr(ocw, "delay", wide)
    ds = synth.cfg3()
    lo, hi = ds["prior_lo"].copy(), ds["prior_hi"].copy()
    lo[-6], hi[-6], lo[-5], hi[-5] = 3.0, 12.0, -12.0, -5.0
    ds["prior_lo"], ds["prior_hi"] = lo, hi
    th = synth.injected_theta(ds, 5, rn=(-14.0, 3.5), cw=(0.3, 1.0, 9.0, -8.0, 0.5, 0.6, 0.9, -14.0))
    X = synth.random_points(ds, 17, 6, theta=th, theta_jitter=0.0)
    X[:, lo.size - 6] = np.linspace(7.0, 10.0, 17)      # log10 Mc
    tmax = float(ds["t"].max())
    for c in range(17):
        p = X[c, lo.size - 8: lo.size]
        p[3] = -8.0
        p[3] += 3.0 / 8.0 * np.log10(y_max / ocw.max_y(p, tmax))
    assert np.all(X[:, lo.size - 5] > lo[-5]) and np.all(X[:, lo.size - 5] < hi[-5])
    check(ds, X, run(api, ds, X))
