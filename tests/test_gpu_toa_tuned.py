"""GPU parity of the TOA pass at a caller's number of waves a chunk, which is
taken as it is: one, two and four waves on chunks of several tiles, with the
continuous wave and without, from a few chunks to more than the compute units;
the last pulsar's last tile holds one TOA.  Without a tuning the same data sets
take the library's own number.  Bars as in test_gpu_parity."""
import numpy as np
import pytest

import synth
from paper_2607_06834_amd import autotune
from test_gpu_parity import api, check, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def array(seed, counts, nf, cw):
    return synth.make_array(seed, len(counts), counts, 9 * synth.YEAR_S,
                            backends_per_psr=[1 + i % 3 for i in range(len(counts))], nu_range=(0.4e9, 2e9),
                            nf_rn=nf[0], nf_gw=nf[1], nf_dm=nf[2], has_cw=cw)


def near(ds, n, cw):
    th = synth.injected_theta(ds, 5, rn=(-14.0, 3.5), dm=(-14.0, 3.5),
                              cw=(0.3, 1.0, 8.7, -8.2, 0.5, 0.6, 0.9, -14.0) if cw else None)
    return synth.random_points(ds, n, 6, theta=th, theta_jitter=0.1)


@pytest.mark.parametrize("cw", [False, True])
@pytest.mark.parametrize("nf", [(6, 5, 0), (30, 14, 30)])
def test_small_array(api, nf, cw):  # noqa: F811
    ds = array(980, [500, 257, 513], nf, cw)
    X = near(ds, 17, cw)
    ref = check(ds, X, run(api, ds, X))
    for tuning in ((16, 1, 1), (16, 2, 1), (16, 4, 1), (33, 1, 0), (7, 2, 1)):
        check(ds, X, run(api, ds, X, tuning=tuning), ref=ref)


@pytest.mark.parametrize("waves", [1, 2])
def test_more_chunks_than_the_rule_takes(api, waves):  # noqa: F811
    """45 ragged pulsars with a CW, 17 chains, chunks as a server cuts them."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    counts = [300 + 53 * i % 977 for i in range(44)] + [705]
    ds = array(981, counts, (17, 17, 17), True)
    tiles = autotune.serving_tuning(ds["toa_offsets"], 17, n_cu)[0]
    chunks = sum(-(-((c + 15) // 16) // tiles) for c in counts)
    assert tiles > 1 and 3 * chunks >= n_cu
    X = near(ds, 17, True)
    pick = [0, 8, 16]
    got = run(api, ds, X, tuning=(tiles, waves, 2))
    check(ds, X[pick], tuple(g[pick] for g in got))
