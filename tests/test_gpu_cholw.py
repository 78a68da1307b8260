"""GPU parity of the four-wave per-frequency factorisation and adjoint
(k_cholw, arrays of 81 to 128 pulsars): full tiles, one row of a tile and the
sizes whose block columns pair differently (six, seven and eight tiles), with
the diagonal-frequency workgroups of the same launch (frequencies beyond the
common ones, DM), more dense problems than two per compute unit, chains outside
the prior box beside valid ones, common-only and noise-free frequencies, and
whole trajectories through a graph.  Bars as in test_gpu_parity."""
import numpy as np
import pytest

import synth
from oracle import model
from test_gpu_parity import api, check, near, run  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def array(n, nf, seed):
    return synth.make_array(seed, n, [14 + (i % 5) for i in range(n)], 10 * synth.YEAR_S,
                            backends_per_psr=[1 + i % 2 for i in range(n)], nu_range=(0.4e9, 2e9),
                            nf_rn=nf[0], nf_gw=nf[1], nf_dm=nf[2])


@pytest.mark.parametrize("n,nf,chains", [(82, (4, 2, 3), 3), (96, (3, 3, 0), 17), (111, (0, 2, 1), 2),
                                         (112, (2, 4, 2), 5), (120, (5, 1, 5), 18), (127, (3, 3, 2), 4)])
def test_tile_remainders(api, n, nf, chains):  # noqa: F811
    ds = array(n, nf, 900 + n)
    X = np.concatenate([near(ds, chains, 9), synth.random_points(ds, 2, 10)])
    X[0, 0] = ds["prior_hi"][0] + 1.0
    check(ds, X, run(api, ds, X))


def test_many_problems(api):  # noqa: F811
    """116 pulsars, 20 common frequencies, 40 chains: 800 dense problems."""
    ds = array(116, (20, 20, 4), 950)
    X = near(ds, 40, 11)
    lp, gr, st = run(api, ds, X)
    idx = [0, 17, 39]
    check(ds, X[idx], (lp[idx], gr[idx], st[idx]))
    again = run(api, ds, X)
    np.testing.assert_array_equal(lp, again[0])
    np.testing.assert_array_equal(gr, again[1])


def test_graph_matches_eager(api):  # noqa: F811
    ds = array(115, (4, 3, 2), 960)
    g = api.Dataset(ds)
    x0 = torch.tensor(near(ds, 6, 12), device="cuda")
    got = []
    for use_graph in (True, False):
        x = x0.clone()
        lp, gr, _ = g.ptafs_logp_grad(x)
        acc = torch.zeros(6, dtype=torch.int64, device="cuda")
        im = torch.ones(g.d, dtype=torch.float64, device="cuda")
        im[: ds["prior_lo"].size] = 1e-8
        for t in range(3):
            g.ptafs_hmc_run(x, lp, gr, acc, n_traj=1, n_leapfrog=4, eps=1e-3, seed=5, traj0=t, inv_mass=im,
                            use_graph=use_graph)
            torch.cuda.synchronize()
        got.append((x.cpu(), lp.cpu(), gr.cpu(), acc.cpu()))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    ref = model.logp_grad(model.Prepared(ds), got[0][0].numpy())
    check(ds, got[0][0].numpy(), (got[0][1].numpy(), got[0][2].numpy(), ref["status"]), ref=ref)
