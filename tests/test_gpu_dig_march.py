"""The pseudo-time iteration where its kernels' tiles end, against the CPU
oracle: sixteen cells to a wave and 64 to a workgroup (meshes of fewer cells
than a wave, of whole tiles and of ragged ones), and the state in either of the
two arrays that an iteration goes between (odd and even iteration counts, one
step for all cells, a solve that fails).

Tolerances are those of the coupling tests: residual 1e-11 of the column's
flux scale, states 1e-10 relative (pow within an ulp on each side, quotients
within one, over a few stable iterations); counts and flags exact.
"""
import numpy as np
import pytest

from paper_2607_08195_amd import workloads as W
from oracle import Oracle

pytestmark = pytest.mark.gpu

KB = 1.380649e-23
NITROGEN = dict(mass=4.65e-26, d_ref=4.17e-10, omega=0.74, T_ref=273.0, alpha=1.0, dof_rot=2, z_rot=2.59)


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_08195_amd import dsmc
    return dsmc


def _state(wl, nt, nv, spread):
    rng = np.random.default_rng(7)
    cs = np.sqrt(KB / wl.species.mass * wl.run.T0)
    p0 = wl.run.n0 * KB * wl.run.T0
    prim = np.empty((nt, nv))
    prim[:, 0] = wl.species.mass * wl.run.n0 * (1 + spread * rng.random(nt))
    prim[:, 1:4] = spread * cs * rng.standard_normal((nt, 3))
    prim[:, 4:] = wl.run.T0 * (1 + spread * rng.random((nt, nv - 4)))
    nh = 12 if nv == 6 else 9
    hot = 0.01 * p0 * rng.standard_normal((nt, nh))
    hot[:, 6:] *= cs
    return prim, hot


@pytest.mark.parametrize("gas", ["argon", "nitrogen"])
@pytest.mark.parametrize("n_hex", [1, 2, 3, 4])  # 6, 48, 162 and 384 cells
def test_tiles_match_oracle(D, gas, n_hex):
    kw = {} if gas == "argon" else dict(species=W.Species(**NITROGEN))
    wl = W.cavity(n_hex=n_hex, Kn=0.1, ppc=4, vel_fp32=0, jitter=0.1, lid_speed=50.0, **kw)
    o, g = Oracle(wl), D.Simulation(wl)
    nv = 5 if gas == "argon" else 6
    prim, hot = _state(wl, o.nt, nv, 0.05)
    rg, ro = g.dig_residual(prim, hot), o.dig_residual(prim, hot)
    assert np.all(np.abs(rg - ro) <= 1e-11 * np.abs(ro).max(axis=0, keepdims=True))
    hot *= 0.1
    for opt in [dict(n_m=1), dict(n_m=2), dict(n_m=7), dict(n_m=7, global_dt=1), dict(n_m=400, eps_m=0.3)]:
        opt = dict(dict(eps_m=0.0, cfl=0.4), **opt)
        pg, a = g.dig_solve(prim, hot, **opt)
        po, b = o.dig_solve(prim, hot, **opt)
        assert [a[k] for k in ("iters", "converged", "failed")] == [b[k] for k in ("iters", "converged", "failed")], opt
        scale = np.abs(po)
        scale[:, 1:4] = np.maximum(scale[:, 1:4], np.sqrt(KB / wl.species.mass * wl.run.T0))
        assert np.all(np.abs(pg - po) <= 1e-10 * scale), opt
    g.close()


@pytest.mark.parametrize("cfl", [2.0, 6.0, 40.0])
def test_failing_solve_matches_oracle(D, cfl):
    """Steps too long for the scheme: the solve fails at the oracle's
    iteration, and the state returned is that of the last good one."""
    wl = W.cavity(n_hex=3, Kn=0.1, ppc=4, vel_fp32=0, jitter=0.1, lid_speed=50.0)
    o, g = Oracle(wl), D.Simulation(wl)
    prim, hot = _state(wl, o.nt, 5, 0.3)
    opt = dict(n_m=60, eps_m=0.0, cfl=cfl)
    pg, a = g.dig_solve(prim, hot, **opt)
    po, b = o.dig_solve(prim, hot, **opt)
    assert (a["iters"], a["failed"]) == (b["iters"], b["failed"])
    assert np.isfinite(pg).all() and (pg[:, [0, 4]] > 0).all()
    if a["iters"] < 8:  # before rounding differences have grown with the instability
        assert np.all(np.abs(pg - po) <= 1e-8 * np.abs(po).max(axis=0, keepdims=True))
    g.close()
