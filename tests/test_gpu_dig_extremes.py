"""Macroscopic solves at the ends of their range, against the CPU oracle.

Tolerances are those of the marching's tests: states 1e-10 relative (velocities
against the thermal speed), counts and flags exact."""
import numpy as np
import pytest

from paper_2607_08195_amd import workloads as W
from oracle import Oracle

pytestmark = pytest.mark.gpu

KB = 1.380649e-23
GASES = {"argon": W.Species(),
         "nitrogen": W.Species(mass=4.65e-26, d_ref=4.17e-10, omega=0.74, T_ref=273.0, alpha=1.0, dof_rot=2, z_rot=2.59)}


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_08195_amd import dsmc
    return dsmc


def _states_close(pg, po, wl, rel):
    scale = np.abs(po)
    scale[:, 1:4] = np.maximum(scale[:, 1:4], np.sqrt(KB / wl.species.mass * wl.run.T0))
    assert np.all(np.abs(pg - po) <= rel * scale)


# A normal number, the largest density whose reciprocal overflows, subnormal
# ones, and one where the viscous rate overflows (the cell's step is zero).
@pytest.mark.parametrize("rho", [1e-300, 5e-309, 1e-310, 1e-312])
@pytest.mark.parametrize("gas", ["argon", "nitrogen"])
def test_near_vacuum_matches_oracle(D, gas, rho):
    """Half of the cells at a density close to zero, by which their conserved
    values are divided at every stage."""
    wl = W.cavity(n_hex=5, Kn=0.1, ppc=4, vel_fp32=0, jitter=0.1, lid_speed=50.0, species=GASES[gas])
    o, g = Oracle(wl), D.Simulation(wl)
    nv = 5 if gas == "argon" else 6
    prim = np.zeros((o.nt, nv))
    prim[:, 0] = wl.species.mass * wl.run.n0
    prim[:, 1] = 0.1
    prim[:, 4:] = wl.run.T0
    prim[wl.mesh.xyz[wl.mesh.tets].mean(axis=1)[:, 0] < 0.5, 0] = rho
    hot = np.zeros((o.nt, 9 if nv == 5 else 12))
    for n_m, one in [(1, 0), (4, 0), (4, 1)]:
        kw = dict(n_m=n_m, eps_m=0.0, cfl=0.4, global_dt=one)
        pg, a = g.dig_solve(prim, hot, **kw)
        po, b = o.dig_solve(prim, hot, **kw)
        assert (a["iters"], a["failed"]) == (b["iters"], b["failed"]) == (n_m, 0)
        _states_close(pg, po, wl, 1e-10)
    g.close()
