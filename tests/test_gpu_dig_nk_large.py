"""The Newton-Krylov solve on meshes of many blocks: where the normalising
kernel stops adding the blocks' partial sums itself (1,536 blocks of 256 cells),
against the oracle, and its time beyond.  Tolerances are those of
test_gpu_dig_nk: counts exact, states within 1e-6 of the column's scale."""
import numpy as np
import pytest

from paper_2607_08195_amd import workloads as W
from oracle import Oracle

pytestmark = pytest.mark.gpu

GASES = {"argon": W.Species(),
         "nitrogen": W.Species(mass=4.65e-26, d_ref=4.17e-10, omega=0.74, T_ref=273.0, alpha=1.0, dof_rot=2,
                               z_rot=2.59)}


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_08195_amd import dsmc
    return dsmc


def _state(wl, nt):
    rng = np.random.default_rng(5)
    nv = 6 if wl.species.dof_rot else 5
    c = np.sqrt(W.KB / wl.species.mass * wl.run.T0)
    prim = np.empty((nt, nv))
    prim[:, 0] = wl.species.mass * wl.run.n0 * (1 + 0.01 * rng.random(nt))
    prim[:, 1:4] = 0.01 * c * rng.standard_normal((nt, 3))
    prim[:, 4:] = wl.run.T0 * (1 + 0.01 * rng.random((nt, nv - 4)))
    return prim, np.zeros((nt, 9 if nv == 5 else 12))


@pytest.mark.parametrize("n_hex,gas", [(40, "argon"), (41, "argon"), (41, "nitrogen")])  # 1,500 and 1,616 blocks
def test_many_blocks_match_oracle(D, n_hex, gas):
    wl = W.cavity(n_hex=n_hex, Kn=0.01, ppc=1, lid_speed=50.0, jitter=0.1, mesh_seed=1, species=GASES[gas])
    o = Oracle(wl, fill=False)
    o.set_reference(wl.run.n0, wl.run.T0)
    g = D.Simulation(wl, fill=False, capacity=1024)
    prim, hot = _state(wl, o.nt)
    kw = dict(n_m=1, eps_m=0.0, cfl=10.0, solver=1, krylov=4)
    pg, rg = g.dig_solve(prim, hot, **kw)
    po, ro = o.dig_solve(prim, hot, **kw)
    assert [rg[k] for k in ("iters", "krylov_steps", "failed")] == [ro[k] for k in ("iters", "krylov_steps", "failed")]
    scale = np.abs(po).max(axis=0, keepdims=True)
    scale[:, 1:4] = np.abs(po[:, 1:4]).max()
    assert np.all(np.abs(pg - po) <= 1e-6 * scale)
    g.close()


def test_time_of_normalising_grows_with_the_cells(D):
    """6,144 blocks: normalising a basis vector takes no more than twice the
    time of scaling the first one, which reads and writes as much."""
    from torch.profiler import ProfilerActivity, profile
    import torch
    wl = W.cavity(n_hex=64, Kn=0.05, ppc=1)
    g = D.Simulation(wl, fill=False, capacity=1024)
    prim, hot = _state(wl, g.nt)
    kw = dict(n_m=2, eps_m=0.0, cfl=100.0, solver=1, krylov=12)
    g.dig_solve(prim, hot, **kw)
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        g.dig_solve(prim, hot, **kw)
        torch.cuda.synchronize()
    t = {k: sorted(e.device_time_total for e in p.events() if k in e.name) for k in ("k_nk_normalize", "k_nk_scale")}
    g.close()
    if not all(t.values()):
        pytest.skip("no kernel times from the profiler")
    norm, scale = (v[len(v) // 2] for v in t.values())
    print(f"normalise {norm:.1f} us, scale {scale:.1f}")
    assert norm <= 2.0 * scale, (norm, scale)
