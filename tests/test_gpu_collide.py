"""The collide and sample kernel at the edges of its stage, against the oracle.

Sorted cells of very unequal occupancy: empty, one particle, two, around the
ids a lane ranks at once (32, 33, 48, 49, 64, 65), runs of cells that do not
fit the LDS stage together (several windows), and one cell beyond the stage
(worked on in the particle store); on a mesh of few workgroups (16 cells
each) and of many (64 cells, every stage size), FP32 and FP64 velocities,
monatomic and rotating gas, every sort that changes how the kernel reaches
the particles.  Sort, collisions and sampling only (no move), so that the
occupancies stay; criteria of test_gpu_parity (pair counts bit-exact,
velocities within 1 float32 ulp or 1e-12, sums within 1e-12)."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2607_08195_amd import workloads as W
from parity_util import compare_particles, compare_sums

pytestmark = pytest.mark.gpu

STAGES = 4 | 8 | 16


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_08195_amd import dsmc
    return dsmc


def _state(wl, big):
    """Particles of the cells' prescribed counts: uniform in the cell,
    Maxwellian at T0, ids shuffled."""
    rng = np.random.default_rng(7)
    m = wl.mesh
    counts = rng.integers(0, 9, m.n_tets)
    edge = [0, 1, 2, 3, 31, 32, 33, 47, 48, 49, 63, 64, 65, 0, 130, 700]
    counts[:len(edge)] = edge
    counts[100:180] = 45                       # several windows of a chunk
    counts[250] = big                          # beyond any stage
    counts[-1] = 40
    cell = np.repeat(np.arange(m.n_tets), counts).astype(np.int32)
    b = rng.exponential(1.0, (len(cell), 4))
    b /= b.sum(axis=1, keepdims=True)
    x = np.einsum("ij,ijk->ik", b, m.xyz[m.tets[cell]])
    v = rng.normal(0.0, np.sqrt(W.KB * wl.run.T0 / wl.species.mass), (len(cell), 3))
    if wl.run.vel_fp32:
        v = v.astype(np.float32).astype(np.float64)
    pid = rng.permutation(len(cell)).astype(np.uint32)
    ir = rng.exponential(W.KB * wl.run.T0, len(cell)) if wl.species.dof_rot else None
    return x, v, cell, pid, ir


@pytest.mark.parametrize("n_hex,collide,sort,vel_fp32,gas", [
    (5, 3, 1, 1, "argon"), (5, 3, 1, 0, "vss"), (5, 3, 3, 1, "nitrogen"), (5, 3, 2, 0, "argon"),
    (5, 1, 1, 1, "nitrogen"), (5, 2, 3, 0, "argon"), (5, 4, 1, 1, "vss"), (5, 4, 2, 1, "argon"), (5, 0, 1, 0, "argon"),
    (18, 3, 1, 1, "argon"), (18, 3, 1, 0, "nitrogen")])
def test_uneven_cells_match_oracle(D, n_hex, collide, sort, vel_fp32, gas):
    sp = {"argon": W.Species(), "vss": W.Species(d_ref=4.11e-10, alpha=1.40),
          "nitrogen": W.Species(mass=4.65e-26, omega=0.74, dof_rot=2, z_rot=2.59)}[gas]
    wl = W.cavity(n_hex=n_hex, Kn=0.1, ppc=20, vel_fp32=vel_fp32, n_ss=0, species=sp)
    wl.run.dt *= 0.02  # the big cells' candidates grow with the square of their particles
    x, v, cell, pid, ir = _state(wl, 5000)
    o = Oracle(wl)  # (its initial (sigma c)_max)
    o.set_particles(x, v, cell, pid, 3, len(pid), ir=ir)
    g = D.Simulation(wl, fill=False, capacity=2 * len(pid))
    g.set_state(x, v, cell, pid, 3, len(pid), o.smax(), ir=ir)
    g.set_tuning(15, collide, sort)
    for k in range(2):
        o.step_stages(STAGES)
        g.step_stages(STAGES)
    gc, ga = g.pair_counts()
    oc, oa = o.pair_counts()
    assert np.array_equal(gc, oc) and np.array_equal(ga, oa)
    assert gc[250] > 256 and oa.sum() > 100
    gs, os_ = g.state(), o.particles()
    compare_particles(gs, os_, vel_fp32)
    if ir is not None:
        assert np.all(np.abs(gs["ir"] - os_["ir"]) <= 1e-12 * (np.abs(os_["ir"]) + W.KB * wl.run.T0))
        compare_sums(g.rot_sums(D.SAMPLE_STEADY)[0], o.rot_sums(0))
    compare_sums(g.sums(D.SAMPLE_STEADY)[0], o.sums(0))
    g.close()


@pytest.mark.parametrize("vel_fp32,gas", [(1, "argon"), (0, "vss"), (1, "nitrogen"), (0, "nitrogen")])
def test_gather_in_collide_matches_scatter(D, vel_fp32, gas):
    """The whole particle (position, velocity, id, cell, rotational energy)
    comes through the collide kernel's gather as it does through a scatter,
    bit for bit, over cells of every size and a few steps of motion."""
    sp = {"argon": W.Species(), "vss": W.Species(d_ref=4.11e-10, alpha=1.40),
          "nitrogen": W.Species(mass=4.65e-26, omega=0.74, dof_rot=2, z_rot=2.59)}[gas]
    wl = W.cavity(n_hex=5, Kn=0.1, ppc=20, vel_fp32=vel_fp32, n_ss=0, species=sp)
    wl.run.dt *= 0.02  # the big cells' candidates grow with the square of their particles
    x, v, cell, pid, ir = _state(wl, 5000)
    smax = Oracle(wl).smax()
    out = []
    for sort in (0, 1):
        g = D.Simulation(wl, fill=False, capacity=2 * len(cell))
        g.set_tuning(15, 3, sort)
        g.set_state(x, v, cell, pid, 0, len(cell), smax, ir=ir)
        g.step_stages(STAGES)
        first = g.state()
        g.step(3)
        out.append((first, g.state(), g.sums(D.SAMPLE_STEADY)[0]))
        g.close()
    for a, b in zip(out[0][:2], out[1][:2]):
        for k in ("x", "v", "cell", "pid") + (("ir",) if sp.dof_rot else ()):
            assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(out[0][2], out[1][2])
