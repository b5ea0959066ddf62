"""The scan of the cell counts where its launches change, against the oracle:
one workgroup (up to 4,096 entries), block sums added by the workgroups behind
them (up to 128 blocks), block sums scanned by a kernel of their own.  Cells,
ids and their order are exact after steps that sort by it (criteria of
compare_particles)."""
import pytest

from oracle import Oracle
from paper_2607_08195_amd import workloads as W
from parity_util import compare_particles

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_08195_amd import dsmc
    return dsmc


# 6, 3,072 (one block), 4,374 (two), 16,464 (five), 546,750 cells (134 blocks)
@pytest.mark.parametrize("n_hex,ppc", [(1, 30), (8, 5), (9, 5), (14, 3), (45, 0.5)])
def test_sorted_order_matches_oracle(D, n_hex, ppc):
    wl = W.cavity(n_hex=n_hex, Kn=0.5, ppc=ppc, vel_fp32=0, n_ss=0)
    o, g = Oracle(wl), D.Simulation(wl)
    for _ in range(2):
        o.step(1)
        g.step(1)
        compare_particles(g.state(), o.particles(), 0)
    assert g.state(particles=False)["n"] == o.np
    g.close()


def test_inflow_counts_match_oracle(D):
    """The scan of the injected counts, over one and over two blocks."""
    for n in ((6, 4, 4), (8, 50, 50)):  # 224 and 8,200 inflow faces
        wl = W.open_box(n=n, ppc=2, vel_fp32=0)
        o, g = Oracle(wl), D.Simulation(wl)
        o.step(2)
        g.step(2)
        assert g.state(particles=False)["n"] == o.np
        compare_particles(g.state(), o.particles(), 0)
        g.close()
