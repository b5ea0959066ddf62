"""MLP closure kernels (BF16 matrix cores, FP32 accumulation) against the
FP64 oracle, through the C ABI.

The oracle is evaluated with the kernels' precision contract (inputs,
weights, hidden activations and pre-activation gradients rounded to
bfloat16); the remaining differences are FP32 accumulation order and the
rare bfloat16 rounding flip of an activation whose FP32 value sits within an
ulp of a rounding boundary.  Criteria:
  * outputs: Frobenius 2e-3 relative; per element 1e-2 |ref| + 2e-3 rms(ref);
    against the plain FP64 network on bf16-rounded weights and inputs,
    Frobenius 2e-2;
  * gradients: per layer Frobenius 5e-3 relative; per element
    2e-2 |ref| + 5e-3 rms(layer); loss 1e-5 relative;
  * Adam from one gradient: within 2 FP32 ulps of the FP64 update;
  * ten full-batch Adam steps: parameter change within 5e-2 of the
    oracle's (Frobenius relative).
Row counts include ragged last tiles (the tile is 32 rows).
"""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_08195_amd import dsmc
    return dsmc


def _params(seed, scale=1.0):
    rng = np.random.default_rng(seed)
    ps = []
    for i, o in zip(M.LAYERS[:-1], M.LAYERS[1:]):
        ps.append(rng.uniform(-1, 1, i * o) * scale / np.sqrt(i))
        ps.append(rng.uniform(-0.1, 0.1, o))
    return np.concatenate(ps).astype(np.float32).astype(np.float64)


def _layer_slices():
    out, k = [], 0
    for i, o in zip(M.LAYERS[:-1], M.LAYERS[1:]):
        out.append(("W", slice(k, k + i * o)))
        k += i * o
        out.append(("b", slice(k, k + o)))
        k += o
    return out


@pytest.mark.parametrize("n", [1, 31, 32, 1000, 4133])
def test_forward_matches_oracle(D, n):
    p = _params(1)
    x = np.random.default_rng(2).standard_normal((n, 13)).astype(np.float32)
    net = D.Mlp()
    net.set_weights(p)
    y = net.forward(x).astype(np.float64)
    yo, _ = M.forward(p, x.astype(np.float64), bf16=True)
    d = np.abs(y - yo)
    rms = np.sqrt(np.mean(yo ** 2))
    assert np.linalg.norm(y - yo) <= 2e-3 * np.linalg.norm(yo)
    assert np.all(d <= 1e-2 * np.abs(yo) + 2e-3 * rms), d.max()
    y64, _ = M.forward(M.bf16_round(p), M.bf16_round(x.astype(np.float64)))
    assert np.linalg.norm(y - y64) <= 2e-2 * np.linalg.norm(y64)
    net.close()


@pytest.mark.parametrize("n", [7, 64, 1000])
def test_backward_matches_oracle(D, n):
    p = _params(3)
    rng = np.random.default_rng(4)
    x = rng.standard_normal((n, 13)).astype(np.float32)
    t = (0.3 * rng.standard_normal((n, 9))).astype(np.float32)
    net = D.Mlp()
    net.set_weights(p)
    loss, g = net.backward(x, t)
    lo, go = M.loss_and_grad(p, x.astype(np.float64), t.astype(np.float64), bf16=True)
    assert abs(loss - lo) <= 1e-5 * lo
    g = g.astype(np.float64)
    for kind, sl in _layer_slices():
        a, b = g[sl], go[sl]
        rms = np.sqrt(np.mean(b ** 2))
        assert np.linalg.norm(a - b) <= 5e-3 * np.linalg.norm(b), (kind, sl)
        assert np.all(np.abs(a - b) <= 2e-2 * np.abs(b) + 5e-3 * rms), (kind, sl)
    net.close()


def test_adam_step_matches_oracle(D):
    p = _params(5)
    g = (np.random.default_rng(6).standard_normal(p.size) * 1e-2).astype(np.float32)
    net = D.Mlp()
    net.set_weights(p)
    net.adam_step(g, lr=1e-3)
    net.adam_step(g * 0.5, lr=1e-3)
    q = net.get_weights().astype(np.float64)
    m = np.zeros_like(p); v = np.zeros_like(p)
    po, m, v = M.adam_step(p, g.astype(np.float64), m, v, 1, lr=1e-3)
    po, m, v = M.adam_step(po, 0.5 * g.astype(np.float64), m, v, 2, lr=1e-3)
    ulp = np.spacing(np.abs(po).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(q - po) <= 2 * ulp + 1e-9)
    net.close()


def test_full_batch_training_tracks_oracle(D):
    p = _params(7)
    rng = np.random.default_rng(8)
    teacher = _params(9, scale=1.5)
    x = rng.standard_normal((200, 13)).astype(np.float32)
    t, _ = M.forward(teacher, x.astype(np.float64))
    t = t.astype(np.float32)
    net = D.Mlp()
    net.set_weights(p)
    rep = net.train(x, t, steps=10, batch=0, lr=1e-3)
    q = net.get_weights().astype(np.float64)
    po, losses = M.train(p, x.astype(np.float64), t.astype(np.float64), [np.arange(200)] * 10, lr=1e-3, bf16=True)
    assert np.linalg.norm(q - po) <= 5e-2 * np.linalg.norm(po - p)
    assert abs(rep["loss_first"] - losses[0]) <= 1e-5 * losses[0]
    assert rep["loss_last"] == pytest.approx(losses[-1], rel=2e-2)
    net.close()


def test_minibatch_training_learns_a_teacher(D):
    rng = np.random.default_rng(10)
    teacher = _params(11, scale=1.5)
    x = rng.standard_normal((20000, 13)).astype(np.float32)
    t, _ = M.forward(teacher, x.astype(np.float64))
    net = D.Mlp()
    net.set_weights(_params(12))
    rep = net.train(x, t.astype(np.float32), steps=600, batch=512, lr=2e-3, seed=3)
    assert rep["loss_last"] < 0.1 * rep["loss_first"]
    xv = rng.standard_normal((2000, 13)).astype(np.float32)
    tv, _ = M.forward(teacher, xv.astype(np.float64))
    yv = net.forward(xv)
    assert np.mean((yv - tv) ** 2) < 0.1 * np.mean(tv ** 2)
    net.close()


def test_closure_in_couple_matches_oracle(D):
    """Closure inputs, network outputs and the gate inside dig_couple against
    the oracle's gradients, Kn_Delta and HoT composed with the MLP oracle."""
    from paper_2607_08195_amd import workloads as W
    from oracle import Oracle
    KB = 1.380649e-23
    wl = W.cavity(n_hex=6, Kn=0.1, ppc=20, vel_fp32=0, lid_speed=50.0)
    wl.run.ewma_on = 1
    wl.run.n_a = 50
    o = Oracle(wl)
    o.step(40)
    st = o.particles()
    g = D.Simulation(wl, fill=False, capacity=4 * o.np)
    g.set_state(st["x"], st["v"], st["cell"], st["pid"], o.step_index, o.next_pid, o.smax())
    g.set_sums(D.SAMPLE_EWMA, o.sums(1), o.ewma_counts())
    n_s = o.sums(1)[:, 0] * np.minimum(o.ewma_counts(), wl.run.n_a)
    assert n_s.min() > 0
    p = _params(21, scale=0.5)
    net = D.Mlp()
    net.set_weights(p)
    smp = o.dig_sampled()
    ok = np.isfinite(smp[:, 0]) & (smp[:, 0] > 0)
    prim = np.where(ok[:, None], smp[:, :5], o.mprev())
    kn = o.dig_kn_cell(prim, 1.0)
    grad = o.dig_gradients(prim)
    hot = np.where(ok[:, None], smp[:, 5:] - o.dig_nsf(prim, grad), 0.0)
    R = KB / wl.species.mass
    dc = 2.0 * np.cbrt(3.0 * o.volumes() / (4.0 * np.pi))
    x_o = M.closure_inputs(grad[:, :9], grad[:, 9:], prim[:, 4], kn, kn * dc, R)
    t_o = M.closure_targets(hot, prim[:, 0], prim[:, 4], R)
    s_o = M.closure_targets(smp[:, 5:], prim[:, 0], prim[:, 4], R)
    y_o, _ = M.forward(p, x_o.astype(np.float32).astype(np.float64), bf16=True)
    use_o, e_o = M.gate(y_o, t_o, s_o, tol=1e30, n_samples=n_s)
    assert use_o.all()
    # every cell takes the network: HoT = network output in physical units
    g.set_closure(net, gate_tol=1e30)
    kw = dict(kn_max=1e9, passes=0, n_m=0, feedback=0)
    r = g.dig_couple(**kw)
    assert r["n_closure"] == o.nt and r["n_fallback"] == 0
    xg, tg, vg = g.closure_data()
    assert vg.all()
    assert np.allclose(xg, x_o, rtol=2e-6, atol=1e-7 * np.abs(x_o).max())
    assert np.allclose(tg, t_o, rtol=2e-6, atol=1e-7 * np.abs(t_o).max())
    pp = prim[:, 0] * R * prim[:, 4]
    cs = np.sqrt(R * prim[:, 4])
    hot_exp = np.concatenate([y_o[:, :6] * pp[:, None], y_o[:, 6:] * (pp * cs)[:, None]], 1)
    hg = g.dig_get("hot")
    scale = np.abs(hot_exp).max(axis=0, keepdims=True)
    assert np.all(np.abs(hg - hot_exp) <= 1e-2 * np.abs(hot_exp) + 2e-3 * scale)
    # a threshold in the middle of the distance distribution: decisions agree
    # wherever the oracle's margin exceeds the bf16 resolution
    _, e_o = M.gate(y_o, t_o, s_o, tol=0.0, n_samples=n_s)
    tol = float(np.median(e_o))
    use_o, _ = M.gate(y_o, t_o, s_o, tol=tol, n_samples=n_s)
    g.set_closure(net, gate_tol=tol)
    r = g.dig_couple(**kw)
    assert r["n_closure"] + r["n_fallback"] == o.nt
    hg = g.dig_get("hot")
    took = np.all(np.isclose(hg, hot_exp, rtol=1e-2, atol=0), axis=1) & ~np.all(np.isclose(hg, hot, rtol=1e-9), axis=1)
    clear = np.abs(e_o - tol) > 2e-2 * tol
    assert np.array_equal(took[clear], use_o[clear])
    assert abs(r["n_closure"] - use_o.sum()) <= (~clear).sum()
    g.set_closure(None)
    r = g.dig_couple(**kw)
    assert r["n_closure"] == 0
    assert np.allclose(g.dig_get("hot"), hot, rtol=1e-9, atol=1e-9 * np.abs(hot).max())
    net.close()
    g.close()


@pytest.mark.parametrize("n", [33, 32768, 32769, 70001])
def test_forward_tiles_agree(D, n):
    """32-row tiles up to 32,768 rows, 64-row ones that the workgroups stride
    over beyond: a row's result does not depend on the tile it falls in, bit
    for bit, with inputs far into the SiLU's tails, infinities and NaN among
    them."""
    x = np.random.default_rng(12).standard_normal((n, 13)).astype(np.float32)
    x[::7] *= 1e3
    x[5] = np.inf
    x[n - 1, 3] = np.nan
    net = D.Mlp()
    net.set_weights(_params(1, 3.0))
    y = net.forward(x)
    for a in sorted({0, 16, 32752, max(0, n - 40)}):
        if a < n:
            part = net.forward(x[a:a + 40])
            assert np.array_equal(y[a:a + 40], part, equal_nan=True), a
    assert np.isnan(y[n - 1]).all() and np.isfinite(y[6:n - 1]).all()
    yo, _ = M.forward(_params(1, 3.0), x[6:32].astype(np.float64), bf16=True)
    assert np.linalg.norm(y[6:32] - yo) <= 2e-3 * np.linalg.norm(yo)
    net.close()


@pytest.mark.parametrize("n", [1, 33, 513, 4097])
def test_training_step_is_backward_then_adam(D, n):
    """A training step (reduction, optimiser and operand copies in one kernel)
    gives the weights, the loss and the next outputs of its parts, bit for bit."""
    rng = np.random.default_rng(13)
    x = rng.standard_normal((n, 13)).astype(np.float32)
    t = rng.standard_normal((n, 9)).astype(np.float32)
    a, b = D.Mlp(), D.Mlp()
    a.set_weights(_params(14))
    b.set_weights(_params(14))
    rep = a.train(x, t, steps=1, batch=0, lr=1e-2)
    loss, g = b.backward(x, t)
    b.adam_step(g, lr=1e-2)
    assert np.array_equal(a.get_weights(), b.get_weights()) and rep["loss_first"] == loss
    assert np.array_equal(a.forward(x), b.forward(x))
    a.close()
    b.close()
