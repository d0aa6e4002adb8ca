"""Several steps of a two-dimensional FP32 domain in one launch.

pflb_step and pflb_step_many take such domains several steps at a time: a workgroup steps
its tile and the sites around it in LDS.  The state may not depend on that by a single bit,
so every case is compared with the same steps taken one launch each (the PFLB_BZ override
of the launch shape), whose parity with the oracle has its own tests."""
import os

import pytest
import torch

import pfinputs

pytestmark = pytest.mark.gpu

W_, P_ = "wall", "periodic"


def _cfg(shape, bc, **kw):
    d = dict(lattice=9, shape=shape + (1,), bc=bc + (P_,), rho_L=1.0, rho_H=1000.0, nu_L=0.05,
             nu_H=0.01, M=0.1, W=4.0, sigma=1e-3, g=(2e-5, -1e-5, 0.0), eps=1e-10, hoc=1,
             dtheta_C=0.0)
    d.update(kw)
    return d


def _sim(cfg, seed, single):
    from paper_1812_00118_amd import Sim
    assert "PFLB_BZ" not in os.environ
    if single:
        os.environ["PFLB_BZ"] = "2"
    try:
        sim = Sim(cfg)
    finally:
        os.environ.pop("PFLB_BZ", None)
    sim.set_state(*pfinputs.random_state(9, cfg["shape"], seed=seed, h_noise=0.01, g_noise=0.01))
    return sim


def _same(a, b):
    # (random states of this density ratio diverge in places after some steps: both sides
    # then hold NaN in the same places)
    for x, y in zip(a.get_state(), b.get_state()):
        differ = (x != y) & ~(torch.isnan(x) & torch.isnan(y))
        assert not differ.any(), int(differ.sum())
        assert torch.isfinite(y).float().mean() > 0.9
    assert a.steps == b.steps


# the smallest periodic domains that take such launches and one site less (tile + 6), the
# ragged edges of each tile, each rule's side of its lines (512 tiles of 8x8, 256 of 16x16),
# domains narrower than a tile between walls
SIZES = [(14, 14), (13, 14), (64, 64), (65, 63), (128, 256), (129, 256), (250, 250), (272, 241),
         (257, 260), (22, 3000), (38, 2200), (37, 2200), (300, 700)]
BCS = [(P_, P_), (P_, W_), (W_, P_), (W_, W_)]


@pytest.mark.parametrize("bc", BCS, ids=["periodic", "walls-y", "walls-x", "walls-xy"])
@pytest.mark.parametrize("shape", SIZES + [(5, 3), (1, 40)], ids=lambda s: "%dx%d" % s)
def test_steps_per_launch(shape, bc):
    """2 to 7 steps in one call (every remainder a launch can leave)."""
    a, b = _sim(_cfg(shape, bc), 3, False), _sim(_cfg(shape, bc), 3, True)
    for n in (3, 2, 4, 7):
        a.step(n)
        b.step(n)
        _same(a, b)


@pytest.mark.parametrize("shape,n", [((20, 23), 3), ((67, 45), 17), ((131, 97), 5)],
                         ids=["small", "two-launches", "ragged"])
def test_batches(shape, n):
    """Contexts of different parameters and buffer parities in batched launches."""
    kinds = [dict(), dict(rho_H=10.0, sigma=5e-3, hoc=0), dict(rho_H=500.0, dtheta_C=0.1),
             dict(nu_L=0.02, nu_H=0.004, M=0.05, W=5.0)]
    from paper_1812_00118_amd import Sim
    cfgs = [_cfg(shape, (P_, W_), **kinds[k % 4]) for k in range(n)]
    a = [_sim(c, 10 + k, False) for k, c in enumerate(cfgs)]
    b = [_sim(c, 10 + k, True) for k, c in enumerate(cfgs)]
    for k in range(n):
        a[k].step(k % 5)
        b[k].step(k % 5)
    Sim.step_many(a, 11)
    for x, y in zip(a, b):
        y.step(11)
        _same(x, y)


@pytest.mark.parametrize("n", [4, 7, 8])
def test_graph_replays(n):
    """Replayed graphs of an odd and an even number of launches, eager steps between."""
    cfg = _cfg((90, 70), (P_, W_))
    a, b = _sim(cfg, 5, False), _sim(cfg, 5, True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        st.wait_stream(torch.cuda.default_stream())
        for k in range(4):
            a.step_graph(n)
            a.step(k)
            b.step(n + k)
            st.synchronize()
            _same(a, b)
    torch.cuda.synchronize()
