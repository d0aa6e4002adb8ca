"""In-place steps of every compiled wall set on domains whose neighbour offsets wrap at once
(one and two sites an axis) and on ragged ones, against the float64 oracle.

Each step is a chain of fewer than 100 roundings of terms within a few times the largest
population: 300 u of it a step, u = 2^-24."""
import numpy as np
import pytest

import pfinputs
from oracle import pflbm as O

pytestmark = pytest.mark.gpu

W_, P_ = "wall", "periodic"
U32 = 2.0 ** -24
CASES = [(9, shape + (1,), bc + (P_,))
         for bc in ((P_, P_), (W_, P_), (P_, W_), (W_, W_)) for shape in ((1, 2), (2, 1), (33, 19))]
CASES += [(19, shape, bc) for bc in ((P_, P_, P_), (P_, P_, W_), (W_, P_, P_), (W_, W_, W_))
          for shape in ((1, 1, 1), (2, 1, 2), (17, 6, 9))]


@pytest.mark.parametrize("q,shape,bc", CASES, ids=str)
def test_inplace_steps_of_every_wall_set(q, shape, bc):
    from paper_1812_00118_amd import Sim
    cfg = dict(lattice=q, shape=shape, bc=bc, rho_L=1.0, rho_H=10.0, nu_L=0.05, nu_H=0.05, M=0.1,
               W=4.0, sigma=1e-3, g=(2e-5, -1e-5, 0.0), eps=1e-10, hoc=1, dtheta_C=0.0)
    prm = pfinputs.model_params(cfg)
    h0, g0 = pfinputs.random_state(q, shape, seed=3, h_noise=0.01, g_noise=0.01)
    sim = Sim(prm, storage="fp32_inplace")
    sim.set_state(h0, g0)
    for _ in range(3):
        # from the state that the domain holds, in either layout
        h, g = (t.cpu().numpy().astype(np.float64) for t in sim.get_state())
        h, g = O.step(O.Params.from_dict(prm), h, g)
        sim.step(1)
        h1, g1 = (t.cpu().numpy().astype(np.float64) for t in sim.get_state())
        for a, r in ((h1, h), (g1, g)):
            assert np.abs(a - r).max() <= 300 * U32 * max(np.abs(h).max(), np.abs(g).max())
