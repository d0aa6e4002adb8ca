"""The read-out at the edges of its tiles: domains of one site, smaller than a tile, ragged in
every axis and of several chunks along z, with and without walls and contact angles.

The reference is the float64 oracle on the populations that the state holds, so only the
read-out's own rounding differs: phi is a sum of Q terms (Q u sum|h|, u = 2^-24), and the
other fields are chains of fewer than 60 roundings of terms within 5 times the field's
largest value (300 u of it)."""
import numpy as np
import pytest

import pfinputs
from oracle import pflbm as O

pytestmark = pytest.mark.gpu

W_, P_ = "wall", "periodic"
U32 = 2.0 ** -24


def cases():
    for bc in ((P_, P_), (W_, P_), (P_, W_), (W_, W_)):
        for shape in ((1, 1), (5, 3), (31, 8), (33, 9), (64, 64), (100, 37)):
            yield 9, shape + (1,), bc + (P_,), None
    yield 9, (40, 30, 1), (P_, W_, P_), (0.0, 0.0, 0.5, -0.3, 0.0, 0.0)
    for bc in ((P_, P_, P_), (P_, P_, W_), (W_, W_, W_)):
        for shape in ((1, 1, 1), (3, 5, 2), (63, 4, 7), (65, 9, 13), (130, 5, 40)):
            yield 19, shape, bc, None
    yield 19, (66, 6, 9), (P_, P_, W_), (0.0, 0.0, 0.0, 0.0, 0.5, -0.3)
    # past the size from which three-dimensional domains are read in one pass
    for bc in ((P_, P_, P_), (W_, W_, W_)):
        yield 19, (131, 106, 113), bc, None
    yield 19, (131, 106, 113), (P_, P_, W_), (0.0, 0.0, 0.0, 0.0, 0.5, -0.3)


@pytest.mark.parametrize("storage", ["fp32", "fp16s"])
@pytest.mark.parametrize("q,shape,bc,wet", list(cases()), ids=str)
def test_read_matches_the_oracle(q, shape, bc, wet, storage):
    from paper_1812_00118_amd import Sim
    cfg = dict(lattice=q, shape=shape, bc=bc, rho_L=1.0, rho_H=10.0, nu_L=0.05, nu_H=0.01, M=0.1,
               W=4.0, sigma=1e-3, g=(2e-5, -1e-5, 0.0), eps=1e-10, hoc=1, dtheta_C=0.0)
    if wet:
        cfg["wet_cos"] = wet
    prm = pfinputs.model_params(cfg)
    sim = Sim(prm, storage=storage)
    sim.set_state(*pfinputs.random_state(q, shape, seed=7, h_noise=0.01, g_noise=0.01))
    h, g = (t.cpu().numpy().astype(np.float64) for t in sim.get_state())
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in sim.read(("phi", "P", "J")).items()}
    ref = O.read(O.Params.from_dict(prm), h, g)
    shape_of = ref["phi"].shape
    err = np.abs(got["phi"].reshape(shape_of) - ref["phi"])
    assert np.all(err <= q * U32 * np.abs(h).sum(0))
    assert np.array_equal(got["phi"], sim.read(("phi",))["phi"].cpu().numpy())
    D = 3 if q == 19 else 2
    for k, r in (("P", ref["P"]), ("J", ref["J"][:D])):
        assert np.abs(got[k].reshape(r.shape) - r).max() <= 300 * U32 * np.abs(r).max(), k
