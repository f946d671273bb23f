"""Population arrays past 4 GiB, where a byte offset no longer fits 32 bits.

A periodic pattern repeated over the box evolves as one period of it does: the large box is compared
with a box of one period at every node. Both are FP64 and take the same operations per node, so they
agree to rounding; the bounds are those of the step's other parity tests (1e-12).
"""
import numpy as np
import pytest

import lbm_inputs as L
from tests.gpu_cases import Case

pytestmark = pytest.mark.gpu

PX, PY = 64, 16             # the period
NX, NY = 32768, 16400       # 2**29 + 524,288 nodes: the last 16 rows lie past 4 GiB


# the step in one pass and in two passes, with and without walls
@pytest.mark.parametrize("two_pass,walls", [("0", False), ("1", False), ("0", True)])
def test_box_past_4_gib_per_population_matches_its_period(two_pass, walls, monkeypatch):
    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_TWO_PASS", two_pass)
    n = PX * PY
    mask = L.random_mask(PX, PY, 1, 0.1, 21) if walls else None
    small = Case(2, PX, PY, a=0.02, T_reduced=0.8, rho_wall=2.0, mask=mask)
    rho0, u0 = L.random_state(n, 2, 1.0, 1.3, 0.02, 22)
    tile = lambda a: np.broadcast_to(a.reshape(1, PY, 1, PX), (NY // PY, PY, NX // PX, PX)).reshape(-1)
    p = small.params()
    big = Case(2, NX, NY, a=0.02, T_reduced=0.8, rho_wall=2.0, mask=None if mask is None else tile(mask)).params()
    with P.Simulation(p) as s:
        s.init(rho0, u0).step(3)
        r1, U1, _ = s.moments()
        pt1 = P.lbm_pressure_tensor(s.ctx, n, p.lattice) if not walls and two_pass == "0" else None
    with P.Simulation(big) as s:
        big.mask, big._keep = None, []
        s.init(tile(rho0), np.stack([tile(v) for v in u0])).step(3)
        r, U, _ = s.moments()
        pt = P.lbm_pressure_tensor(s.ctx, NX * NY, p.lattice) if not walls and two_pass == "0" else None

    def worst(field, one):
        one = one.reshape(PY, 1, PX)
        return max(np.abs(b - one).max() for b in field.reshape(NY // PY, PY, NX // PX, PX))

    assert worst(r, r1) <= 1e-12 * np.abs(r1).max()
    for a in range(2):
        assert worst(U[a], U1[a]) <= 1e-12
    if pt is not None:
        for a in range(3):
            assert worst(pt[a], pt1[a]) <= 1e-12


def test_batch_case_past_4_gib_per_population_matches_its_period():
    import paper_2112_01975_amd as P
    n = PX * PY
    rho0, u0 = L.random_state(n, 2, 1.0, 1.3, 0.02, 23)
    tile = lambda a: np.broadcast_to(a.reshape(1, PY, 1, PX), (NY // PY, PY, NX // PX, PX)).reshape(-1)
    with P.Simulation(Case(2, PX, PY, a=0.02, T_reduced=0.8).params()) as s:
        s.init(rho0, u0).step(3)
        r1 = s.moments()[0].reshape(PY, 1, PX)
    b = P.lbm_batch_create([Case(2, NX, NY, a=0.02, T_reduced=0.8).params()])
    try:
        P.lbm_batch_init_fields(b, 0, tile(rho0), np.stack([tile(v) for v in u0]))
        P.lbm_batch_step(b, 3)
        r = P.lbm_batch_moments(b, 0, NX * NY, 2)[0]
    finally:
        P.lbm_batch_destroy(b)
    worst = max(np.abs(x - r1).max() for x in r.reshape(NY // PY, PY, NX // PX, PX))
    assert worst <= 1e-12 * np.abs(r1).max()
