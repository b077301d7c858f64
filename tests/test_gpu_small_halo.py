"""Tile launches whose halo is four cells (compile-time extents of their own):
the coarse up launches of V(2,2), and with one pass the down and the finest up
launches.  One cycle against the oracle, element by element, on grids that hold
one tile of the shape in each direction and several; and a mixed-precision step,
whose FP32 up launches all have that halo, against the oracle's solution.
"""
import numpy as np
import pytest

import oracle as O
from paper_1208_2643_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1208_2643_amd import api  # noqa: E402
from paper_1208_2643_amd import _lib as L  # noqa: E402

DEV = torch.device("cuda:0")


def one_step(m, n, bc, nu1, nu2, **kw):
    d = dict(eps=0.025, beta=0.9, M=1.0, h=0.5, dt=0.05, scheme=2)
    po, pg = O.Params(**d, bc=(bc & 1, bc >> 1)), api.Params(**d, bc=bc)
    phik = I.noise(m, n, mean=0.1, amp=0.1, seed=23)
    phi0 = torch.from_numpy(phik).to(DEV)
    st = api.Stepper(m, n, pg, energy=0, nu1=nu1, nu2=nu2, **kw)
    phi, _ = st.step(phi0, phi0, torch.zeros_like(phi0), allow_fail=True)
    got = phi.cpu().numpy()
    st.close()
    S = O.source(po, phik, phik, np.zeros_like(phik))
    return got, po, phik, S, O.complete_guess(po, phik.copy(), S, phik)


def relmax(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("m,n,bc", [(64, 64, 0), (64, 32, 3), (128, 256, 2)])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1), (2, 1), (1, 2)])
@pytest.mark.parametrize("shape", [0, 1, 2, 3, 4])
def test_one_cycle_matches_oracle(shape, nu1, nu2, m, n, bc, monkeypatch):
    monkeypatch.setenv("MPFC_TILE_SHAPE", str(shape))
    got, po, phik, S, u0 = one_step(m, n, bc, nu1, nu2, tol=1e-30, max_cycles=1)
    u, _, _ = O.fas_solve(po, u0, S, phik=phik, nu1=nu1, nu2=nu2, tol=1e-30, max_cycles=1)
    assert relmax(got, u[0]) <= 1e-12


@pytest.mark.parametrize("bc", [0, 2])
@pytest.mark.parametrize("nu", [1, 2])
@pytest.mark.parametrize("shape", [0, 1, 2, 3, 4])
def test_mixed_step_matches_oracle(shape, nu, bc, monkeypatch):
    monkeypatch.setenv("MPFC_TILE_SHAPE", str(shape))
    got, po, phik, S, u0 = one_step(128, 128, bc, nu, nu, tol=1e-10, precision=L.MPFC_MIXED)
    # (the oracle takes some 150 cycles for these inputs)
    u, hist, _ = O.fas_solve(po, u0, S, phik=phik, nu1=2, nu2=2, tol=1e-12, max_cycles=400)
    assert hist[-1] <= 1e-12
    assert relmax(got, u[0]) <= 1e-9
