"""The persistent kernel of the levels up to 32 x 32 on every shape it can meet:
tops of two, four and eight rows, one and several waves, the 2 x 2 coarsest grid
and both 8-cell ones, each with every boundary condition (the 8-cell solve takes
the sign-pattern basis with a periodic 4-cell axis, elimination with a Neumann
one).

One V-cycle from a rough guess must give the oracle's iterate.  Its rounding is
a few hundred operations deep at condition numbers up to c/h^4 ~ 1e2 of the local
systems at dt = 0.5: 1e-15 * 1e2 * 1e1 stays below the 1e-11 asked for.  A mixed
step must give the FP64 step to the solver's tolerance (1e-10 residual over
fields of norm ~ 1: 1e-9).
"""
import math

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
SHAPES = [(2, 2), (2, 4), (4, 2), (4, 4), (8, 4), (8, 16), (16, 16), (32, 16), (32, 32), (32, 64)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def relmax(a, b):
    return float(np.max(np.abs(a - b)) / max(1e-300, np.max(np.abs(b))))


@pytest.mark.parametrize("bc", [0, 1, 2, 3])
@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("scheme", [1, 2])
def test_one_cycle_iterate_matches_oracle(scheme, m, n, bc):
    d = dict(eps=0.025, beta=0.9, M=1.0, h=math.pi / 4, dt=0.5, scheme=scheme)
    po = O.Params(**d, bc=(bc & 1, bc >> 1))
    phik = I.noise(m, n, mean=0.1, amp=0.1, seed=51)
    prev = I.noise(m, n, mean=0.1, amp=0.1, seed=52)
    st = api.Stepper(m, n, api.Params(**d, bc=bc), tol=1e-30, max_cycles=1, energy=0)
    psi = torch.zeros(n, m, dtype=torch.float64, device=DEV)
    mu, ka = torch.empty_like(psi), torch.empty_like(psi)
    phi_g, info = st.step(dev(phik), dev(prev), psi, mu=mu, kappa=ka, allow_fail=True)
    S = O.source(po, phik, prev, np.zeros_like(phik))
    u0 = O.complete_guess(po, 2 * phik - prev, S, phik)
    u, _, _ = O.fas_solve(po, u0, S, phik=phik, tol=1e-30, max_cycles=1)
    for a, b in zip((host(phi_g), host(mu), host(ka)), u):
        assert relmax(a, b) <= 1e-11
    st.close()


@pytest.mark.parametrize("bc", [0, 1, 2, 3])
@pytest.mark.parametrize("m,n", [(8, 8), (32, 16), (64, 32)])
def test_mixed_step_equals_fp64_step(m, n, bc):
    p = api.Params(0.025, 0.9, 1.0, math.pi / 4, 0.05, 2, bc)
    phi0 = dev(I.noise(m, n, seed=53))
    out = []
    for precision in (L.MPFC_FP64, L.MPFC_MIXED):
        st = api.Stepper(m, n, p, tol=1e-10, precision=precision)
        phi, _, psi, infos = api.run(st, phi0, 3)
        out.append((host(phi), infos[-1].energy_mod))
        st.close()
    assert relmax(out[1][0], out[0][0]) <= 1e-9
    assert abs(out[1][1] - out[0][1]) <= 1e-9 * abs(out[0][1])
