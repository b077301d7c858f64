"""The small levels of a three-dimensional cycle in one workgroup: every kind of
shape of its top level (cubic, thin in each axis, rows longer than a wave's lanes,
a single level, coarsest levels that are not 2 x 2 x 2), as the finest level
(complete right-hand side) and below one (completed in the kernel).  One cycle
against the oracle, element by element, at the tolerance of the other one-cycle
tests.  And the half-sweeps of larger levels, whose threads take two neighbouring
cells of a colour where a row has them.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1208_2643_amd import api  # noqa: E402

DEV = torch.device("cuda:0")
K = 6


def relmax(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 2)])
@pytest.mark.parametrize("m,n,l", [
    (2, 2, 2), (4, 2, 2), (2, 8, 2), (2, 2, 1024), (4, 4, 4),      # one level, or two
    (16, 16, 16), (64, 8, 8), (8, 64, 8), (8, 8, 64), (128, 8, 4), (512, 4, 2), (4, 16, 64),
    (32, 32, 32), (16, 32, 16), (256, 8, 8), (8, 512, 8), (32, 16, 8),
    (2, 64, 64), (4, 64, 64), (8, 64, 32)])                     # rows of one, two, four pairs
def test_one_cycle(m, n, l, nu1, nu2):
    d = dict(eps=0.025, beta=0.9, M=1.0, h=0.5, dt=0.05, scheme=2)
    rng = np.random.default_rng(29)
    phi0 = 0.1 + 0.1 * (rng.random((l, n, m)) - 0.5)
    st = api.Stepper3(m, n, l, api.Params(**d), tol=1e-30, max_cycles=1, coarse_sweeps=K,
                      nu1=nu1, nu2=nu2, energy=0)
    x = torch.from_numpy(phi0).to(DEV)
    phi, info = st.step(x, x, torch.zeros_like(x), allow_fail=True)
    got = phi.cpu().numpy()
    st.close()
    po = O.Params(**d)
    S = O.source3(po, phi0, phi0, np.zeros_like(phi0))
    u0 = O.complete_guess3(po, phi0.copy(), S, phi0)
    u, _, _ = O.fas_solve3(po, u0, S, phik=phi0, nu1=nu1, nu2=nu2, tol=1e-30, max_cycles=1,
                           coarse_sweeps=K)
    assert relmax(got, u[0]) <= 1e-12


@pytest.mark.parametrize("scheme", [1, 2])
@pytest.mark.parametrize("m,n,l", [
    (2, 2, 2), (32, 32, 32), (64, 64, 32), (2, 256, 256),       # a cell per thread
    (128, 64, 32), (2, 512, 256), (64, 64, 64)])                # a block per thread
def test_residual_norms(m, n, l, scheme):
    """The norms of the guess and of two cycles, on both sides of the size from which
    a thread takes a block of cells."""
    d = dict(eps=0.025, beta=0.9, M=1.0, h=0.5, dt=0.05, scheme=scheme)
    rng = np.random.default_rng(31)
    phi0 = 0.1 + 0.1 * (rng.random((l, n, m)) - 0.5)
    st = api.Stepper3(m, n, l, api.Params(**d), tol=1e-30, max_cycles=2, coarse_sweeps=K, energy=0)
    x = torch.from_numpy(phi0).to(DEV)
    _, info = st.step(x, x, torch.zeros_like(x), allow_fail=True)
    st.close()
    po = O.Params(**d)
    S = O.source3(po, phi0, phi0, np.zeros_like(phi0))
    u0 = O.complete_guess3(po, phi0.copy(), S, phi0)
    _, hist, _ = O.fas_solve3(po, u0, S, phik=phi0, tol=1e-30, max_cycles=2, coarse_sweeps=K)
    np.testing.assert_allclose(info.history, hist, rtol=1e-9)
