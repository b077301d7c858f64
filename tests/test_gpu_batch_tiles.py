"""The tiled forms of a batch's launches against single-grid contexts.

Each tile shape forced on every phase (the halo of all members agrees or not,
the tile is the shape's or clamped to a small level), and the smallest members a
batch takes.  A member's arithmetic per cell is the single context's: FP64 states
agree to 1e-12.  In mixed precision the FP32 correction of an outer iteration
may round differently where a multiply-add is contracted differently; what is
left of 1e-7 of a correction after the next outer iteration is far below 1e-10.
"""
import math

import numpy as np
import pytest

from paper_1208_2643_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1208_2643_amd import api  # noqa: E402
from paper_1208_2643_amd import _lib as L  # noqa: E402

DEV = torch.device("cuda:0")
BAR = {L.MPFC_FP64: 1e-12, L.MPFC_MIXED: 1e-10}


def rel_l2(a, b):
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


def check(sizes, precision, bcs=(0,), **kw):
    sims, phi0 = [], []
    for k, (m, n) in enumerate(sizes):
        p = api.Params(0.025 + 0.02 * k, 0.9, 1.0, math.pi / 4, 0.05, 2, bc=bcs[k % len(bcs)])
        sims.append((m, n, p))
        phi0.append(torch.from_numpy(I.noise(m, n, mean=0.07, amp=0.05, seed=31 + k)).to(DEV))
    b = api.Batch(sims, precision=precision, **kw)
    phi_b, _, psi_b, infos = api.run_batch(b, phi0, 2)
    b.close()
    for k, (m, n, p) in enumerate(sims):
        st = api.Stepper(m, n, p, energy=0, precision=precision, **kw)
        phi, _, psi, single = api.run(st, phi0[k], 2)
        assert rel_l2(phi_b[k], phi) <= BAR[precision], k
        assert rel_l2(psi_b[k], psi) <= 100 * BAR[precision], k
        assert [i[k].n_cycles for i in infos] == [i.n_cycles for i in single], k
        st.close()


@pytest.mark.parametrize("precision", [L.MPFC_FP64, L.MPFC_MIXED])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1)])
@pytest.mark.parametrize("shape", [0, 1, 2, 3, 4])
def test_every_shape(shape, nu1, nu2, precision, monkeypatch):
    monkeypatch.setenv("MPFC_TILE_SHAPE", str(shape))
    check([(128, 128), (64, 64), (64, 128), (256, 128)], precision, nu1=nu1, nu2=nu2)


@pytest.mark.parametrize("precision", [L.MPFC_FP64, L.MPFC_MIXED])
@pytest.mark.parametrize("shape", [0, 2])
def test_neumann_members(shape, precision, monkeypatch):
    monkeypatch.setenv("MPFC_TILE_SHAPE", str(shape))
    check([(128, 128), (128, 64)], precision, bcs=(0, 3))


@pytest.mark.parametrize("precision", [L.MPFC_FP64, L.MPFC_MIXED])
def test_smallest_members(precision):
    check([(32, 64), (64, 32)], precision)
