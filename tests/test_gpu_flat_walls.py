"""Lattices between flat walls on the last axis form the values of ghost cells
inside the stencil kernels, and D2Q9 lattices without solid cells form the
potential inside the collide; profiled steps store fills and potential, a
launch per stage.  Both have to give bitwise the same populations, down to one
cell per axis (where a neighbour two steps away is the cell itself, and both
walls fill from one layer), in every storage; ternary lattices are held to the
oracle at the FP32 parity bars (1e-5; 2e-6 on the potentials)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2212_01617_amd import frelbm as F
from paper_2212_01617_amd import synth

from _pair import ensure_gpu_lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ensure_gpu_lib()


def _inputs(kind, shape, walls=True):
    nx, ny, nz = shape
    sh, axis = (nz, ny, nx), (1 if kind == 0 else 2)
    bc = tuple(int(walls and a == axis) for a in range(3))
    wu = np.zeros((3, 2, 3)); wu[axis, 0, 0] = -0.01; wu[axis, 1, 0] = 0.012
    if kind == 1:
        wu[axis, 1, 1] = 0.004
    phi0 = 0.8 * synth.smooth_random_field(sh, 3) + synth.uniform(5, nx * ny * nz, -0.05, 0.05).reshape(sh)
    rho0 = 1.0 + 0.01 * synth.smooth_random_field(sh, 4)
    u0 = 0.01 * np.stack([synth.smooth_random_field(sh, 7 + a) for a in range(3)])
    if kind == 0:
        u0[2] = 0.0
    return bc, wu, phi0, rho0, u0


SHAPES = [(0, (1, 1, 1)), (0, (2, 1, 1)), (0, (3, 2, 1)), (0, (64, 3, 1)), (0, (65, 9, 1)), (0, (130, 14, 1)),
          (1, (1, 1, 1)), (1, (2, 3, 1)), (1, (3, 1, 2)), (1, (64, 2, 1)), (1, (65, 5, 2)), (1, (130, 9, 7))]


@pytest.mark.parametrize("storage,sr", [(0, False), (1, False), (1, True)])
@pytest.mark.parametrize("kind,shape", SHAPES)
def test_fused_steps_equal_staged_steps(kind, shape, storage, sr):
    _equal(kind, shape, storage, sr, True)


@pytest.mark.parametrize("storage,sr", [(0, False), (1, False), (1, True)])
@pytest.mark.parametrize("kind,shape", [s for s in SHAPES if s[0] == 0])
def test_fused_steps_equal_staged_steps_periodic(kind, shape, storage, sr):
    _equal(kind, shape, storage, sr, False)


def _equal(kind, shape, storage, sr, walls):
    bc, wu, phi0, rho0, u0 = _inputs(kind, shape, walls)
    p = F.make_params(kind, shape, storage=storage, bc=bc, wall_u=wu, stochastic_rounding=sr,
                      kappa1=0.16, kappa2=0.12, alpha=1.0, tau_f=0.8, tau_g=1.1, M=0.1)
    a, b = (F.Lattice(p, phi0, rho0, u0, stream=torch.cuda.Stream()) for _ in range(2))
    a.step(7)
    b.profile(7)
    for x, y in zip(a.populations(), b.populations()):
        assert np.isfinite(x).all() and np.array_equal(x, y)
    a.close()
    b.close()


@pytest.mark.parametrize("kind,shape", [(0, (66, 9, 1)), (1, (66, 6, 5)), (1, (3, 2, 1))])
def test_ternary_between_flat_walls(kind, shape):
    bc, wu, phi0, rho0, u0 = _inputs(kind, shape)
    psi0 = 0.2 + 0.1 * synth.smooth_random_field(phi0.shape, 9)
    phi0 = 0.5 * phi0
    kw = dict(bc=bc, wall_u=wu, kappa1=0.16, kappa2=0.12, alpha=1.0, tau_f=0.8, tau_g=1.1, M=0.1)
    third = (0.2, 0.07, 0.9)
    g = F.Lattice(F.make_params(kind, shape, ternary=third, **kw), phi0, rho0, u0, psi0=psi0,
                  stream=torch.cuda.Stream()).step(12)
    o = O.Lattice3(O.make_params(kind, shape, **kw), *third, phi0, psi0, rho0, u0)
    o.step(12)
    have, want = g.read(), o.observe()
    for k, bar in (("rho", 1e-5), ("phi", 1e-5), ("psi", 1e-5), ("mu_rho", 2e-6), ("mu_phi", 2e-6), ("mu_psi", 2e-6)):
        have_k = g.read((k,))[k] if k not in have else have[k]
        assert np.abs(have_k - want[k]).max() <= bar, k
    for a, k in enumerate(("ux", "uy", "uz")):
        assert np.abs(have["u"][a] - want[k]).max() <= 1e-5
    g.close()
