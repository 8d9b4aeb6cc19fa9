"""Field reads in pieces: a read whose doubles span several pieces, end inside
one or fall exactly on a boundary gives the same fields as reads of one field
at a time and as the oracle; two threads reading two lattices do not meet.

Tolerances are the parity bars of the FP32 path (1e-5 on rho, phi, u; 1e-6 on
the potentials and the pressure)."""
import threading

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2212_01617_amd import frelbm as F
from paper_2212_01617_amd import synth

from _pair import ensure_gpu_lib

pytestmark = pytest.mark.gpu

PIECE = 1 << 18  # doubles per piece


@pytest.fixture(scope="module", autouse=True)
def _lib():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ensure_gpu_lib()


def _lattice(shape, storage=0, wall=1):
    nx, ny, _ = shape
    wu = np.zeros((3, 2, 3)); wu[1, 0, 0] = -0.01; wu[1, 1, 0] = 0.01
    sh = (1, ny, nx)
    phi0 = synth.droplet_phi(sh, 0.2 * min(nx, ny) + 1.0, 2.0, noise=1e-4, seed=nx, dims=2)
    u0 = synth.shear_velocity(sh, 0.02 / ny, axis_normal=1)
    kw = dict(bc=(0, wall, 0), wall_u=wu, A=0.04, kappa=0.09, tau_f=1.0, tau_g=1.0, M=0.1)
    L = F.Lattice(F.make_params(0, shape, storage=storage, **kw), phi0, None, u0, stream=torch.cuda.Stream())
    return L, O.Lattice(O.make_params(0, shape, **kw), phi0, None, u0)


# 8 doubles a cell in a full read: one short piece, exactly one piece, one
# piece and a few doubles, many pieces with a ragged end
@pytest.mark.parametrize("shape", [(3, 2, 1), (256, 128, 1), (257, 128, 1), (1001, 413, 1)])
def test_pieces_agree_with_single_fields_and_oracle(shape):
    L, R = _lattice(shape)
    assert shape != (256, 128, 1) or 8 * shape[0] * shape[1] == PIECE
    L.step(5)
    R.step(5)
    both = L.read()
    for k in both:
        assert np.array_equal(both[k], L.read((k,))[k]), k
    o = R.observe()
    for k, bar in (("rho", 1e-5), ("phi", 1e-5), ("mu_rho", 1e-6), ("mu_phi", 1e-6), ("P", 1e-6)):
        if k in o:
            assert np.abs(both[k] - o[k]).max() <= bar, k
    for a, k in enumerate(("ux", "uy", "uz")):
        assert np.abs(both["u"][a] - o[k]).max() <= 1e-5
    L.close()


def test_two_threads_read_two_lattices():
    lats = [_lattice((700, 300, 1), storage)[0] for storage in (0, 1)]
    want = [L.step(4).read(("phi", "u")) for L in lats]
    got = [None, None]

    def read(k):
        for _ in range(3):
            got[k] = lats[k].read(("phi", "u"))

    th = [threading.Thread(target=read, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for w, g in zip(want, got):
        for k in w:
            assert np.array_equal(w[k], g[k])
    for L in lats:
        L.close()
