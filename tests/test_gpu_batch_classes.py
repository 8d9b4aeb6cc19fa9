"""The classes of a batch run side by side: calls that follow each other without
a wait, long and short runs, odd counts, a class that leaves and comes back,
and reads right after a step all see every class's lattices at the same step,
bitwise as stepped alone."""
import numpy as np
import pytest
import torch

from paper_2212_01617_amd import frelbm as F

from _pair import case_inputs, ensure_gpu_lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ensure_gpu_lib()


CLASSES = [(0, (70, 33, 1), 0), (0, (64, 40, 1), 1), (1, (66, 12, 9), 0), (1, (40, 20, 16), 1)]


def _make(kind, shape, storage):
    axis = 1 if kind == 0 else 2
    bc = tuple(int(a == axis) for a in range(3))
    wu = np.zeros((3, 2, 3)); wu[axis, 0, 0] = -0.01; wu[axis, 1, 0] = 0.01
    phi0, _, u0 = case_inputs(kind, shape, radius=5, xi=1.5, u_amp=0.004, seed=shape[0])
    p = F.make_params(kind, shape, storage=storage, bc=bc, wall_u=wu, A=0.04, kappa=0.09)
    return F.Lattice(p, phi0, None, u0, stream=torch.cuda.Stream())


@pytest.mark.parametrize("present", [(0, 1, 2, 3), (1, 2), (3,)])
def test_consecutive_runs_equal_solo(present):
    mem = [_make(*CLASSES[k]) for k in present]
    solo = [_make(*CLASSES[k]) for k in present]
    needs = [F.Batch.needs(L) for L in mem]
    B = F.Batch(len(mem) + 1, 2 * sum(w for w, _ in needs), 2 * sum(f for _, f in needs))
    slots = [B.add(L) for L in mem]
    for n in (20, 4, 1, 37, 3, 16):   # 81 steps, nothing waits between the calls
        B.step(n)
    for L, S in zip(mem, solo):
        S.step(81)
        assert L.info()[0] == 81
        assert np.array_equal(L.read(("phi",))["phi"], S.read(("phi",))["phi"])
    B.remove(slots[0])
    B.step(18)
    B.add(mem[0])                     # one step more on its own: 81 is odd, 99 too
    B.step(21)
    for k, (L, S) in enumerate(zip(mem, solo)):
        S.step((0 if k == 0 and len(mem) > 1 else 18 if len(mem) > 1 else 0) + 21)
        assert L.info()[0] == S.info()[0]
        for a, b in zip(L.populations(), S.populations()):
            assert np.array_equal(a, b)
    B.close()


@pytest.mark.parametrize("kind,shape", [(0, (70, 33, 1)), (1, (66, 12, 9))])
@pytest.mark.parametrize("storage", [0, 1])
def test_roller_lattice_joins_and_leaves_a_class_of_flat_walls(kind, shape, storage):
    """The class's fills run for the roller lattice alone, from when it joins
    until it leaves; the member between flat walls never notices."""
    nx, ny, nz = shape
    mask = np.zeros((nz, ny, nx), np.uint8)
    mask[:, 2:5, 10:13] = 2
    rp = F.make_params(kind, shape, storage=storage, rollers=[((11.0, 3.0, 0.0), 0.002, 2, 2.0)], A=0.04, kappa=0.09)
    phi0, _, _ = case_inputs(kind, shape, radius=5, xi=1.5, seed=3)

    def roller():
        return F.Lattice(rp, phi0, mask=mask, stream=torch.cuda.Stream())

    flat, rol = _make(kind, shape, storage), roller()
    sflat, srol = _make(kind, shape, storage), roller()
    needs = [F.Batch.needs(L) for L in (flat, rol)]
    B = F.Batch(2, sum(w for w, _ in needs), sum(f for _, f in needs))

    def same(*pairs):
        for L, S in pairs:
            assert L.info()[0] == S.info()[0]
            for a, b in zip(L.populations(), S.populations()):
                assert np.isfinite(a).all() and np.array_equal(a, b)

    B.add(flat)
    B.step(22)                 # a run of 16 steps and pairs: both graphs
    sflat.step(22)
    same((flat, sflat))
    slot = B.add(rol)
    B.step(22)
    sflat.step(22)
    srol.step(22)
    same((flat, sflat), (rol, srol))
    B.remove(slot)
    B.step(22)
    sflat.step(22)
    same((flat, sflat), (rol, srol))
    B.add(rol)
    B.step(22)
    sflat.step(22)
    srol.step(22)
    same((flat, sflat), (rol, srol))
    B.close()


@pytest.mark.parametrize("room", [False, True])
def test_flat_walls_beside_rollers_with_and_without_room_for_their_fills(room):
    """D2Q9 FP32: beside a roller lattice the member between flat walls is filled as
    well, unless the batch's list holds the roller lattice's fills alone."""
    shape = (70, 33, 1)
    nx, ny, nz = shape
    mask = np.zeros((nz, ny, nx), np.uint8)
    mask[:, 2:5, 10:13] = 2
    rp = F.make_params(0, shape, rollers=[((11.0, 3.0, 0.0), 0.002, 2, 2.0)], A=0.04, kappa=0.09)
    phi0, _, _ = case_inputs(0, shape, radius=5, xi=1.5, seed=3)
    pairs = [[_make(0, shape, 0) for _ in range(2)],
             [F.Lattice(rp, phi0, mask=mask, stream=torch.cuda.Stream()) for _ in range(2)]]
    needs = [F.Batch.needs(p[0]) for p in pairs]
    B = F.Batch(2, sum(w for w, _ in needs), needs[1][1] + (needs[0][1] if room else 0))
    for p in pairs:
        B.add(p[0])
    B.step(21)
    for a, b in pairs:
        b.step(21)
        for x, y in zip(a.populations(), b.populations()):
            assert np.isfinite(x).all() and np.array_equal(x, y)
    B.close()
