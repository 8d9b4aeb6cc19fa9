"""What the library's host code asks of the HIP runtime, on the CPU: the host
side of libfrelbm linked with a runtime that logs its calls and can make them
fail (tests/hip_stub.cpp).  No kernel runs, so only the order of launches,
waits and events, the devices they are made on and what follows an error are
looked at."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2212_01617_amd import build as hipbuild
from paper_2212_01617_amd import frelbm as F

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("hipcc not found")
    tmp = tmp_path_factory.mktemp("host")
    flags = ["--offload-host-only", "-O1", "-std=c++17", "-fPIC"]
    objs, bins = [], []
    for src in hipbuild.SOURCES:
        o = str(tmp / src.replace(".hip", ".o"))
        subprocess.check_call([hipbuild.hipcc(), *flags, "-c", os.path.join(hipbuild.CSRC, src), "-o", o])
        names = subprocess.check_output(["nm", "-u", o], text=True).split()
        bins += [n for n in names if n.startswith("__hip_fatbin")]
        objs.append(o)
    so = str(tmp / "libfrelbm_host.so")
    subprocess.check_call(["g++", "-shared", "-fPIC", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(HERE, "hip_stub.cpp"), *objs, "-Wl,-Bsymbolic",
                           *[f"-Wl,--defsym={b}=0" for b in bins], "-lpthread", "-o", so])
    L = C.CDLL(so)
    for name, res, args in F._SIGS:
        fn = getattr(L, name)
        fn.restype, fn.argtypes = res, args
    L.stub_log.restype = C.c_char_p
    L.stub_stream.restype = C.c_void_p
    L.stub_stream.argtypes = [C.c_int, C.c_int, C.c_uint32]
    return L


@pytest.fixture
def rt(host):
    host.stub_reset()
    r = Runtime(host)
    yield r
    r.close()


class Runtime:
    """The library on the logging runtime, with the handles a test makes."""

    def __init__(self, lib):
        self.lib, self.lats, self.bats, self.bufs = lib, [], [], []

    def log(self):
        return self.lib.stub_log().decode().split("\n")[:-1]

    def clear(self):
        self.lib.stub_clear()

    def fail(self, name, nth=1):
        self.lib.stub_fail(name.encode(), nth)

    def buffer(self, n):
        a = np.zeros(n + 256, np.uint8)
        self.bufs.append(a)
        return a.ctypes.data + (-a.ctypes.data) % 256

    def stream(self, dev=0, prio=0, mask=0xFFFFFFFF):
        return C.c_void_p(self.lib.stub_stream(dev, prio, mask))

    def params(self, shape, kind=1, storage=0, rollers=False, **kw):
        axis = 1 if kind == 0 else 2
        r = [((2.0, 2.0, 0.0), 0.001, 2, 1.0)] if rollers else []
        return F.make_params(kind, shape, storage=storage, bc=tuple(int(a == axis) for a in range(3)), rollers=r,
                             A=0.04, kappa=0.09, **kw)

    def lattice(self, shape, kind=1, storage=0, stream=None, rollers=False):
        p = self.params(shape, kind, storage, rollers)
        n = C.c_size_t()
        assert self.lib.fre_footprint(C.byref(p), C.byref(n)) == 0
        N = shape[0] * shape[1] * shape[2]
        phi = np.zeros(N)
        mask = np.zeros(N, np.uint8)
        if rollers:
            mask[N // 2] = 2
        h = C.c_void_p()
        assert self.lib.fre_lattice_init(C.byref(p), self.buffer(n.value), n.value, stream or self.stream(),
                                         phi.ctypes.data, None, None, mask.ctypes.data if rollers else None,
                                         C.byref(h)) == 0
        self.lats.append(h)
        return h

    def read(self, h, n_doubles, field=F.FRE_F_PHI):
        out = np.zeros(n_doubles)
        return self.lib.fre_read_moments(h, field, out.ctypes.data, n_doubles)

    def batch(self, members, stream=None):
        n, B = C.c_size_t(), C.c_void_p()
        assert self.lib.fre_batch_footprint(8, 4096, 4096, C.byref(n)) == 0
        st = stream or self.stream()
        assert self.lib.fre_batch_create(self.buffer(n.value), n.value, st, 8, 4096, 4096, C.byref(B)) == 0
        self.bats.append(B)
        for h in members:
            self.add(B, h)
        return B, f"s{self.stream_id(st)}"

    def add(self, B, h):
        slot = C.c_int32()
        assert self.lib.fre_batch_add(B, h, C.byref(slot)) == 0
        return slot.value

    def stream_id(self, st):
        return C.cast(st, C.POINTER(C.c_int * 3)).contents[2]

    def steps(self, h):
        t, s = C.c_int64(), C.c_int32()
        assert self.lib.fre_info(h, C.byref(t), C.byref(s)) == 0
        return t.value, s.value

    def close(self):
        for B in self.bats:
            self.lib.fre_batch_destroy(B)
        for h in self.lats:
            self.lib.fre_lattice_destroy(h)


def test_failed_short_read_waits_before_its_buffer_is_given_back(rt):
    """Three pieces (a read that starts no thread): the second launch fails,
    and the first piece is still being written."""
    st = rt.stream()
    h = rt.lattice((1024, 600, 1), kind=0, stream=st)
    rt.clear()
    rt.fail("hipLaunchKernel", 2)
    assert rt.read(h, 1024 * 600) == F.FRE_EDEVICE
    log = rt.log()
    assert log[0].startswith("launch k_pack")
    assert f"sync s{rt.stream_id(st)}" in log[1:]
    assert rt.read(h, 1024 * 600) == 0


def test_reads_of_a_lattice_on_another_device(rt):
    st = rt.stream(dev=1)
    h = rt.lattice((1024, 1100, 1), kind=0, stream=st)
    assert rt.read(h, 1024 * 1100) == 0, rt.lib.fre_last_error()   # five pieces: events
    assert rt.lib.stub_current_device() == 0


def test_steps_of_a_batch_on_another_device(rt):
    st = rt.stream(dev=1)
    mem = [rt.lattice((70, 9, 1), kind=0, stream=st), rt.lattice((70, 9, 8), stream=st)]
    B, _ = rt.batch(mem, stream=st)
    rt.clear()
    assert rt.lib.fre_batch_step(B, 20) == 0, rt.lib.fre_last_error()
    assert [line.split()[2] for line in rt.log() if line.startswith("newstream")] == ["dev1"]
    assert rt.lib.stub_current_device() == 0


def graphs(log):
    """(graph, stream) of every graph launch."""
    return [tuple(line.split()[1::2]) for line in log if line.startswith("graph ")]


TURN = 64     # runs of 16 steps that a class is given before the next one


def test_classes_of_a_batch_are_queued_in_turn(rt):
    """Each class gets a bounded number of steps before the others get theirs: a
    queue filled with one class's whole call would hold the others back."""
    B, st = rt.batch([rt.lattice((70, 9, 1), kind=0), rt.lattice((70, 9, 8)), rt.lattice((64, 8, 8), storage=1)])
    rt.clear()
    assert rt.lib.fre_batch_step(B, 2 * 16 * TURN + 52) == 0
    turns = []
    for _, s in graphs(rt.log()):
        if not turns or turns[-1][0] != s:
            turns.append([s, 0])
        turns[-1][1] += 1
    assert [n for _, n in turns] == 6 * [TURN] + 3 * [5]       # 52 steps: three runs and two pairs
    for k in (0, 3, 6):
        assert [s for s, _ in turns[k:k + 3]] == [s for s, _ in turns[:3]]
    assert len({s for s, _ in turns}) == 3


def test_a_failed_launch_between_turns_leaves_the_members_usable(rt):
    mem = [rt.lattice((70, 9, 1), kind=0), rt.lattice((70, 9, 8))]
    B, st = rt.batch(mem)
    for nth, taken in ((1, 0), (2 * TURN + 1, 16 * TURN), (2, None)):
        before = [rt.steps(h)[0] for h in mem]
        rt.clear()
        rt.fail("hipGraphLaunch", nth)
        assert rt.lib.fre_batch_step(B, 16 * TURN + 48) == F.FRE_EDEVICE
        after = [rt.steps(h) for h in mem]
        if taken is None:     # one class is a run ahead of the other
            assert all(s == 1 for _, s in after)
            assert rt.lib.fre_batch_step(B, 1) == F.FRE_ESTATE
            continue
        # every class at the same step, and that step is reported
        assert after == [(b + taken, 0) for b in before]
        assert [s for _, s in graphs(rt.log())].count(st) == taken // 16
        # what ran is joined to the batch's stream, what did not run is not
        assert (f"wait {st}" in rt.log()) == (taken > 0)
        assert rt.lib.fre_batch_step(B, 16) == 0


def test_a_failed_launch_of_a_single_class_keeps_the_steps_taken(rt):
    mem = [rt.lattice((70, 9, 8)), rt.lattice((40, 9, 8))]
    B, _ = rt.batch(mem)
    for nth, taken in ((3, 32), (5, 50)):
        before = [rt.steps(h)[0] for h in mem]
        rt.fail("hipGraphLaunch", nth)
        assert rt.lib.fre_batch_step(B, 52) == F.FRE_EDEVICE
        assert [rt.steps(h) for h in mem] == [(b + taken, 0) for b in before]


def test_steps_on_a_capturing_stream_draw_in_no_other(rt):
    """The caller captures the batch's stream: nothing is recorded on, or waited
    for by, the batch's own streams, which the capture would swallow."""
    cap = rt.stream()
    B, st = rt.batch([rt.lattice((70, 9, 1), kind=0), rt.lattice((70, 9, 8))], stream=cap)
    assert rt.lib.fre_batch_step(B, 18) == 0        # both classes' graphs
    assert rt.lib.hipStreamBeginCapture(cap, 0) == 0
    rt.clear()
    assert rt.lib.fre_batch_step(B, 16) == F.FRE_EDEVICE
    g = C.c_void_p()
    assert rt.lib.hipStreamEndCapture(cap, C.byref(g)) == 0
    assert not any(line.startswith(("wait", "record", "graph")) for line in rt.log())
    assert [rt.steps(h) for h in rt.lats] == [(18, 0)] * 2


@pytest.mark.parametrize("how", [dict(prio=-1), dict(mask=0xFFFF)])
def test_a_batch_keeps_to_a_stream_of_its_own_kind(rt, how):
    """A stream with a priority, or limited to some CUs: the batch's own streams
    would not have them."""
    B, st = rt.batch([rt.lattice((70, 9, 1), kind=0), rt.lattice((70, 9, 8))], stream=rt.stream(**how))
    for n in (20, 36):
        rt.clear()
        assert rt.lib.fre_batch_step(B, n) == 0
        assert [s for _, s in graphs(rt.log())] == [st] * 2 * (n // 16 + n % 16 // 2)
        assert not any(line.startswith("wait") for line in rt.log())


def test_members_that_join_or_leave_recapture_only_their_class(rt):
    flat2, flat3 = rt.lattice((70, 9, 1), kind=0), rt.lattice((70, 9, 8))
    B, _ = rt.batch([flat2, flat3])

    def captures(n=18):
        rt.clear()
        assert rt.lib.fre_batch_step(B, n) == 0
        return [line.split()[2:] for line in rt.log() if line.startswith("instantiate")]

    assert len(captures()) == 4                     # a run and a pair for each class
    assert captures() == []
    slot = rt.add(B, rt.lattice((40, 9, 8)))        # another one of the same kind
    assert captures() == []
    roller = rt.add(B, rt.lattice((24, 12, 8), rollers=True))   # its class needs fills now
    new = captures()
    assert len(new) == 2 and all("k_batch_fill" in g for g in new)
    assert rt.lib.fre_batch_remove(B, slot) == 0 and captures() == []
    assert rt.lib.fre_batch_remove(B, roller) == 0
    new = captures()
    assert len(new) == 2 and not any("k_batch_fill" in g for g in new)
    half = rt.add(B, rt.lattice((70, 9, 8), storage=1))         # a class more
    assert len(captures()) == 2
    assert rt.lib.fre_batch_remove(B, half) == 0 and captures() == []
    for k in range(2):                              # empty, and filled again
        assert rt.lib.fre_batch_remove(B, k) == 0
    rt.add(B, flat2)
    assert captures() == []


def launches(log):
    return [line.split()[1] for line in log if line.startswith("launch ")]


@pytest.mark.parametrize("kind,shape", [(0, (70, 9, 1)), (1, (70, 9, 8))])
@pytest.mark.parametrize("storage", [0, 1])
def test_the_tuner_times_the_kernels_that_steps_launch(rt, kind, shape, storage):
    h = rt.lattice(shape, kind=kind, storage=storage)
    rt.clear()
    assert rt.lib.fre_step(h, 2) == 0
    step = launches(rt.log())
    assert step.count("k_fill") == 0 and ("k_collide_2d" in step) == (kind == 0)
    cfg, ms = (C.c_int32 * 6)(), (C.c_double * 3)()
    rt.clear()
    assert rt.lib.fre_autotune(h, 2, cfg, ms) == 0
    tuned = launches(rt.log())
    assert tuned[-1] == "k_cells"                   # M of the restored state
    assert tuned[:-1] == step * (len(tuned) // len(step))
    if kind == 0:     # no kernel of a step takes the potential's shape, and the tile has four rows
        assert list(cfg[:4])[2:] == [4, 1] and ms[1] == -1.0 and cfg[4] == 4
    assert ms[0] > 0 and ms[2] > 0
    per, n = (C.c_double * 8)(), C.c_int32()
    rt.clear()
    assert rt.lib.fre_profile_step(h, 2, per, 8, C.byref(n)) == 0
    assert launches(rt.log()).count("k_fill") == 4  # profiles keep every stage


def test_the_batch_tuner_times_steps_as_the_batch_takes_them(rt):
    B, st = rt.batch([rt.lattice((70, 9, 1), kind=0), rt.lattice((70, 9, 8))])
    bpc, ms = C.c_int32(), C.c_double()
    rt.clear()
    assert rt.lib.fre_batch_autotune(B, 32, C.byref(bpc), C.byref(ms)) == 0
    log = rt.log()
    assert not any(k.startswith("k_batch") for k in launches(log))
    # every candidate: a run that captures, then the timed one, side by side
    marks = [k for k, line in enumerate(log) if line == f"record {st}"]
    assert len(graphs(log)) == 4 * 2 * 2 * 2 and len({s for _, s in graphs(log)}) == 2
    assert marks and [rt.steps(h) for h in rt.lats] == [(0, 0), (0, 0)]
    assert rt.lib.fre_batch_step(B, 20) == 0


@pytest.mark.parametrize("kind,shape,sums", [(0, (100, 90, 1), False), (0, (1025, 1024, 1), True),
                                             (1, (32, 32, 31), False)])
def test_ternary_steps_sum_moments_only_on_large_lattices(rt, kind, shape, sums):
    p = rt.params(shape, kind, ternary=(0.2, 0.07, 0.9))
    n, h, N = C.c_size_t(), C.c_void_p(), shape[0] * shape[1] * shape[2]
    assert rt.lib.fre_footprint(C.byref(p), C.byref(n)) == 0
    z = np.zeros(N)
    assert rt.lib.fre_lattice_init3(C.byref(p), rt.buffer(n.value), n.value, rt.stream(), z.ctypes.data, z.ctypes.data,
                                    None, None, None, C.byref(h)) == 0
    rt.lats.append(h)
    rt.clear()
    assert rt.lib.fre_step(h, 1) == 0
    assert launches(rt.log()) == ["k3_potential", "k3_collide", "k3_combine" if sums else "k3_moments"]


@pytest.mark.parametrize("kind,small,large,sums", [(0, (1024, 1022, 1), (1024, 1023, 1), 12.0),
                                                   (1, (128, 128, 62), (128, 128, 63), 36.0)])
def test_only_ternary_lattices_that_sum_moments_hold_the_sums(rt, kind, small, large, sums):
    """With the walls' ghost layers the small one has 2^20 cells."""
    def bytes_per_cell(shape):
        n = C.c_size_t()
        assert rt.lib.fre_footprint(C.byref(rt.params(shape, kind, ternary=(0.2, 0.07, 0.9))), C.byref(n)) == 0
        return n.value / (shape[0] * (shape[1] + 2) if kind == 0 else shape[0] * shape[1] * (shape[2] + 2))

    assert sums <= bytes_per_cell(large) - bytes_per_cell(small) < sums + 2.5
