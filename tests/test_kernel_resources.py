"""Registers of the built kernels (the compiler's own records in libfrelbm.so):
what decides how many blocks a CU holds."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2212_01617_amd import frelbm as F

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("ROCm LLVM tools not found")
    if not os.path.exists(F.LIB_PATH):
        from paper_2212_01617_amd import build
        build.build()
    tmp = tmp_path_factory.mktemp("objects")
    shutil.copy(F.LIB_PATH, tmp)
    subprocess.check_call([f"{LLVM}/llvm-objdump", "--offloading", os.path.basename(F.LIB_PATH)], cwd=tmp,
                          stdout=subprocess.DEVNULL)
    out = {}
    for name in os.listdir(tmp):
        if "gfx950" in name:
            notes = subprocess.check_output([f"{LLVM}/llvm-readelf", "--notes", str(tmp / name)], text=True)
            for m in re.finditer(r"\.name:\s+(\S+)\n(.*?)\.wavefront_size", notes, re.S):
                out[m.group(1)] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", m.group(2))}
    return out


def test_single_lattice_potential_holds_eight_blocks_without_spills(kernels):
    """Above 80 scalar registers a CU holds 7 blocks of the potential; capped
    there by spilling, it is slower on every lattice."""
    pot = {n: r for n, r in kernels.items() if "k_potential_zm" in n}
    assert len(pot) == 12          # velocity set, storage, kind of walls
    for n, r in pot.items():
        assert r["sgpr_count"] <= 80 and r["sgpr_spill_count"] == 0 and r["vgpr_spill_count"] == 0, (n, r)


def test_plain_collides_hold_four_waves(kernels):
    """D3Q19 collides of lattices without masks (walls 1 and 2): at most 128
    vector registers, and no population spilled."""
    col = {n: r for n, r in kernels.items() if re.search(r"k_cellsILi19ELi[01]ELi2ELi[01]ELi[12]E", n)}
    assert len(col) == 12          # storage, parity, walls, rounding
    for n, r in col.items():
        assert r["vgpr_count"] <= 128 and r["vgpr_spill_count"] == 0, (n, r)
