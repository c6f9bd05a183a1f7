"""What the slab and tile kernels of the built library ask of a compute unit, from the metadata that the compiler leaves beside them: arguments and
registers decide how soon a workgroup starts and how many share a unit, and nothing else here would notice a change."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_27390_amd", "libevospec.so")
LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: {template arguments: its metadata}} of the built library"""
    if not os.path.exists(LIB) or not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no built library, or no tools to read it")
    tmp = tmp_path_factory.mktemp("lib")
    shutil.copy(LIB, tmp / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    out = {}
    for f in tmp.glob("lib.so.*gfx950*"):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", f.name], cwd=tmp, check=True, capture_output=True, text=True).stdout
        for k in notes.split("- .agpr_count")[1:]:
            m = re.search(r"\.name:\s+\S*?\d(lmhead_\w+_kernel)I((?:L[ib]n?\d+E)+)E", k)
            if m:
                args = tuple(int(x.replace("n", "-")) for x in re.findall(r"L[ib](n?\d+)E", m.group(2)))
                out.setdefault(m.group(1), {})[args] = {
                    x: int(re.search(r"\.%s:\s+(\d+)" % x, k).group(1)) for x in ("vgpr_count", "kernarg_segment_size")}
    return out


@pytest.fixture(scope="module")
def slab_kernels(kernels):
    """by (tiles, wavefronts to a tile, ring, blocks, whole chunks, packed, past the caches, segments, core)"""
    return kernels["lmhead_partials_kernel"]


def test_tiles_carry_what_they_bring(kernels):
    """Blocks of an extension's draft rows: 0 (nothing beside the tiles), -1 (a bound of the rows), or more (a table of chunks)."""
    size = {}
    for name, blocks in (("lmhead_tile_kernel", 3), ("lmhead_packed_tile_kernel", 0)):
        for args, v in kernels[name].items():
            size.setdefault(min(args[blocks], 1), set()).add(v["kernarg_segment_size"])
    assert {x: len(s) for x, s in size.items()} == {0: 1, -1: 1, 1: 1}
    nothing, bound, table = size[0].pop(), size[-1].pop(), size[1].pop()
    assert bound >= nothing + 256 and table >= nothing + 1280


def test_only_joint_launches_carry_a_core(slab_kernels):
    alone = {v["kernarg_segment_size"] for k, v in slab_kernels.items() if not k[8]}
    core = {v["kernarg_segment_size"] for k, v in slab_kernels.items() if k[8]}
    assert len(alone) == 1 and len(core) == 1 and core.pop() >= alone.pop() + 64


def test_two_workgroups_of_seven_or_eight_wavefronts(slab_kernels):
    """Two blocks of draft rows on a matrix of several rounds: 14 to 16 wavefronts, four to a SIMD of 512 registers."""
    two = {k: v["vgpr_count"] for k, v in slab_kernels.items() if k[:2] in ((7, 1), (8, 1)) and k[3] == 2 and (k[5] or k[7] == 2)}
    assert two and all(v <= 128 for v in two.values()), two
