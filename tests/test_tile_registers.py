"""The tile kernels, as they are in the built library: not a register in scratch memory.

A kernel of the product on 32x32x16 matrix products, built with every option of every solver in it, once kept 65 in scratch, and conjugate
gradients at n = 65536, d = 11, t = 65 took 10 % longer than the streaming kernels it had replaced.  Of those on 16x16x32, the shapes of
three and more groups of operands kept up to 26 there, addresses of the output computed ahead of the main loop: 2 us more for a short
product (n = 2000, d = 48, t = 33 19.5 us, now 17.0), 2 to 6 % for long ones."""
import os
import re
import shutil
import struct
import subprocess
import tempfile

import pytest

from paper_2405_18328_amd.build import LIB

READELF = shutil.which("llvm-readelf", path=os.pathsep.join([os.environ.get("PATH", ""), "/opt/rocm/llvm/bin"]))
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
FORMS = {"plain": 0, "columns": 1, "gather": 2, "window": 3}


def _gpu_objects(data):
    """The gfx950 code objects of the library's uncompressed offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        q = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, q)
            triple = data[q + 24:q + 24 + length]
            q += 24 + length
            if b"gfx950" in triple and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def _kernels(part):
    """(name, spilled vector registers) of the library's kernels with `part` in their names"""
    if not READELF:
        pytest.skip("llvm-readelf is not installed")
    with open(LIB, "rb") as f:
        data = f.read()
    for obj in _gpu_objects(data):
        if part.encode() not in obj:
            continue
        with tempfile.NamedTemporaryFile(suffix=".o") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name: +(\S+)", entry).group(1)
            if part in name:
                yield name, int(re.search(r"\.vgpr_spill_count: +(\d+)", entry).group(1))


@pytest.fixture(scope="module")
def spills():
    """{(wide, KIND, DS, XP, NT, form): spilled vector registers, with or without the vector-ALU column; DS: shape of the distance operands}"""
    found = {}
    for name, spilled in _kernels("kmv_tile_f16"):
        m = re.search(r"kmv_tile_f16_(wide_)?kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb\dELi(\d)E", name)
        assert m, name
        key = (bool(m.group(1)),) + tuple(int(v) for v in m.groups()[1:])
        found[key] = max(found.get(key, 0), spilled)
    return found


@pytest.mark.parametrize("form", ["plain", "columns", "gather", "window"])
@pytest.mark.parametrize("wide,DS,NT", [(False, 1, 1), (False, 1, 2), (False, 2, 1), (False, 2, 2)])
@pytest.mark.parametrize("KIND", [0, 1])
def test_solver_tile_kernels_hold_their_registers(spills, form, wide, DS, NT, KIND):
    """Shapes that are built once per form."""
    for XP in (2, 3):
        assert spills[(wide, KIND, DS, XP, NT, FORMS[form])] == 0


@pytest.mark.parametrize("KIND,XP", [(0, 2), (0, 3), (1, 2), (1, 3)])
def test_every_tile_kernel_holds_its_registers(spills, KIND, XP):
    found = {k: v for k, v in spills.items() if (k[1], k[3]) == (KIND, XP)}
    for wide, most in ((False, 9), (True, 6 if XP == 2 else 4)):      # shapes that are built with two and with four row tiles per wave
        for NT in (3, 4) if wide else (0, 1, 2, 3, 4):
            assert {k[2] for k in found if (k[0], k[4]) == (wide, NT)} == set(range(1, most + 1)), (wide, NT)
    assert {k: v for k, v in found.items() if v} == {}


def test_gradient_kernels_hold_their_registers():
    """A wave of the four-wave kernels may have all 512 registers.  One of the eight-wave kernels has 256, and 4 XP KH + 8 KT + 16 NT of
    them hold operands and accumulators: from 141 on it keeps the excess in scratch memory, which measured faster
    than four waves all the same wherever eight are chosen by size."""
    found = {}
    for name, spilled in _kernels("grad_tile_f16"):
        KH, XP, KT, NT, W = map(int, re.search(r"ILi\dELi(\d)ELi(\d)ELi(\d+)ELi(\d)ELi(\d)E", name).groups())
        found[W] = found.get(W, 0) + 1
        need = 4 * XP * KH + 8 * KT + 16 * NT
        assert spilled <= (max(0, need - 132) if W == 8 and need > 140 else 0), name
    assert found == {4: 240, 8: 144}
