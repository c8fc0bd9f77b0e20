"""The tile kernels the column solvers launch, as they are in the built library: hardly a register in scratch memory.

The shape of the most registers (KH = 1, two contraction tiles, two sub-tiles per wave) holds 250 of its 256 in its main
loop.  Built with every option of every solver in it, it kept 65 of them in scratch, and conjugate gradients
at n = 65536, d = 11, t = 65 took 10 % longer than the streaming kernels it had replaced."""
import os
import re
import shutil
import struct
import subprocess

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


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{(wide, KIND, KH, XP, NT, form): spilled vector registers, the worst over the rest of the template arguments}"""
    if not READELF:
        pytest.skip("llvm-readelf is not installed")
    with open(LIB, "rb") as f:
        data = f.read()
    found = {}
    path = tmp_path_factory.mktemp("objects") / "gpu.o"
    for obj in _gpu_objects(data):
        if b"kmv_tile_f16" not in obj:
            continue
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name: +(\S+)", entry).group(1)
            m = re.search(r"kmv_tile_f16_(wide_)?kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)E(?:Li\dE)?Lb\dELi(\d)E", name)
            if m:
                key = (bool(m.group(1)),) + tuple(int(v) for v in m.groups()[1:])
                found[key] = max(found.get(key, 0), int(re.search(r"\.vgpr_spill_count: +(\d+)", entry).group(1)))
    assert found
    return found


@pytest.mark.parametrize("form", ["columns", "gather", "window"])
@pytest.mark.parametrize("wide,KH,NT", [(False, 1, 1), (False, 1, 2), (False, 2, 1), (True, 2, 2)])
@pytest.mark.parametrize("KIND", [0, 1])
def test_solver_tile_kernels_hold_their_registers(spills, form, wide, KH, NT, KIND):
    for XP in (2, 3):
        assert spills[(wide, KIND, KH, XP, NT, FORMS[form])] <= 4 * (XP - 1)
