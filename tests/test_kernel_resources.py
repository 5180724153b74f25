"""Register spills of the built kernels, read from the resource notes of the library's code object
(no GPU).  A spill's reload in a loop waits for every memory operation in flight, which costs these
kernels more than the register is worth."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1503_07659_amd import dgvol

READELF = next((p for p in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf"))
                if p and os.path.exists(p)), None)


def _code_object(path):
    """The AMD GPU ELF inside the library (e_machine 224)."""
    with open(path, "rb") as fh:
        blob = fh.read()
    for m in re.finditer(b"\x7fELF\x02", blob):
        if struct.unpack_from("<H", blob, m.start() + 18)[0] == 224:
            return blob[m.start():]
    return None


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if READELF is None:
        pytest.skip("llvm-readelf is not installed")
    code = _code_object(dgvol.LIB_PATH)
    assert code is not None, "no gfx950 code object in the library"
    path = tmp_path_factory.mktemp("co") / "dgvol.co"
    path.write_bytes(code)
    notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
    out = {}
    for part in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
        symbol = re.search(r"\n\s+\.symbol:\s+(\S+?)\.kd", part)[1]
        out[symbol] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", part)[1])
    return out


@pytest.mark.parametrize("prefix", ["adj_f64_kernel", "adjcr_gu_kernel", "adjcr_gG_kernel", "fwd_f64_direct_kernel",
                                    "fwd_f64_kernel", "fwd_f32s_kernel", "batched_f64_kernel", "batched_f32s_kernel"])
def test_no_spills(kernels, prefix):
    mine = {k: v for k, v in kernels.items() if re.match(rf"_ZN5dgvol\d+{prefix}I", k)}
    assert mine
    assert not {k: v for k, v in mine.items() if v}


def test_no_spills_in_the_loops_of_the_cotangent_of_d(kernels):
    """The whole-part forms at Np = 56 and 84 keep 1 and 3 registers in scratch across the loop (stored
    before it, read after it); the others must not spill at all."""
    mine = {re.match(r"_ZN5dgvol\d+gd_partial_kernelILi(\d+)ELi(\d)ELi(\d)E", k): v for k, v in kernels.items()}
    spilled = {tuple(int(x) for x in m.groups()): v for m, v in mine.items() if m and v}
    assert set(spilled) <= {(56, 3, 1), (84, 3, 1)}, spilled
