"""Registers of the 256^3 row and y passes, from the notes of the built
library. Both keep 16 loads per thread in flight and hide the latency of HBM with
resident wavefronts: the FP32 row pass's LDS leaves room for eight waves per
SIMD, which 512 / 8 = 64 registers allow, the FP32 register pencils' for four, and
FP64 and the LDS pencils are held by their LDS at four (128 registers) or two. An
address computed per element (a division by the block height of the spectrum's
layout) took 89 instead of 60 registers in the row pass and 1.3 to 1.8% of the step's
time (P_6, P_5)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1801_06364_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _vgprs(path, tmp):
    """{kernel: vgpr count} over the gfx950 code objects embedded in a library."""
    data = open(path, "rb").read()
    starts = [m.start() for m in re.finditer(b"\x7fELF", data)][1:]
    out = {}
    for a, b in zip(starts, starts[1:] + [len(data)]):
        if data[a + 18:a + 20] != b"\xe0\x00":   # EM_AMDGPU
            continue
        f = os.path.join(tmp, "co")
        with open(f, "wb") as fh:
            fh.write(data[a:b])
        notes = subprocess.run([READELF, "--notes", f], capture_output=True, text=True).stdout
        for blk in notes.split(".agpr_count:")[1:]:
            out[re.search(r"\.name:\s+(\S+)", blk).group(1)] = int(re.search(r"\.vgpr_count:\s+(\d+)", blk).group(1))
    return out


def test_registers_of_the_256_row_and_y_passes(tmp_path):
    if not (os.path.exists(READELF) and shutil.which("c++filt")):
        pytest.skip("needs llvm-readelf and c++filt")
    if not os.path.exists(build.LIB):
        build.build()
    regs = _vgprs(build.LIB, str(tmp_path))
    names = subprocess.run(["c++filt"], input="\n".join(regs), capture_output=True, text=True).stdout.split("\n")
    regs = {n.split("(")[0].replace("void ", "").replace("rte::", ""): v for n, v in zip(names, regs.values())}
    rows = {n: v for n, v in regs.items() if n.startswith(("k_rows_inv<float, 256", "k_rows_fwd<float, 256"))}
    assert len(rows) >= 8
    assert {n: v for n, v in rows.items() if v > 64} == {}
    pencils = {n: v for n, v in regs.items() if n.startswith(("k_rows_inv<double, 256", "k_rows_fwd<double, 256",
                                                              "pen::k_pencil_reg<256"))}
    assert len(pencils) >= 10
    assert {n: v for n, v in pencils.items() if v > 128} == {}
