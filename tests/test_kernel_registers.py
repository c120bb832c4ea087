"""What the notes of the built library say of its kernels.

Registers of the 256^3 row and y passes: both keep 16 loads per thread in flight and
hide the latency of HBM with resident wavefronts. The FP32 row pass's LDS leaves
room for eight waves per SIMD, which 512 / 8 = 64 registers allow, the FP32 register
pencils' for four, and FP64 and the LDS pencils are held by their LDS at four (128
registers) or two. An address computed per element (a division by the block height
of the spectrum's layout) took 89 instead of 60 registers in the row pass and 1.3 to
1.8% of the step's time (P_6, P_5).

Wavefronts of the streaming pass at 16^3 P_7: 36 moments, two to a wavefront, in at
most eight rounds (each a chain of loads, transforms and barriers), so three or
more; with two, nine rounds, a step took 4 us longer than with two passes."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1801_06364_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _notes(path, tmp):
    """{kernel: (registers, threads)} over the gfx950 code objects embedded in a
    library, by demangled name."""
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
            name, threads, vgpr = (re.search(rf"\.{k}:\s+(\S+)", blk).group(1)
                                   for k in ("name", "max_flat_workgroup_size", "vgpr_count"))
            out[name] = int(vgpr), int(threads)
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True).stdout.split("\n")
    return {n.split("(")[0].replace("void ", "").replace("rte::", ""): v for n, v in zip(names, out.values())}


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (os.path.exists(READELF) and shutil.which("c++filt")):
        pytest.skip("needs llvm-readelf and c++filt")
    if not os.path.exists(build.LIB):
        build.build()
    return _notes(build.LIB, str(tmp_path_factory.mktemp("notes")))


def test_registers_of_the_256_row_and_y_passes(kernels):
    regs = {n: v for n, (v, _) in kernels.items()}
    rows = {n: v for n, v in regs.items() if n.startswith(("k_rows_inv<float, 256", "k_rows_fwd<float, 256"))}
    assert len(rows) >= 8
    assert {n: v for n, v in rows.items() if v > 64} == {}
    pencils = {n: v for n, v in regs.items() if n.startswith(("k_rows_inv<double, 256", "k_rows_fwd<double, 256",
                                                              "pen::k_pencil_reg<256"))}
    assert len(pencils) >= 10
    assert {n: v for n, v in pencils.items() if v > 128} == {}


@pytest.mark.parametrize("T", ["float", "double"])
def test_wavefronts_of_the_16_p7_streaming_pass(kernels, T):
    assert kernels[f"strm::k_stream<{T}, 16, 7>"][1] >= 3 * 64
    assert kernels[f"strm::k_stream<{T}, 16, 6>"][1] == 2 * 64
