"""Registers of the built kernels, from the code objects' own metadata: kernels whose speed
depends on how many wavefronts or workgroups a CU holds, or on not spilling."""
import os
import re
import struct
import subprocess

import pytest

from paper_2309_10292_amd import gs

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{symbol: (vector registers, spilled vector registers)} of every kernel in libgs.so."""
    d = tmp_path_factory.mktemp("code")
    fat = str(d / "fat")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, gs.LIB_PATH, os.devnull], check=True)
    blob, out, pos = open(fat, "rb").read(), {}, 0
    while (pos := blob.find(b"\x7fELF", pos)) >= 0:
        shoff, = struct.unpack_from("<Q", blob, pos + 0x28)
        shnum, = struct.unpack_from("<H", blob, pos + 0x3C)
        obj = d / "object"
        obj.write_bytes(blob[pos:pos + shoff + 64 * shnum])
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        for k in notes.split("- .agpr_count:")[1:]:
            f = {n: v for n, v in re.findall(r"\.(symbol|vgpr_count|vgpr_spill_count):\s+'?([^\s']+)", k)}
            out[f["symbol"]] = (int(f["vgpr_count"]), int(f["vgpr_spill_count"]))
        pos += 64
    assert out
    return out


# symbols, largest number of registers (512 a SIMD lane slot: 128 let 4 wavefronts in, 96 let 5), largest number spilled
@pytest.mark.parametrize("symbol, vgprs, spilled", [
    # the single-step kernel streams: its loads in flight are its wavefronts (FP16 tiles of up to 39 KB of LDS)
    (r"stencil_tileIDF16_Li(128ELi16|64ELi32)ELi8ELi2ELb0ELb0E", 128, 0),
    (r"stencil_tileINS_4bf16E\w+ELi2ELb0ELb0E", 128, 0),
    (r"stencil_tileIfLi\d+ELi\d+ELi4ELi2ELb0ELb0E", 96, 0),
    # the FP64 kernels of 768 and 1024 lanes with noise, which leave no register
    (r"10stencil_tbIdLi16ELi38ELi2ELi768ELi[12]E", 168, 0),
    (r"10stencil_tbIdLi16ELi54ELi1ELi1024ELi[12]E", 128, 2),
    # FP32: three steps in 1024 lanes; one in 768, two workgroups of which share a CU at 80 registers
    (r"10stencil_tbIfLi16ELi50ELi3ELi1024E", 128, 0),
    (r"10stencil_tbIfLi16ELi40ELi1ELi768E", 80, 0),
    # workgroups per CU that the launch estimates count on: two steps in 256 lanes (FP64 two, the others four) and in
    # 512 lanes (two), surrogate layers of 8 channels (three; four of the last weight gradient)
    (r"10stencil_tbIdLi16ELi10ELi2ELi256E", 256, 0),
    (r"10stencil_tbI(f|DF16_|NS_4bf16E|NS_5bf16cE)Li16ELi10ELi2ELi256E", 128, 2),
    (r"10stencil_tbI(f|DF16_|NS_4bf16E|NS_5bf16cE)Li(16ELi24|8ELi47|12ELi32)ELi2ELi512E", 128, 2),
    # two workgroups of the batches' FP64 kernel of three steps in 256 lanes, where more wait than are resident
    (r"16stencil_tb_batchIdLi16ELi8ELi3ELi256ELi0ELi2E", 256, 0),
    (r"12conv8_kernel", 168, 0),
    (r"18wgrad_shift_kernelILb1E", 168, 0),
    (r"18wgrad_shift_kernelILb0E", 128, 0),
])
def test_registers(kernels, symbol, vgprs, spilled):
    found = {k: v for k, v in kernels.items() if re.search(symbol, k)}
    assert found
    for k, (n, s) in found.items():
        assert n <= vgprs and s <= spilled, (k, n, s)
