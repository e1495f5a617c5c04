"""Registers of the packing kernel for layers that fill the chip: it is bound by memory, and its loads in flight are those of
the wavefronts that a SIMD holds at once. 72 of 512 registers per lane leave room for seven; eighty-odd would for five."""
import os
import re
import subprocess

from paper_2608_15602_amd import build as b


def test_packing_keeps_seven_wavefronts_per_simd(tmp_path):
    out = tmp_path / "pack.s"
    cmd = [b.hipcc()] + b.COMMON + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(b.CSRC, "fluxbin_pack.hip"),
                                    "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    asm = out.read_text()
    used = re.findall(r"^\s*\.amdhsa_kernel (\S*k_pack_signsILi16E\S*)$.*?\.amdhsa_next_free_vgpr (\d+)$", asm, re.M | re.S)
    assert len(used) == 1, used
    assert int(used[0][1]) <= 72, used
