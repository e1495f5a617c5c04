"""The many-row matrix-core kernel's LDS-direct copies: a wavefront waits for its own before each barrier that hands them to
the others. A barrier waits for no memory operation, so the wait has to stand in the source; waits that the compiler puts
before LDS reads because it cannot tell two buffers apart do not count. Checked on the assembly of this build's flags."""
import os
import re
import subprocess

import pytest

from paper_2608_15602_amd import build as b

COPY = re.compile(r"\bglobal_load_lds_|\bbuffer_load_.*\blds\b")
MEMORY = re.compile(r"^\s*(global_|buffer_|flat_|scratch_)")
WAIT = re.compile(r"^\s*s_waitcnt\b.*\bvmcnt\(0\)")


def _functions(asm):
    """The instruction lines and labels of every kernel."""
    out = {}
    for name, body in re.findall(r"^(\w+):\s*; @\1\n(.*?)^\s*s_endpgm", asm, re.M | re.S):
        out[name] = [l for l in body.splitlines() if re.match(r"^(\.LBB\w+:|\s+[a-z])", l)]
    return out


def test_every_barrier_follows_a_wait_for_the_copies(tmp_path):
    out = tmp_path / "pf.s"
    cmd = [b.hipcc()] + b.COMMON + ["-x", "hip", "--cuda-device-only", "-S",
                                    os.path.join(b.CSRC, "fluxbin_gemm_prefill.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels = {n: f for n, f in _functions(out.read_text()).items() if "k_gemm_prefill" in n}
    assert len(kernels) == 2, sorted(kernels)
    for name, lines in kernels.items():
        assert sum(bool(COPY.search(l)) for l in lines) >= 10, name   # before the loop and in it
        barriers = [i for i, l in enumerate(lines) if re.match(r"^\s+s_barrier", l)]
        assert barriers, name
        for i in barriers:
            waited = False
            for l in reversed(lines[:i]):
                if WAIT.match(l):
                    waited = True
                if waited or MEMORY.match(l) or l.startswith(".LBB"):
                    break
            assert waited, f"{name}: no wait for the copies before the barrier at instruction {i}"
