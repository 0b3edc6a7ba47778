"""Order of memory operations that the language leaves to the code generator, read from the assembly
that the library's own kernels compile to (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_1410_6685_amd import build as b


@pytest.mark.parametrize("kernel", ["lean_kernel<1, true>", "lean_kernel<4, true>"])
def test_finalizer_timeout_is_recorded_before_the_barrier(tmp_path, kernel):
    """The finalizing block's threads OR their timeout into the result's error word, and its first
    thread reads that word behind a barrier for the host.  s_barrier does not wait for memory
    operations of the other waves, so each of them has to wait for its own before it.  (The lean
    kernel's only ORs are these; the finalizer is every streaming kernel's.)"""
    src = tmp_path / "k.hip"
    src.write_text('#include <hip/hip_runtime.h>\n#include "sg_lean_kernel.h"\n'
                   f"template __global__ void sg::{kernel}(const sg::StreamArgs);\n")
    out = tmp_path / "k.s"
    r = subprocess.run([b.hipcc(), *[f for f in b.FLAGS if f != "-fPIC"], "-I", b.CSRC, "--offload-device-only", "-S",
                        "-o", os.fspath(out), os.fspath(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln.split(";")[0].strip() for ln in out.read_text().splitlines()]
    ors = [i for i, ln in enumerate(lines) if ln.startswith("global_atomic_or ")]
    assert ors
    waited = 0
    for i in ors:
        for ln in lines[i + 1:]:
            if ln.startswith("s_barrier"):
                pytest.fail(f"{kernel}: atomic or at line {i + 1} reaches a barrier unwaited")
            if ln.startswith("s_waitcnt") and ("vmcnt(0)" in ln or re.fullmatch(r"s_waitcnt (0|0x0)", ln)):
                waited += 1
                break
            if ln.startswith(("s_endpgm", "s_setpc")):
                break
    assert waited
