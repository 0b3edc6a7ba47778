"""Compile the HIP sources into libsafegpu.so (gfx950) in this directory.

Every translation unit is built with hipcc in parallel, then linked into one shared
library.  Flags: -ffp-contract=off keeps every float32 node a separately rounded operation
(no fused multiply-adds across operations); packed fp32 instructions are disabled.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(os.path.dirname(HERE), "_build")
LIB = os.path.join(HERE, "libsafegpu.so")
SOURCES = ["stream.hip", "gemm.hip", "product.hip", "runtime.hip", "planner.hip", "exec.hip", "batch.hip", "mlp.hip", "tune.hip",
           "jit.hip", "host_checks.hip", "qsort.hip", "radix.hip", "nodes.hip", "gauss.hip", "linalg.hip",
           "persist.hip", "expr.hip", "noalloc.hip"]
# kernel sources compiled again at run time (hiprtc) for specialized passes; embedded in the
# library as strings
RTC_HEADERS = ["sg_stream_kernel.h", "sg_kernels.h", "sg_exp.h", "sg_exp_table.h", "sg_stream_ops.inc"]
ARCH = os.environ.get("SG_OFFLOAD_ARCH", "gfx950")
FLAGS = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-result"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def write_rtc_headers() -> None:
    """_build/sg_rtc_headers.h: the kernel headers as raw string literals."""
    out = ["// generated by build.py: kernel headers for run-time compilation", "#pragma once"]
    out.append(f"#define SG_RTC_NHEADERS {len(RTC_HEADERS)}")
    texts = []
    for name in RTC_HEADERS:
        with open(os.path.join(CSRC, name)) as fh:
            text = fh.read()
        if ")SGRTC\"" in text:
            raise RuntimeError(f"{name} contains the raw-string delimiter")
        texts.append(f'R"SGRTC({text})SGRTC"')
    out.append("static const char* const SG_RTC_HEADER_TEXT[] = {\n" + ",\n".join(texts) + "};")
    out.append("static const char* const SG_RTC_HEADER_NAME[] = {" + ", ".join(f'"{n}"' for n in RTC_HEADERS) + "};")
    path = os.path.join(BUILD, "sg_rtc_headers.h")
    new = "\n".join(out) + "\n"
    if not os.path.exists(path) or open(path).read() != new:
        with open(path, "w") as fh:
            fh.write(new)


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    cmd = [hipcc(), *FLAGS, "-I", BUILD, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    write_rtc_headers()
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    jobs = max(1, min(len(srcs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4))))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", f"--offload-arch={ARCH}", "-o", tmp, *objs, "-lhiprtc"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
