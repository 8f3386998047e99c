"""Compile the HIP sources under csrc/ into paper_1810_09868_amd/libvgg_mi355x.so (gfx950)."""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
SOURCES = ["conv_igemm.hip", "conv_f32x3.hip", "conv_first.hip", "conv_pair.hip", "conv_wgrad.hip", "conv_wgrad_f32x3.hip", "conv_wgrad_bf16.hip", "pointwise.hip", "fc.hip", "probe.hip", "api.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-inline-asm"]
LIB = os.path.join(HERE, "libvgg_mi355x.so")
# Kernels that must not spill: their weight loads are in flight where the compiler takes the registers as written, and
# a load that lands in a register whose spilled value has been put back would be lost without an error.
NO_SPILLS = {"conv_igemm.hip": "conv3x3_igemm_wreg_kernel"}
REMARKS = ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics"]


def spilling_kernels(remarks: str, kernel: str):
    """(number of kernels whose name holds `kernel`, names of those that spill a vector register or use scratch memory)
    in the compiler's resource remarks."""
    name, seen, bad = "", 0, []
    for line in remarks.splitlines():
        m = re.search(r"remark:\s+Function Name: (\S+)", line)
        if m:
            name = m.group(1) if kernel in m.group(1) else ""
            seen += bool(name)
        m = re.search(r"remark:\s+(?:VGPRs Spill|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and name and int(m.group(1)) and name not in bad:
            bad.append(name)
    return seen, bad


def _compile(src: str) -> str:
    obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, *(REMARKS if src in NO_SPILLS else []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and "kernel-resource-usage" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if src in NO_SPILLS:
        seen, bad = spilling_kernels(r.stderr, NO_SPILLS[src])
        if bad or not seen:
            os.remove(obj)
            raise RuntimeError(f"{src}: {len(bad)} of {seen} variants of {NO_SPILLS[src]} spill: {bad}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build() -> str:
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    with ThreadPoolExecutor(max_workers=6) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build())
