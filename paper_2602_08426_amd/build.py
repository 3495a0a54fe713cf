"""Builds libprism.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libprism.so")
SOURCES = ["prism_estimate.hip", "prism_attn.hip"]
# bench-only probes of the machine's achievable peaks (bench.py --peaks); not part of libprism
PEAKS_LIB_PATH = os.path.join(HERE, "libprism_peaks.so")
PEAKS_SOURCES = ["prism_peaks.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # no packed-fp32 VALU code generation
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # queue pulls stay plain returning atomics whose result is waited for where it is used
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    # the registers of every kernel, for check_registers
    "-Rpass-analysis=kernel-resource-usage",
]
# of libprism alone (the probes keep their accumulators where the compiler puts them): accumulators of the compiler's MFMAs stay in
# VGPRs.  At head dim 256, the only kernels with more than 256 registers a lane, it otherwise puts them in AGPRs and moves each in
# and out for every rescale (330 of the 746 vector instructions of a 64 x 256 step, now none).
LIB_FLAGS = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]


def _compile(sources: list[str], out_path: str, verbose: bool, extra_flags: list[str] | None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *(extra_flags or []), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in sources], "-o", out_path]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = ("is not a recognized feature for this target", "kernel-resource-usage")
    err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    if SOURCES[-1] in sources:
        try:
            check_registers(res.stderr, row_loop_registers(CSRC))
        except RuntimeError:
            os.remove(out_path)
            raise
    return out_path


def row_loop_registers(folder: str) -> dict[int, tuple[int, int]]:
    """VGPRs and AGPRs of the generated row loops in `folder`, by queries per wave."""
    bodies = {}
    for q, name in ((64, "prism_attn_w64_body.inc"), (32, "prism_attn_w32_body.inc")):
        with open(os.path.join(folder, name)) as f:
            m = re.search(r"registers: (\d+) VGPRs, (\d+) AGPRs", f.read(400))
        bodies[q] = (int(m.group(1)), int(m.group(2)))
    return bodies


def check_registers(remarks: str, bodies: dict[int, tuple[int, int]]) -> None:
    """The generated row loops name their registers themselves.  A kernel around one is right only if the compiler set
    aside as many VGPRs and AGPRs as the loop goes up to (the first AGPR lies behind the last VGPR it counted) and
    spilled none, and the four-wave form shares a CU with another workgroup only within 256 registers together.  The
    compiler warns that the four-wave loop clobbers registers it has reserved and gives no word on what that means for
    the count, so every build holds the counts it reports (`remarks`) against the loops' own (`bodies`)."""
    for q, (vgprs, agprs) in bodies.items():
        m = re.search(rf"Function Name: \S*sparse_attn_w64_kernelILi{q}E(.*?)LDS Size", remarks, re.S)
        if m is None:
            raise RuntimeError(f"the compiler reports no registers of sparse_attn_w64_kernel<{q}>")
        got = {k: int(v) for k, v in re.findall(r"(VGPRs|AGPRs|VGPRs Spill|ScratchSize \[bytes/lane\]): (\d+)", m.group(1))}
        together = -(-got["VGPRs"] // 4) * 4 + got["AGPRs"]
        if (got["VGPRs"] < vgprs or got["AGPRs"] < agprs or got["VGPRs Spill"] or got["ScratchSize [bytes/lane]"] or
                together > (512 if q == 64 else 256)):
            raise RuntimeError(f"sparse_attn_w64_kernel<{q}>: its row loop needs {vgprs} VGPRs and {agprs} AGPRs, "
                               f"the compiler counted {got}")


def build_library(verbose: bool = False, extra_flags: list[str] | None = None) -> str:
    """Compile every HIP source into paper_2602_08426_amd/libprism.so (and the bench-only
    libprism_peaks.so beside it) and return the path of libprism.so."""
    # the hand-scheduled row loop of the 64-queries-per-wave attention kernel is generated
    gen = subprocess.run([sys.executable, os.path.join(CSRC, "gen_attn_w64.py"),
                          os.path.join(CSRC, "prism_attn_w64_body.inc")], capture_output=True, text=True)
    if gen.returncode != 0:
        raise RuntimeError(f"gen_attn_w64.py failed:\n{gen.stderr}")
    if verbose:
        print(gen.stderr.strip(), flush=True)
    _compile(PEAKS_SOURCES, PEAKS_LIB_PATH, verbose, None)
    return _compile(SOURCES, LIB_PATH, verbose, [*LIB_FLAGS, *(extra_flags or [])])


SELECT_ABLATION_BITS = {"select_noscores": 1, "select_nosearch": 2, "select_norefetch": 4}


def build_ablation(experiment: str, out_path: str, verbose: bool = False) -> str:
    """A measurement-only variant of libprism.so that leaves parts out; results are wrong by construction,
    control flow and bounds are unchanged.  `experiment` is a space-separated list of
      nosoft nocopy nowait nobar_mid nobar_end   parts of the 64-queries-per-wave attention row loop
                                                 (PRISM_W64_EXPERIMENT of gen_attn_w64.py),
      select_noscores select_nosearch select_norefetch   parts of the selection kernel
                                                 (PRISM_SELECT_ABLATION of prism_estimate.hip).
    The generated loop and the library go to the given path; the product library is not touched."""
    import shutil
    import tempfile
    with tempfile.TemporaryDirectory() as tmp:
        for name in os.listdir(CSRC):
            if name.endswith((".hip", ".h")):
                shutil.copy(os.path.join(CSRC, name), tmp)
        env = dict(os.environ, PRISM_W64_EXPERIMENT=experiment)
        gen = subprocess.run([sys.executable, os.path.join(CSRC, "gen_attn_w64.py"),
                              os.path.join(tmp, "prism_attn_w64_body.inc")], capture_output=True, text=True, env=env)
        if gen.returncode != 0:
            raise RuntimeError(f"gen_attn_w64.py failed:\n{gen.stderr}")
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        bits = sum(SELECT_ABLATION_BITS.get(tok, 0) for tok in experiment.split())
        cmd = [hipcc, *HIPCC_FLAGS, *LIB_FLAGS, f"-DPRISM_SELECT_ABLATION={bits}", "-I", os.path.join(ROOT, "include"), "-I", tmp,
               *[os.path.join(tmp, s) for s in SOURCES], "-o", out_path]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed ({res.returncode}):\n{res.stderr}")
        check_registers(res.stderr, row_loop_registers(tmp))
    return out_path


if __name__ == "__main__":
    if len(sys.argv) == 4 and sys.argv[1] == "--ablation":
        print(build_ablation(sys.argv[2], sys.argv[3], verbose=True))
    else:
        print(build_library(verbose=True))
