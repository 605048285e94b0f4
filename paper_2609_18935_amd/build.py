"""Builds libtailupdate.so (HIP for gfx950) in-tree.

    python -m paper_2609_18935_amd.build        # or build() from Python

Every .hip file under csrc/ is compiled with hipcc for gfx950 and linked into
paper_2609_18935_amd/libtailupdate.so. Packed-FP32 instructions are disabled
(-Xclang -target-feature -Xclang -packed-fp32-ops). The compiler's per-kernel resource
report (registers, scratch, LDS, occupancy) is kept in _build/kernel_resources.json.
"""
import concurrent.futures
import glob
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libtailupdate.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


RESOURCES = os.path.join(BUILD, "kernel_resources.json")
_FIELDS = {"VGPRs": "vgprs", "AGPRs": "agprs", "ScratchSize [bytes/lane]": "scratch_bytes",
           "Occupancy [waves/SIMD]": "waves_per_simd", "LDS Size [bytes/block]": "lds_bytes"}


def _resources(remarks: str) -> dict:
    """Per-kernel figures from hipcc's kernel-resource-usage remarks."""
    out, cur = {}, None
    for line in remarks.splitlines():
        m = re.search(r"remark:\s+Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+([A-Za-z][^:]*): (\d+)", line)
        if m and cur is not None and m.group(1).strip() in _FIELDS:
            cur[_FIELDS[m.group(1).strip()]] = int(m.group(2))
    return out


# Per-file options: MFMA accumulators in ordinary vector registers. The attention kernel runs
# two waves per SIMD (256 registers each) and may then use the whole budget, instead of
# splitting it in equal accumulator and vector halves; the delta rule's direct chain is
# spared 90 register moves per chunk, the probe's score passes one per score.
_VGPR_MFMA = ["-mllvm", "-amdgpu-mfma-vgpr-form=true"]
FILE_FLAGS = {"attention.hip": _VGPR_MFMA, "delta.hip": _VGPR_MFMA, "probe.hip": _VGPR_MFMA}


def _compile(src: str):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-Rpass-analysis=kernel-resource-usage", "-c",
           src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj, _resources(r.stderr)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    workers = max(1, min(len(sources), int(os.environ.get("MAX_JOBS", "8"))))
    with concurrent.futures.ThreadPoolExecutor(workers) as ex:
        done = list(ex.map(_compile, sources))
    objs = [o for o, _ in done]
    kernels = {}
    for _, res in done:
        kernels.update(res)
    with open(RESOURCES, "w") as f:
        json.dump(kernels, f, indent=1, sort_keys=True)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-Wl,--no-undefined", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
