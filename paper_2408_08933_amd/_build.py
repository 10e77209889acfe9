"""Compile the HIP/C++ sources into libroargraph.so (gfx950) in-tree."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libroargraph.so")
SOURCES = ["beam.hip", "knn.hip", "quant.hip", "canon.hip", "peaks.hip", "api.cpp", "host_build.cpp", "serve.cpp"]
# sources compiled in parts, with these flags (see beam.hip)
VARIANTS = {"beam.hip": [[]] + [[f"-DRG_BEAM_STORAGE={st}", f"-DRG_BEAM_PART={part}"] for st in (0, 1, 2)
                                for part in (0, 1, 2, 3)]}
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # canonical FP64 host arithmetic must not be contracted into FMAs
    "-ffp-contract=off",
    # never emit packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]


# Kernels whose correctness depends on issuing no vector-memory operation
# beyond their own (the FP16 kNN kernels count their outstanding loads by hand): a
# register spill would add scratch traffic to those counts, so it fails the
# build.
NO_SCRATCH = {"knn.hip": ["k_knn16", "k_scan16"]}


def _check_no_scratch(src: str, remarks: str) -> None:
    for kern in NO_SCRATCH.get(src, []):
        cur = None
        for line in remarks.splitlines():
            if "Function Name:" in line:
                cur = line.split("Function Name:")[1].split()[0]
            elif cur and kern in cur and "ScratchSize [bytes/lane]:" in line:
                size = int(line.split("ScratchSize [bytes/lane]:")[1].split()[0])
                if size != 0:
                    raise RuntimeError(f"{src}: {kern} spills to scratch ({size} bytes per lane)")


def units() -> list[tuple[str, list[str], str]]:
    """(source, extra flags, object file) of every compilation, the longest first."""
    u = []
    for src in SOURCES:
        for i, flags in enumerate(VARIANTS.get(src, [[]])):
            u.append((src, flags, os.path.join(OBJ, f"{src}.{i}.o" if i else f"{src}.o")))
    return sorted(u, key=lambda x: not x[1])


def _compile(unit: tuple[str, list[str], str]) -> str:
    src, flags, obj = unit
    path = os.path.join(CSRC, src)
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    extra = ["-Rpass-analysis=kernel-resource-usage"] if src in NO_SCRATCH else []
    cmd = [HIPCC, *COMMON, *lang, *extra, *flags, "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    _check_no_scratch(src, r.stderr)
    return obj


def build(jobs: int | None = None) -> str:
    """Compile every source (always) and link the shared library."""
    os.makedirs(OBJ, exist_ok=True)
    todo = units()
    jobs = jobs or min(len(todo), os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, todo))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
