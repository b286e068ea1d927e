"""Build the HIP engine (libqsv.so) in-tree for gfx950 with hipcc."""

import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqsv.so")

# Each source with its own definitions; the register-blocked passes compile once per amplitude
# type, direction and launch form, so that their instantiations build in parallel.
SOURCES = [("tile_rb.hip", [f"-DQSV_RB_REAL={r}", f"-DQSV_RB_ADJ={a}", f"-DQSV_RB_MULTI={m}"])
           for r in ("double", "float") for a in ("true", "false") for m in (0, 1)]
SOURCES += [(s, []) for s in ("tile_lds.hip", "qsv_kernels.hip", "pauli_multi.hip", "engine.cpp", "api.cpp", "batch.cpp", "mpnn.hip",
                              "noalloc.hip")]
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # Keep branches on wave-uniform values (the op type of a fused pass) as plain scalar
    # branches: structurizing them makes old and new register blocks live at once, and the
    # pass then copies its whole register block after every op.
    "-mllvm", "-structurizecfg-skip-uniform-regions=true",
    # Matrix-core operands and results in ordinary VGPRs: otherwise the fused-block op pulls
    # the whole register block into accumulation registers, which every other op must then
    # copy in and out.
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-function",
]


def hipcc():
    cand = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    return cand if os.path.exists(cand) else "hipcc"


def run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)


def build(verbose=False):
    """Compile every source and link paper_2406_17248_amd/libqsv.so (always rebuilds)."""
    tmp = LIB + ".tmp"
    inc = ["-I", os.path.join(HERE, "..", "include")]
    jobs = min(8, int(os.environ.get("MAX_JOBS", os.cpu_count() or 1)))
    with tempfile.TemporaryDirectory() as d, concurrent.futures.ThreadPoolExecutor(jobs) as pool:
        objs = [os.path.join(d, f"{i}.o") for i in range(len(SOURCES))]
        cmds = [[hipcc()] + HIPCC_FLAGS + defs + inc + ["-c", os.path.join(CSRC, s), "-o", o]
                for (s, defs), o in zip(SOURCES, objs)]
        list(pool.map(lambda c: run(c, verbose), cmds))
        run([hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared"] + objs + ["-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
