"""Build the HIP library libcurast.so in-tree for gfx950 (MI355X).

Arithmetic flags matter for bit-exact results: -ffp-contract=off (no implicit fused multiply-add;
explicit __builtin_fmaf only), correctly rounded fp32 division, fp32 denormals kept, packed-fp32
instructions disabled.  Run: python -m paper_2604_21749_amd.build
"""
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
# Translation units: (source, object name, macros).  The variants of the stage-1 kernels are units of
# their own, so that they compile in parallel.
UNITS = [("raster.hip", f"raster_strips_{t}", [f"-DCURAST_STRIPS_TPT={t}"]) for t in (8, 4, 2)]
UNITS += [("raster.hip", f"raster_{b}_{t}", [f"-DCURAST_FAST_BLOCK={b}", f"-DCURAST_FAST_TPT={t}"])
          for t in (8, 4, 2, 1) for b in (64, 128, 256, 512)]
UNITS += [(f, f[:-4], []) for f in ("raster.hip", "resolve.hip", "runtime.hip", "autotune.hip", "compress.hip")]
LIB = os.path.join(HERE, "libcurast.so")
ARCH = os.environ.get("CURAST_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-gpu-flush-denormals-to-zero", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False) -> str:
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    objs = [os.path.join(build_dir, name + ".o") for _, name, _ in UNITS]

    def compile_unit(unit, obj):
        src, _, macros = unit
        cmd = [hipcc()] + [f for f in FLAGS if f != "-shared"] + macros + [
            "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        return subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)

    jobs = max(1, min(int(os.environ.get("MAX_JOBS", "0") or 0) or (os.cpu_count() or 1), 16))
    with ThreadPoolExecutor(jobs) as pool:
        results = list(pool.map(compile_unit, UNITS, objs))
    failed = []
    for (src, name, _), p in zip(UNITS, results):
        text = p.stdout.decode(errors="replace")
        # the host pass does not know the packed-fp32 feature name; that warning is harmless
        lines = [ln for ln in text.splitlines() if "packed-fp32-ops" not in ln]
        if lines and (verbose or p.returncode):
            print("\n".join(lines), flush=True)
        if p.returncode:
            failed.append(name)
    if failed:
        raise RuntimeError(f"hipcc failed for {failed}")
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", LIB + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
