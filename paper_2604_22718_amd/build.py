"""Build the HIP library in-tree: ``python -m paper_2604_22718_amd.build``."""
import os
import subprocess
import sys
import tempfile
import threading
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "librtt.so")
CSRC = os.path.join(HERE, "csrc")
# Objects, built in parallel: name, source, extra flags.  The flip-ratio
# passes and the sampler once per core type.  The sampler takes its
# matrix-op results in ordinary vector registers: its rows go straight from
# one matrix op to the vector ALUs and back, and with accumulators in the
# other half of the register file every result word was moved first.
UNITS = [("rtt_lib", "rtt_lib.hip", [])]
for _d in ("DF32", "DBF16", "DFP8"):
    UNITS.append((f"rtt_pass_{_d}", "rtt_pass.hip", [f"-DRTT_CORES={_d}"]))
    UNITS.append((f"rtt_chain_{_d}", "rtt_chain.hip", [f"-DRTT_CORES={_d}", "-mllvm", "-amdgpu-mfma-vgpr-form=1"]))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions stay off: the compiler must not form them
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
    "-Wno-unused-result", "-pthread",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building librtt.so")


def build(verbose: bool = False) -> str:
    # objects in a directory of this build's own: several may run at once
    with tempfile.TemporaryDirectory(prefix="librtt_") as tmp, ThreadPoolExecutor(len(UNITS)) as ex:
        objs = [os.path.join(tmp, f"{name}.o") for name, _, _ in UNITS]
        jobs = [ex.submit(_run, [HIPCC, *FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj], verbose)
                for (_, src, defs), obj in zip(UNITS, objs)]
        for j in jobs:
            j.result()
        out = f"{LIB}.tmp{os.getpid()}_{threading.get_ident()}"   # beside the library: replaced in one step
        try:
            _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", *objs, "-o", out], verbose)
            os.replace(out, LIB)
        finally:
            if os.path.exists(out):
                os.remove(out)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
