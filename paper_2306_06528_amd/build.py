"""Build the C-ABI library (csrc/*.hip -> libsvgd.so) for gfx950 with hipcc."""
import glob
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
LIB = os.path.join(HERE, "libsvgd.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _run(cmd):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    return out


def build(verbose: bool = False) -> str:
    """Compile unconditionally, the sources side by side; returns the path of the library."""
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1, 8)) as pool:
            outs = list(pool.map(lambda so: _run(["hipcc", *HIPCC_FLAGS, "-c", "-o", so[1], so[0]]), zip(SOURCES, objects)))
        outs.append(_run(["hipcc", *HIPCC_FLAGS, "-shared", "-o", LIB, *objects]))
    if verbose:
        for out in outs:
            if out.strip():
                print(out)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
