"""Build the C-ABI library (csrc/*.hip -> libsvgd.so) for gfx950 with hipcc, and what Python calls it through
(csrc/binding.cpp -> _binding.<ABI of this Python>.so, host code against torch's C++ interface)."""
import glob
import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
LIB = os.path.join(HERE, "libsvgd.so")
BINDING = os.path.join(HERE, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))  # (another Python does not take it for its own)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _run(cmd):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    return out


def _binding_flags():
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    includes = [f for p in include_paths() + [sysconfig.get_paths()["include"]] for f in ("-isystem", p)]  # (their warnings are not ours)
    libs = [f for p in library_paths() for f in (f"-L{p}", f"-Wl,-rpath,{p}")]
    return (["-O2", "-std=c++17", "-fPIC", "-Wall", "-Wextra", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
             f'-DSVGD_TORCH_VERSION="{torch.__version__}"', *includes],
            [f"-L{HERE}", "-Wl,-rpath,$ORIGIN", "-lsvgd", *libs, "-ltorch_python", "-ltorch_cpu", "-lc10"])


def build(verbose: bool = False) -> str:
    """Compile unconditionally, the sources side by side; returns the path of the library."""
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, os.cpu_count() or 1, 8)) as pool:
            compile_flags, link_flags = _binding_flags()
            binding = os.path.join(tmp, "binding.o")
            host = pool.submit(_run, ["g++", *compile_flags, "-c", "-o", binding, os.path.join(HERE, "csrc", "binding.cpp")])
            outs = list(pool.map(lambda so: _run(["hipcc", *HIPCC_FLAGS, "-c", "-o", so[1], so[0]]), zip(SOURCES, objects)))
            outs.append(host.result())
        outs.append(_run(["hipcc", *HIPCC_FLAGS, "-shared", "-o", LIB, *objects]))
        outs.append(_run(["g++", "-shared", "-o", BINDING, binding, *link_flags]))
    if verbose:
        for out in outs:
            if out.strip():
                print(out)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
