"""Builds libpvq.so (host code + gfx950 kernels) in-tree with hipcc, and the binding's native half for the installed
torch.  The library needs neither torch nor Python's headers."""
from __future__ import annotations

import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
_CSRC = os.path.join(_HERE, "csrc")
_INC = os.path.join(os.path.dirname(_HERE), "include")
LIB_PATH = os.path.join(_HERE, "libpvq.so")
# The binding's native half (csrc/pvq_torch.cpp), host code for one version of Python, which its name says, and one of
# torch, which it holds as a text (built_for).
TORCH_PATH = os.path.join(_HERE, "_pvq_torch" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))

SOURCES = ["pvq_host.cpp", "pvq_fast8_tables.cpp", "pvq_kernels.hip", "pvq_fast8.hip",
           "pvq_encode8.hip", "pvq_size_table.hip", "pvq_hadamard.hip", "pvq_wide.hip", "pvq_correct.hip", "pvq_walk.hip",
           "pvq_exact_check.hip"]

HEADERS = ["pvq_internal.h", "pvq_fast8.h", "pvq_hadamard_dev.h", "pvq_quantize_dev.h", "pvq_diagnostics.h", "pvq_small_table.h",
           "pvq_walk.h", "pvq_exact_dev.h"]

# -ffp-contract=off: the encoder's float32 results are part of the format (no fused multiply-adds
# unless written as fmaf); correctly rounded float32 division and square root likewise.
# The target-feature pair keeps the compiler from forming packed float32 instructions.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return [os.path.join(_CSRC, s) for s in SOURCES]


def _older(path, deps) -> bool:
    return not os.path.exists(path) or any(os.path.getmtime(d) > os.path.getmtime(path) for d in deps)


def library_is_stale() -> bool:
    return _older(LIB_PATH, sources() + [os.path.join(_CSRC, h) for h in HEADERS] + [os.path.join(_INC, "pvq.h")])


def built_for() -> str:
    """What a module for the installed torch holds."""
    import torch
    return f"pvq_torch built for torch {torch.__version__}"


def binding_fits() -> bool:
    """Whether the built module is there and is one for this Python and the installed torch."""
    if not os.path.exists(TORCH_PATH):
        return False
    with open(TORCH_PATH, "rb") as f:
        return built_for().encode() + b"\0" in f.read()


def binding_is_stale() -> bool:
    return not binding_fits() or _older(TORCH_PATH, [os.path.join(_CSRC, "pvq_torch.cpp"), os.path.join(_INC, "pvq.h")])


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("compilation failed:\n" + " ".join(cmd) + "\n" + err)
    return err


def _have_torch() -> bool:
    try:
        import torch  # noqa: F401
    except ImportError:
        return False
    return True


def _torch_object_command(obj: str):
    """Compiles the binding's native half against the headers of the installed torch and Python."""
    import torch
    from torch.utils import cpp_extension
    include = [f"-I{p}" for p in (*cpp_extension.include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"], _INC)]
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DPVQ_BUILT_FOR="{built_for()}"', *include,
            "-c", os.path.join(_CSRC, "pvq_torch.cpp"), "-o", obj]


def _torch_link_command(obj: str):
    """torch's libraries are the ones its import has loaded; libpvq.so lies beside the module."""
    import torch
    return [os.environ.get("CXX", "g++"), "-shared", "-o", TORCH_PATH, obj, f"-L{_HERE}", "-l:libpvq.so", "-Wl,-rpath,$ORIGIN",
            f"-L{os.path.join(os.path.dirname(torch.__file__), 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build(force: bool = True, verbose: bool = False, library: bool = True, binding: bool | None = None) -> str:
    """Compile the library and the binding's native half: every source to an object of its own (side by side), then
    the links.  binding: None = where torch is installed.
    Always compiles unless force=False, which leaves out what is up to date."""
    if binding is None:
        binding = _have_torch()
    library = library and (force or library_is_stale())
    binding = binding and (force or binding_is_stale())
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(_HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    objs, jobs = [], []
    if library:
        for src in sources():
            objs.append(os.path.join(objdir, os.path.basename(src) + ".o"))
            jobs.append([hipcc, *compile_flags, "-x", "hip", f"-I{_INC}", f"-I{_CSRC}", "-c", src, "-o", objs[-1]])
    if binding:
        torch_obj = os.path.join(objdir, "pvq_torch.cpp.o")
        jobs.append(_torch_object_command(torch_obj))
    with ThreadPoolExecutor(max_workers=8) as pool:
        errs = list(pool.map(_run, jobs))
    if library:
        errs.append(_run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB_PATH, *objs]))
    if binding:
        errs.append(_run(_torch_link_command(torch_obj)))
    if verbose:
        print("\n".join(e for e in errs if e.strip()))
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
