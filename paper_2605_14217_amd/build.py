"""Builds libpreft.so (hand-written HIP for gfx950) and _marshal.so (the binding's marshalling) in-tree."""
from __future__ import annotations

import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libpreft.so")
MARSHAL_PATH = os.path.join(_HERE, "_marshal.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # scalar fp32 code only: no packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def sources():
    """preft_api.hip (the C ABI, the launch logic and the few kernels it instantiates itself), slots.hip, and
    the kernel instantiations of csrc/instances/ (written by csrc/gen_instances.py)."""
    inst = os.path.join(CSRC, "instances")
    groups = sorted(os.path.join(inst, n) for n in os.listdir(inst) if n.endswith(".hip")) if os.path.isdir(inst) else []
    return [os.path.join(CSRC, "preft_api.hip"), os.path.join(CSRC, "slots.hip")] + groups


def built_for() -> str:
    """The torch and Python whose object layouts marshal.cpp compiles in: _marshal.so is used with these only."""
    import sys

    import torch
    return f"torch {torch.__version__} {torch.version.git_version} python {sys.hexversion:x}"


def marshal_command(out: str):
    """g++ line of the extension module (host code only, against this torch's headers)."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DPREFT_BUILT_FOR="{built_for()}"']
    cmd += [f for d in include_paths() + [sysconfig.get_paths()["include"]] for f in ("-isystem", d)]
    return cmd + [os.path.join(CSRC, "marshal.cpp"), "-o", out, "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python"]


def build_marshal(tmpdir: str) -> bool:
    """Compile _marshal.so and put it in place.  The library does without it (calls go through ctypes): where g++, torch's headers or the
    compilation fail, that is said, an older module is removed and the answer is False."""
    import shutil
    import warnings
    try:
        built = os.path.join(tmpdir, "_marshal.so")
        proc = subprocess.run(marshal_command(built), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        why = proc.stdout[-4000:] if proc.returncode != 0 else None
    except (OSError, ImportError, AttributeError) as e:
        why = str(e)
    if why is not None:
        warnings.warn(f"_marshal.so is not built, calls will be marshalled in Python: {why}")
        if os.path.exists(MARSHAL_PATH):
            os.remove(MARSHAL_PATH)
        return False
    tmp = MARSHAL_PATH + f".{os.getpid()}.tmp"
    shutil.copyfile(built, tmp)
    os.chmod(tmp, 0o755)
    os.replace(tmp, MARSHAL_PATH)
    return True


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source (one hipcc per translation unit, in parallel) and link them into
    paper_2605_14217_amd/libpreft.so; returns its path.  Beside it _marshal.so, where that can be built."""
    import concurrent.futures
    import tempfile
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    jobs = max(1, min(len(sources()), int(os.environ.get("MAX_JOBS", "0")) or os.cpu_count() or 1, 16))
    messages = []

    def run(cmd):
        proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
        if proc.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + out)
        if out.strip():
            messages.append(out)

    with tempfile.TemporaryDirectory(prefix="preft_build_") as tmpdir:
        objects = [os.path.join(tmpdir, f"{i}_{os.path.basename(src)}.o") for i, src in enumerate(sources())]
        commands = [[hipcc] + compile_flags + ["-c", src, "-o", obj] for src, obj in zip(sources(), objects)]
        with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
            marshal = pool.submit(build_marshal, tmpdir)
            list(pool.map(run, commands))
            marshal.result()
        tmp = LIB_PATH + f".{os.getpid()}.tmp"
        run([hipcc] + HIPCC_FLAGS + objects + ["-o", tmp])
    if verbose and messages:
        print("\n".join(messages))
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
