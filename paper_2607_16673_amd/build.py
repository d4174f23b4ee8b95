"""Build libsla.so (hand-written HIP for gfx950 behind the C ABI of
include/sla.h) in-tree, next to this file.

Every HIP translation unit is compiled by hipcc for gfx950 only, with packed
fp32 instructions disabled (the library relies on ordinary fp32 VALU and
matrix-core arithmetic), then linked into one shared library.  The Python
binding's marshalling module (_native) is host code linked against it and
against torch; the library needs neither torch nor Python and is installed
first.
"""
import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsla.so")
NATIVE = os.path.join(HERE, "_native.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

# (source, object name, definitions); the tile kernel first, it takes longest
SOURCES = [("verify_tile.hip", "verify_tile_%d_%s_%s" % (dk, form, dt),
            ["-DSLA_TILE_DK=%d" % dk, "-DSLA_TILE_GATES=%d" % (form == "gates"), "-DSLA_TILE_F32=%d" % (dt == "f32")])
           for dk in (128, 256, 64) for form in ("scalar", "gates") for dt in ("bf16", "f32")]
SOURCES += [(src, os.path.splitext(src)[0], []) for src in
            ("api.cpp", "commit.hip", "conv.hip", "decode.hip", "draft.hip", "verify_serial.hip",
             "verify_tile_dispatch.cpp")]
COMMON = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH, "-I" + INCLUDE, "-I" + CSRC,
          "-Wall", "-Wno-unused-result",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(unit, verbose: bool) -> str:
    src, name, defines = unit
    obj = os.path.join(BUILD, name + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [HIPCC] + COMMON + defines + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                    if "packed-fp32-ops" not in l and l.strip())
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out and verbose:
        print(out, flush=True)
    return obj


def _torch_dir() -> str:
    """torch's place without importing it."""
    spec = importlib.util.find_spec("torch")
    if spec is None or not spec.origin:
        raise RuntimeError("torch is not installed: the Python binding's native module cannot be built")
    return os.path.dirname(spec.origin)


def _compile_native(verbose: bool) -> str:
    """The marshalling module's object file (host code only)."""
    torch = _torch_dir()
    obj = os.path.join(BUILD, "torch_binding.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-I" + INCLUDE, "-isystem" + os.path.join(torch, "include"), "-isystem/opt/rocm/include",
           "-isystem" + sysconfig.get_paths()["include"], "-Wall", "-Wno-unused-result",
           "-c", os.path.join(CSRC, "torch_binding.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
    except FileNotFoundError as e:
        raise RuntimeError("g++ is not installed: the Python binding's native module cannot be built") from e
    if r.returncode != 0:
        raise RuntimeError("g++ failed for torch_binding.cpp:\n" + r.stdout + r.stderr)
    return obj


def _link_native(obj: str, verbose: bool) -> None:
    torch = os.path.join(_torch_dir(), "lib")
    cmd = ["g++", "-shared", "-fPIC", "-o", NATIVE + ".tmp", obj, "-L" + HERE, "-l:libsla.so", "-L" + torch, "-ltorch_python",
           "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + torch]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(NATIVE + ".tmp", NATIVE)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        native = ex.submit(_compile_native, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", LIB + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    # the C library stands on its own: a module that cannot be built leaves it in place
    _link_native(native.result(), verbose)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
