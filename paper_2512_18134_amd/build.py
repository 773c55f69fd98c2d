"""Build libmi355attn.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_2512_18134_amd.build

Three files come out.  Two libraries of the same sources: libmi355attn.so (the product) and
libmi355attn_debug.so (-DATTN_DEBUG_ENTRY_POINTS: the same code plus test-only entry
points that let a test pick the kernel, e.g. the program-order reference of the
schedule-equivalence tests).  Nothing in the package loads the debug library.
And _marshal.so, the host-only extension module that takes torch tensors to the entry
points (csrc/marshal.cpp); it is left out where torch or the headers of Python are not
installed (the C ABI needs neither).
"""
import itertools
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", "attn_fwd.hip"), os.path.join(HERE, "csrc", "attn_bwd.hip")]
LIB_PATH = os.path.join(HERE, "libmi355attn.so")
MARSHAL_SOURCE = os.path.join(HERE, "csrc", "marshal.cpp")
MARSHAL_PATH = os.path.join(HERE, "_marshal.so")
DEBUG_LIB_PATH = os.path.join(HERE, "libmi355attn_debug.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 VALU ops are kept out of the generated code on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
]


def _run_generator(cmd, verbose):
    """The generators take everything from their command line: run them with an empty environment so
    that nothing set in the caller's shell can change what is built."""
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True, env={})


def generate_sources(verbose=False, out_dir=None):
    """Run the loop generators: csrc/generated/*.inc (or out_dir)."""
    gen = os.path.join(HERE, "csrc", "gen_attn_loop.py")
    out_dir = out_dir or os.path.join(HERE, "csrc", "generated")
    os.makedirs(out_dir, exist_ok=True)
    for name in ("d64", "d64_w4", "d64_w2", "d128", "d128a", "d128a_w2", "d128_w2", "d128_w4", "d256a"):
        for dtype in ("bf16", "f16"):
            out = os.path.join(out_dir, "attn_loop_%s%s.inc" % (name, "" if dtype == "bf16" else "_" + dtype))
            _run_generator([sys.executable, gen, name, out, dtype], verbose)
    gen3 = os.path.join(HERE, "csrc", "gen_attn_bwd_loop.py")
    for kind, d, dtype in (("kv", 128, "bf16"), ("q", 128, "bf16"), ("kv", 128, "f16"), ("q", 128, "f16"),
                           ("kv", 64, "bf16"), ("q", 64, "bf16"), ("kv", 64, "f16"), ("q", 64, "f16")):
        out = os.path.join(out_dir, "attn_bwd_loop_%s_d%d%s.inc" % (kind, d, "" if dtype == "bf16" else "_" + dtype))
        _run_generator([sys.executable, gen3, kind, str(d), out, dtype], verbose)
    gen4 = os.path.join(HERE, "csrc", "gen_attn_bwd_wide_loop.py")
    for kind, waves, dtype in itertools.product(("kv", "q"), (2, 4), ("bf16", "f16")):
        out = os.path.join(out_dir, "attn_bwd_wide_loop_%s_w%d%s.inc" % (kind, waves, "" if dtype == "bf16" else "_" + dtype))
        _run_generator([sys.executable, gen4, kind, str(waves), out, dtype], verbose)


def _hipcc():
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(lib_path, extra, verbose):
    return _run_compiler([_hipcc()] + HIPCC_FLAGS + extra, SOURCES, [], lib_path, verbose)


def _compile_marshal(verbose):
    """The extension module: host code against torch's headers and libraries (which the importing process has loaded).
    Without torch or Python's headers there is nothing to compile it against: no module, not an older one either, and
    the binding does all of the marshalling in Python."""
    if os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)
    include = sysconfig.get_paths()["include"]
    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        torch = None
    if torch is None or not os.path.exists(os.path.join(include, "Python.h")):
        print("_marshal.so: left out (torch or Python.h is not installed)", flush=True)
        return None
    cmd = [_hipcc(), "-no-hip-rt", "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    cmd += ["-I" + i for i in cpp_extension.include_paths() + [include]]
    libs = ["-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    return _run_compiler(cmd, [MARSHAL_SOURCE], libs, MARSHAL_PATH, verbose)


def _run_compiler(cmd, sources, libs, lib_path, verbose):
    tmp = lib_path + ".tmp.%d" % os.getpid()
    cmd = cmd + ["-o", tmp] + sources + libs
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("%s failed:\n%s" % (cmd[0], out))
    if verbose and out.strip():
        print(out)
    os.replace(tmp, lib_path)
    return lib_path


def build_library(verbose=False, debug=True):
    """Generate the scheduled loops, then compile every HIP source into LIB_PATH (and, with the test-only
    entry points, into DEBUG_LIB_PATH), and the extension module.  Raises on failure."""
    generate_sources(verbose)
    _compile(LIB_PATH, [], verbose)
    if debug:
        _compile(DEBUG_LIB_PATH, ["-DATTN_DEBUG_ENTRY_POINTS"], verbose)
    _compile_marshal(verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)
