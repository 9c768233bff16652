"""Builds libonebit.so (the gfx950 HIP kernels and the C ABI) in-tree, the
binding's native argument checks (args_path()), and the HBM streaming probe's
own library lib/libhbmprobe.so."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", f) for f in ("onebit_kernels.hip", "onebit_abi.hip")]
LIB = os.path.join(HERE, "lib", "libonebit.so")
ARGS_SOURCE = os.path.join(HERE, "csrc", "binding_args.cpp")
PROBE_SOURCE = os.path.join(HERE, "csrc", "hbm_probe.hip")
PROBE = os.path.join(HERE, "lib", "libhbmprobe.so")

# -ffp-contract=off: every fp32 operation is rounded once, as the method's
# arithmetic is specified (no fused multiply-add contraction).
# -packed-fp32-ops: keep the compiler from emitting packed fp32 instructions.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math", "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def args_path() -> str:
    """The argument checks' library for this torch and this Python, whose
    interfaces it is compiled against: both are in its name, so that another
    torch or Python asks for a build of its own instead of loading this one."""
    import torch
    return os.path.join(HERE, "lib", "onebit_args-torch%s%s"
                        % (torch.__version__, sysconfig.get_config_var("EXT_SUFFIX")))


def _compile(compiler, flags, sources, target, verbose, libs=()):
    os.makedirs(os.path.dirname(target), exist_ok=True)
    tmp = target + ".tmp%d" % os.getpid()
    cmd = [compiler] + flags + ["-o", tmp] + sources + list(libs)
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                    if "packed-fp32-ops" not in l and "unused during compilation" not in l)
    if r.returncode != 0:
        sys.stderr.write(out + "\n")
        raise RuntimeError("%s failed building %s" % (compiler, os.path.basename(target)))
    if verbose and out.strip():
        print(out)
    os.replace(tmp, target)
    return target


def _args_flags():
    """Host compiler flags and libraries for an extension against torch."""
    import torch
    from torch.utils import cpp_extension
    flags = ["-O2", "-std=c++17", "-fPIC", "-shared",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for path in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]:
        flags += ["-isystem", path]
    libs = ["-L" + path for path in cpp_extension.library_paths()]
    return flags, libs + ["-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose: bool = False) -> str:
    _compile("hipcc", HIPCC_FLAGS, SOURCES, LIB, verbose)
    flags, libs = _args_flags()
    _compile("g++", flags, [ARGS_SOURCE], args_path(), verbose, libs)
    _compile("hipcc", HIPCC_FLAGS, [PROBE_SOURCE], PROBE, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
