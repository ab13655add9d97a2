"""Compile the HIP sources for gfx950: csrc/ into paper_2603_05168_amd/libsbn.so (the layer) and bench_csrc/ into
paper_2603_05168_amd/libsbn_probe.so (ceiling probes of the benchmark, apart from the layer's library); and the marshalling of the
forward calls, csrc/sbn_fastcall.cpp, against the installed torch into paper_2603_05168_amd/_fastcall.so.  The last is an accelerator of
the Python code that does the same: where it does not compile, a warning says so and the package works without it."""
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsbn.so")
PROBE_SRC = os.path.join(HERE, "bench_csrc")
PROBE_LIB = os.path.join(HERE, "libsbn_probe.so")
FASTCALL_SRC = os.path.join(CSRC, "sbn_fastcall.cpp")
FASTCALL_LIB = os.path.join(HERE, "_fastcall.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                      # quantizer arithmetic must round exactly as written
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def fastcall_command(compiler="g++"):
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    includes = cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"]]
    libs = cpp_extension.library_paths("cuda")
    return ([compiler, "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f'-DSBN_TORCH_VERSION="{torch.__version__}"'] + [f"-I{i}" for i in includes] +
            ["-o", FASTCALL_LIB, FASTCALL_SRC] + [f"-L{l}" for l in libs] + ["-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"] +
            [f"-Wl,-rpath,{libs[0]}"])


def build_fastcall(compiler="g++") -> bool:
    """False, with a warning and without a library of an earlier build left behind, where it does not compile."""
    if os.path.exists(FASTCALL_LIB):
        os.remove(FASTCALL_LIB)
    try:
        command = fastcall_command(compiler)
        p = subprocess.run(command, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out, ok = p.stdout, p.returncode == 0
    except (ImportError, OSError) as e:   # no torch to build against, no compiler
        out, ok = str(e), False
    if not ok:
        sys.stderr.write(f"warning: {FASTCALL_SRC} was not built, forward calls are marshalled in Python\n{out}\n")
    return ok


def fastcall_is_current() -> bool:
    """Built from this source against the torch that is installed."""
    import importlib.util
    if not os.path.exists(FASTCALL_LIB) or os.path.getmtime(FASTCALL_LIB) < os.path.getmtime(FASTCALL_SRC):
        return False
    try:
        import torch
        spec = importlib.util.spec_from_file_location("_fastcall", FASTCALL_LIB)
        return importlib.util.module_from_spec(spec).torch_version == torch.__version__
    except (ImportError, AttributeError):
        return False


def build(force: bool = True, verbose: bool = False) -> str:
    srcs = sources()
    probe_srcs = sorted(glob.glob(os.path.join(PROBE_SRC, "*.hip")))
    fastcall = force or not fastcall_is_current()
    deps = srcs + probe_srcs + glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    if not force and all(os.path.exists(l) and all(os.path.getmtime(l) >= os.path.getmtime(d) for d in deps) for l in (LIB, PROBE_LIB)):
        if fastcall:
            build_fastcall()
        return LIB
    objs = []
    probe_objs = []
    procs = []
    for s in srcs + probe_srcs:
        o = s[:-4] + ".o"
        (probe_objs if s in probe_srcs else objs).append(o)
        cmd = ["hipcc", "-c"] + [f for f in FLAGS if f != "-shared"] + ["-o", o, s]
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    if fastcall:
        build_fastcall()   # beside them
    failed = False
    for s, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = True
            sys.stderr.write(f"--- {s}\n{out}\n")
        elif verbose and out.strip():
            sys.stderr.write(f"--- {s}\n{out}\n")
    if failed:
        raise RuntimeError("compilation failed")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, check=True)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", PROBE_LIB] + probe_objs, check=True)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
