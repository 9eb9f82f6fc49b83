"""Build libmaxsim.so, and libmaxsim_probe.so (the benchmark's diagnostics), HIP for gfx950 only, in-tree with hipcc, and
_marshal.so, the native part of binding.py, which the binding also does without."""
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmaxsim.so")
PROBE_LIB = os.path.join(HERE, "libmaxsim_probe.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["api.hip", "forward.hip", "forward_f16.hip", "forward_bf16.hip", "forward_f32.hip", "forward_argmax.hip", "forward_wide.hip", "forward_wide_f16.hip", "forward_wide_bf16.hip", "forward_wide_f32.hip", "forward_splitd.hip", "backward.hip", "int8.hip", "int8_rows64.hip", "int8_wide.hip"]
PROBE_SOURCES = ["probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed fp32 VALU forms are switched off on purpose (they have produced wrong results on
# the test machines); the host pass warns that it does not know the feature, which is harmless
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # inputs are finite by contract: without this every max is preceded by a NaN-quieting copy
         "-fno-honor-nans",
         "-Wall", "-Wno-unused-function"]
FILE_FLAGS = {"forward_argmax.hip": ["-falign-loops=64"]}  # (the reason is at its top)


def marshal_abi():
    """What _marshal.so depends on beside its own source: the torch it speaks to through C++ and the Python that loads it."""
    import torch
    return "torch %s, Python %d.%d" % (torch.__version__, *sys.version_info[:2])


def marshal_command(out):
    """The compiler's call for the native part of binding.py, against the installed torch's headers and libraries. g++ where there is
    one: with the same source built by hipcc in the process, torch's own autograd step (its engine's thread woken by a backward of a
    cross-entropy alone, none of this package in it) takes 90 us instead of 83, and a step of 8 x 8 texts of 300 tokens 148 instead
    of 136, five processes of each in turn; the calls without autograd take the same."""
    import torch
    t = os.path.dirname(torch.__file__)
    cxx = ["g++"] if shutil.which("g++") else [HIPCC, "-x", "c++", "-no-hip-rt"]
    return (cxx + ["-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(), "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
             '-DMARSHAL_ABI="%s"' % marshal_abi()]
            + ["-isystem" + d for d in (os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include", sysconfig.get_paths()["include"])]
            + [os.path.join(CSRC, "marshal.cpp"), "-o", out, "-L" + os.path.join(t, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"])


def start_marshal():
    """Starts the compilation of _marshal.so and returns what ends it: in its place, or without it and a message where torch's or
    Python's headers are missing or of another kind, since the library does not need it."""
    tmp = MARSHAL + ".tmp%d" % os.getpid()
    try:
        pr = subprocess.Popen(marshal_command(tmp), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    except Exception as e:
        pr, why = None, repr(e)

    def finish():
        out = pr.communicate()[0] if pr else why
        if pr and pr.returncode == 0:
            os.replace(tmp, MARSHAL)
            return True
        sys.stderr.write("marshal.cpp does not compile here; the binding will work in Python alone:\n%s\n" % out)
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)  # (that of an earlier build is not this one's)
        return False
    return finish


def build(verbose: bool = False) -> str:
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    procs = []
    for src in SOURCES + PROBE_SOURCES:
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        cmd = [HIPCC] + FLAGS + FILE_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    finish_marshal = start_marshal()
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            failed = True
            sys.stderr.write("hipcc failed for %s:\n%s\n" % (src, out))
        elif verbose and out.strip():
            print(out)
    finish_marshal()
    if failed:
        raise RuntimeError("hipcc failed")
    n = len(SOURCES)
    for lib, lib_objs in ((LIB, objs[:n]), (PROBE_LIB, objs[n:])):
        tmp = lib + ".tmp%d" % os.getpid()
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + lib_objs
        subprocess.run(cmd, check=True)
        os.replace(tmp, lib)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
