"""Builds the HIP kernels and the C-ABI library (libchipmunk_hip.so) for gfx950, in-tree, and beside it the
device-ceiling probes that bench.py --ceilings times (libchipmunk_ceilings.so) and the compiled part of the
Python binding (_native with Python's own suffix)."""
import glob
import hashlib
import importlib.machinery
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libchipmunk_hip.so")
PROBE_SRC = os.path.join(HERE, "probe", "ceilings.hip")
PROBE_LIB = os.path.join(HERE, "libchipmunk_ceilings.so")
NATIVE_SRC = os.path.join(HERE, "binding", "native.cpp")
NATIVE = os.path.join(HERE, "_native" + importlib.machinery.EXTENSION_SUFFIXES[0])
HEADER = os.path.join(HERE, "..", "include", "chipmunk.h")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-honor-nans",
    # hipcc -O3 must not form packed-fp32 instructions on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def is_stale():
    if not os.path.exists(LIB):
        return True
    if not native_fits() or os.path.getmtime(NATIVE_SRC) > os.path.getmtime(NATIVE):
        return True
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + [HEADER]
    return any(os.path.getmtime(d) > os.path.getmtime(LIB) for d in deps)


def native_stamp():
    """What the compiled binding is built against: the torch and the Python whose objects its code reads, and the declarations
    of the functions that it calls."""
    import torch
    header = hashlib.sha1(open(HEADER, "rb").read()).hexdigest()
    return (f"chipmunk binding for torch {torch.__version__} {getattr(torch.version, 'git_version', None)}, Python {sysconfig.get_config_var('SOABI')}, "
            f"chipmunk.h {header}.")


def native_fits():
    """Whether the compiled binding is there and was built against what runs now.  Read from the file: code for another torch is
    not to be loaded at all."""
    if not os.path.exists(NATIVE) or not os.path.exists(HEADER):
        return False
    with open(NATIVE, "rb") as f:
        return native_stamp().encode() in f.read()


def _native_command():
    """The compiled binding is host code against the headers of the torch that imports it."""
    import torch
    root = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DCHIPMUNK_BINDING_STAMP="{native_stamp()}"',
            "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-I" + sysconfig.get_paths()["include"], NATIVE_SRC, "-o", NATIVE,
            "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose=False):
    """Compile every .hip source into one shared library.  Always recompiles.  Without the compiled binding, which only makes
    calls shorter, the library is built all the same."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    native_command = _native_command()
    try:
        native = subprocess.Popen(native_command, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    except OSError as e:
        native, why = None, str(e)
    procs = []
    for src in sources():
        obj = src[:-4] + ".o"
        cmd = [hipcc] + [f for f in HIPCC_FLAGS if f != "-shared"] + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            failed = True
            sys.stderr.write(f"hipcc failed on {src}:\n{out}\n")
        elif verbose and out.strip():
            print(out)
    if native is not None:
        why, _ = native.communicate()
    if native is None or native.returncode != 0:
        sys.stderr.write(f"no compiled binding: {native_command[0]} failed on {NATIVE_SRC}:\n{why}\n")
        if os.path.exists(NATIVE):   # an earlier one may not fit the library that is built now
            os.remove(NATIVE)
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    for o in objs:
        os.remove(o)
    probe = subprocess.run([hipcc] + HIPCC_FLAGS + [PROBE_SRC, "-o", PROBE_LIB], stdout=subprocess.PIPE,
                           stderr=subprocess.STDOUT, text=True)
    if probe.returncode != 0:
        sys.stderr.write(probe.stdout)
        raise RuntimeError("hipcc failed on the ceiling probes")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
