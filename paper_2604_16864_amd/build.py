"""Builds libhs.so (the C-ABI library) for gfx950 with hipcc and _hs_torch.so (the binding's native part), in-tree."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhs.so")
NATIVE = os.path.join(HERE, "_hs_torch.so")
SOURCES = ["hs_api.hip", "hs_compress.hip", "hs_decode.hip", "hs_prefill.hip", "hs_prefill_mixed.hip", "hs_prefill_narrow.hip", "hs_prefill_narrow_mixed.hip", "hs_probe.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option", "-Wno-inline-asm",
]
# The scheduler's own register trackers: the prefill loops of tensors with one kind of tile come out 0.5 to 5 % faster with them
# (1K prompt 22.9 -> 22.4 us, 16 prompts of 1K 157 -> 150), those of mixed tensors 1 to 3 % slower (8K prompt, dense ends 379 -> 391); with slabs
# of 16 queries every kind gains up to 1.5 % (512 tokens 11.06 -> 10.97, dense ends 13.96 -> 13.85).  Mixed tensors in slabs of 16 want the
# scheduler that looks for parallel instructions (256 queries on 1024 tokens, half of the keys dense 19.9 with the plain one's
# max-ilp, 18.2 with the trackers, 17.9; fp16, dense ends, 512 tokens 14.1 / 13.1 / 12.6).
_TRACKERS = ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"]
FILE_FLAGS = {"hs_prefill.hip": _TRACKERS, "hs_prefill_narrow.hip": _TRACKERS, "hs_prefill_narrow_mixed.hip": ["-mllvm", "-amdgpu-sched-strategy=iterative-ilp"]}


def native_command():
    """The C++ compiler's command line for the Python module, against the torch that is installed."""
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
            f'-DHS_TORCH_VERSION="{torch.__version__}"', "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(root, "include"),
            "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
            "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "hs_torch.cpp"),
            "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10", "-lc10_hip", "-o", NATIVE]


def build_lib(verbose=True, extra=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs, failed = [], []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, *FILE_FLAGS.get(src, []), *extra, "-DHS_BUILD", "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    try:
        procs.append(("hs_torch.cpp", subprocess.Popen(native_command(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    except OSError as e:                    # no such compiler
        failed.append(f"hs_torch.cpp ({e})")
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if verbose and out.strip():
            print(out)
        if p.returncode != 0:
            failed.append(src)
    if not set(failed) & set(SOURCES):      # the library does not need the native part: it is there also where that one cannot be built
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    if failed:
        raise RuntimeError(f"the compiler failed on {', '.join(failed)}")
    return LIB


if __name__ == "__main__":
    print(build_lib(extra=sys.argv[1:]))
