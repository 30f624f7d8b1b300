"""Build the C drivers of the C ABI into tests/native/bin (gcc; with
--sanitize thread also a ThreadSanitizer build, clang, linked against
libcgmi_tsan.so from `python -m paper_2608_09647_amd.build --sanitize thread`).

    python tests/native/build_native.py [--sanitize thread]
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
PKG = os.path.join(ROOT, "paper_2608_09647_amd")
BIN = os.path.join(HERE, "bin")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
DRIVERS = ["cabi_split"]


def build(sanitize: str | None = None, verbose: bool = False) -> list:
    os.makedirs(BIN, exist_ok=True)
    out = []
    for name in DRIVERS:
        src = os.path.join(HERE, name + ".c")
        if sanitize == "thread":
            exe = os.path.join(BIN, name + "_tsan")
            cmd = [f"{ROCM}/llvm/bin/clang", "-O1", "-g", "-std=c11", "-fsanitize=thread", src, "-o", exe,
                   f"-L{PKG}", "-l:libcgmi_tsan.so", f"-Wl,-rpath,{PKG}", "-lm"]
        else:
            exe = os.path.join(BIN, name)
            cmd = ["gcc", "-O2", "-std=c11", "-Wall", src, "-o", exe, f"-L{PKG}", "-l:libcgmi.so",
                   f"-Wl,-rpath,{PKG}", "-lm"]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        out.append(exe)
    return out


HOST_SOURCES = ["cgmi.cpp", "devmatrix.cpp", "staged.cpp", "fsai.cpp"]


def build_host_checks(verbose: bool = False) -> str:
    """tests/native/bin/host_checks: the library's host sources with the HIP
    calls of host_checks.cpp (g++; needs no GPU and not libcgmi.so).  Kernel
    launches that no check reaches stay unresolved."""
    os.makedirs(BIN, exist_ok=True)
    flags = ["-O1", "-g", "-std=c++17", "-fopenmp", "-fno-pie", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", "-w"]
    srcs = [os.path.join(PKG, "csrc", s) for s in HOST_SOURCES] + [os.path.join(HERE, "host_checks.cpp")]
    objs = [os.path.join(BIN, os.path.basename(s).replace(".cpp", ".hc.o")) for s in srcs]
    cmds = [["g++", *flags, "-c", s, "-o", o] for s, o in zip(srcs, objs)]
    if verbose:
        print("\n".join(" ".join(c) for c in cmds), flush=True)
    procs = [subprocess.Popen(c) for c in cmds]
    if any([p.wait() for p in procs]):
        raise RuntimeError("host_checks: a compile step failed")
    exe = os.path.join(BIN, "host_checks")
    subprocess.run(["g++", "-fopenmp", *objs, "-o", exe, "-no-pie", "-Wl,--unresolved-symbols=ignore-all"],
                   check=True)
    return exe


if __name__ == "__main__":
    san = sys.argv[2] if len(sys.argv) > 2 and sys.argv[1] == "--sanitize" else None
    print(build(san, verbose=True))
