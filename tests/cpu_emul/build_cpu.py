"""Builds tests/cpu_emul/libsttm_cpu.so: the library's own sources compiled with g++ against the CPU
stand-in for HIP in this folder (test infrastructure; the product is the hipcc build)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2507_07990_amd", "csrc")
LIB = os.path.join(HERE, "libsttm_cpu.so")
LIB_LARGE = os.path.join(HERE, "libsttm_cpu_large.so")  # every input takes the kernels of the large ones
# ... and a small one has several workgroups that list the elements of a search, more elements than a search keeps, and
# crowded bins
LARGE = ["-DSTTM_PYR_TILES_MAX=0", "-DSTTM_TEMPORAL_TILES_MAX=0", "-DSTTM_SEL_WHOLE=0", "-DSTTM_SEL_THREADS=64", "-DSTTM_SEL_LIST=32",
         "-DSTTM_SEL_REFINE=0", "-DSTTM_SEL_CROWD=40"]
# Every search has its elements listed, and keeps as many as on the device: lists that take several trips to be read.
LIB_LISTED, LISTED = os.path.join(HERE, "libsttm_cpu_listed.so"), ["-DSTTM_SEL_WHOLE=0"]
# Every search looks through all keys, and its bins hold more elements than it keeps (the sanitized build of the kernels of
# small inputs as well).
LIB_CROWDED, CROWDED = os.path.join(HERE, "libsttm_cpu_crowded.so"), ["-DSTTM_SEL_LIST=32"]
SOURCES = ["sttm_api.hip", "sttm_spatial.hip", "sttm_temporal.hip", "sttm_reduce.hip"]
SANITIZE_EXE = os.path.join(HERE, "sanitize_run")
SANITIZE_EXE_LARGE = os.path.join(HERE, "sanitize_run_large")


def _up_to_date(out):
    """Built after the last change of any file that goes into it."""
    if not os.path.exists(out):
        return False
    folders = [CSRC, os.path.join(ROOT, "include"), HERE, os.path.join(HERE, "hip")]
    files = [os.path.join(d, f) for d in folders for f in os.listdir(d) if f.endswith((".h", ".hip", ".cpp", "build_cpu.py"))]
    return os.path.getmtime(out) > max(map(os.path.getmtime, files))


def _compile(flags, extra_sources, out, verbose):
    if _up_to_date(out):
        return out
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", HERE, "-I", CSRC, "-Wno-unknown-pragmas",
           "-Wno-attributes"] + flags
    for s in [os.path.join(CSRC, s) for s in SOURCES] + [os.path.join(HERE, s) for s in ["emul.cpp"] + extra_sources]:
        cmd += ["-x", "c++", s]
    cmd += ["-o", out + ".part"]  # (in place only when it is whole)
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    os.replace(out + ".part", out)
    return out


def build_sanitized(verbose: bool = False, large: bool = False) -> str:
    """tests/cpu_emul/sanitize_main.cpp and the library's sources in one executable, under AddressSanitizer and
    UndefinedBehaviorSanitizer (any report ends the run with a non-zero status)."""
    flags = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-fno-omit-frame-pointer"]
    return _compile(flags + (LARGE if large else CROWDED), ["sanitize_main.cpp"], SANITIZE_EXE_LARGE if large else SANITIZE_EXE,
                    verbose)


def build(verbose: bool = False, large: bool = False) -> str:
    # (two of these live in one process: -fno-gnu-unique keeps the statics of their template functions apart)
    return _compile(["-fPIC", "-shared", "-fno-gnu-unique"] + (LARGE if large else []), [], LIB_LARGE if large else LIB,
                    verbose)


def build_listed(verbose: bool = False) -> str:
    return _compile(["-fPIC", "-shared", "-fno-gnu-unique"] + LISTED, [], LIB_LISTED, verbose)


def build_crowded(verbose: bool = False) -> str:
    return _compile(["-fPIC", "-shared", "-fno-gnu-unique"] + CROWDED, [], LIB_CROWDED, verbose)


if __name__ == "__main__":
    print(build_sanitized(verbose=True) if "--sanitize" in sys.argv else build(verbose=True))
