"""Rules that stand in headers as inline functions, compiled for the host."""
import ctypes
import os
import subprocess

from paper_2311_09431_amd import build


def library(folder, source):
    """`source`, with the library's headers in reach, as a loaded library."""
    (folder / "rule.hip").write_text(source)
    lib = str(folder / "rule.so")
    subprocess.run([build._hipcc(), "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + build.CSRC,
                    "-I" + os.path.join(build.ROOT, "include"), str(folder / "rule.hip"), "-o", lib], check=True, capture_output=True)
    return ctypes.CDLL(lib)
