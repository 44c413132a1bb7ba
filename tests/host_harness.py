"""Small C++ programs against libpsa's internal host code (no GPU).

run(body, tmp_path): compile `body` as the inside of main(), with the
library's headers included and libpsa linked, run it and return its standard
output's lines.
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2601_14476_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def run(body, tmp_path):
    src, exe = tmp_path / "harness.cpp", tmp_path / "harness"
    src.write_text('#include "engine.hpp"\n#include "psa.h"\n#include <cstdio>\nint main() {\n' + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include", f"-I{PKG}/csrc",
                    str(src), "-o", str(exe), os.path.join(PKG, "libpsa.so"), f"-L{ROCM}/lib", "-lamdhip64",
                    f"-Wl,-rpath,{PKG}:{ROCM}/lib"], check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
