"""Build tests/ring_plans/_build/ring_plans: prints the ring-FFT plans of the built
library (linked against libshtx.so; host code only, no kernel is launched)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)
from paper_1908_06097_amd import build as lib_build  # noqa: E402

OUT = os.path.join(HERE, "_build")
EXE = os.path.join(OUT, "ring_plans")


def build() -> str:
    os.makedirs(OUT, exist_ok=True)
    libdir = os.path.dirname(lib_build.LIB)
    subprocess.run(["hipcc", "-x", "hip", *lib_build.FLAGS, "-I", lib_build.CSRC, os.path.join(HERE, "ring_plans.cpp"),
                    "-L", libdir, "-lshtx", "-Wl,-rpath,$ORIGIN/../../../paper_1908_06097_amd", "-o", EXE], check=True)
    return EXE


if __name__ == "__main__":
    print(build())
