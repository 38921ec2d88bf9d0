"""Builds the tests' own device code (next to its source, as the library is)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libsqrt_normal_check.so")


def build() -> str:
    from paper_2409_07148_amd import build as libbuild
    subprocess.run([libbuild.HIPCC, *libbuild.FLAGS, "-shared", os.path.join(HERE, "sqrt_normal_check.hip"), "-o", LIB],
                   check=True, capture_output=True)
    return LIB
