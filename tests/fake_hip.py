"""Runs a piece of Python against the library on a recording stand-in for the HIP runtime (fake_hip.c), in a
process of its own: the library's host path on the CPU, with every launch, copy and allocation in a log."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

_PRELUDE = """
import ctypes, sys, types
fake = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
sys.modules["torch"] = types.ModuleType("torch")  # its own HIP runtime stays out of this process
sys.path[:0] = [{root!r}, {tests!r}]
import numpy as np
from paper_1309_3075_amd import _abi
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import EpochBatchEvaluator, EpochLikelihood, from_problem

def log():
    return fake.fake_log().decode().splitlines()
"""


def run(tmp_path, code):
    """Executes `code` there; an assertion that fails in it fails the calling test."""
    so = os.path.join(str(tmp_path), "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "fake_hip.c"), "-o", so], check=True)
    src = _PRELUDE.format(so=so, root=ROOT, tests=HERE) + textwrap.dedent(code)
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout + r.stderr)
    return r.stdout
