"""The step's FP64 functions, compiled for the host: no further off than the ROCm
device library's functions on the same arguments (measured on gfx950 over every 23-bit
uniform; x in +-50 for the exponential and the hop probability)."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1106_2899_amd", "csrc")

# (largest, root-mean-square) relative error of the library's
LIBRARY = {
    "log": (1.2589e-16, 4.7545e-17),
    "sin": (1.4844e-16, 4.4101e-17),
    "cos": (1.4844e-16, 4.4101e-17),
    "exp": (1.3711e-16, 4.9123e-17),
    "hop": (2.8857e-16, 7.0370e-17),
    "far": (1.3711e-16, 4.9123e-17),  # the whole range, +-700
}


@pytest.fixture(scope="module")
def errors():
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "f64")
        subprocess.check_call([hipcc, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}", "-O2",
                               "-std=c++17", "-march=native", "-ffp-contract=off", "-o", exe,
                               os.path.join(HERE, "f64_functions.cpp")], cwd=d)
        out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split("\n")
    return {r.split()[0]: tuple(float(x) for x in r.split()[1:]) for r in out if r}


@pytest.mark.parametrize("name", list(LIBRARY))
def test_no_further_off_than_the_library(errors, name):
    most, rms = errors[name]
    assert most <= LIBRARY[name][0] and rms <= LIBRARY[name][1], (name, most, rms)
