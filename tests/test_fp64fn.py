"""The FP64 mode functions on the CPU, against 80-bit references over 2e6 arguments.

Errors in units of 2^-53 of the result.  A correctly rounded result is within 1,
so the table functions are held to 1.1 (the logarithm of the draws' uniform
numbers, whose leading terms cancel near 1, to 2.5); q = (f_k / f_knee)^-alpha,
1 / (1 + q) and sqrt(q) are to be no further off than with the C library's
functions, whose error there is the exponent's rounding: 2 % for the sample."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = tmp_path_factory.mktemp("fp64fn") / "fp64fn_host"
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(HERE, "fp64fn_host.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=300).stdout
    print(out)
    return {w[0]: (float(w[1]), float(w[2])) for w in (l.split() for l in out.splitlines())}


def test_ends_of_the_range(errors):
    assert errors["ends"][0] == 1


@pytest.mark.parametrize("name,bound", [("log_k", 1.1), ("log_u", 2.5), ("exp", 1.1), ("sqrt", 1.1), ("rcp", 1.1)])
def test_functions(errors, name, bound):
    assert errors[name][0] <= bound


@pytest.mark.parametrize("name", ["q", "inv", "sq"])
def test_noise_power_as_accurate_as_the_library(errors, name):
    most, rms = errors[name]
    assert most <= 1.02 * errors[name + "_lib"][0] and rms <= 1.02 * errors[name + "_lib"][1]
