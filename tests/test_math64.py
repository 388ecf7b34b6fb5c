"""The float64 functions of the float64 paths, built for the host from their source:
their errors in units of the last place against 64-bit significands. The seeds of the
quotients and square roots are off by as much as their instructions may be."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("math64") / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas", "-I", os.path.join(HERE, "host"),
                    "-o", exe, os.path.join(HERE, "host", "math64_check.cpp")], check=True)
    out = {}
    for line in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines():
        name, e = line.split()
        out[name] = max(out.get(name, 0.0), float(e))
    return out


# the bounds that the source states; a long double's own error is below 0.001 of these units
@pytest.mark.parametrize("name,bound", [("log", 0.6), ("sin", 0.8), ("cos", 0.8), ("pow", 0.6),
                                        ("sqrt", 0.501), ("div", 0.501), ("divby", 0.501)])
def test_error_in_units_of_the_last_place(errors, name, bound):
    assert errors[name] <= bound, errors
