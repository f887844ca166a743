"""Rounding of the P3 tetrahedron's point orbits, on the CPU: the kernels'
element arithmetic compiled for the host, against extended precision. The
orbits may be no further off than the products of the tabulated derivatives,
whatever the nodal field and the coefficient are; the bound is 1 for the ratio
of the RMS errors over the same 3000 elements."""
import os
import pathlib
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    exe = tmp_path_factory.mktemp("p3") / "p3_rounding"
    cxx = pathlib.Path(os.environ.get("ROCM_PATH", "/opt/rocm")) / "llvm" / "bin" / "clang++"
    subprocess.run([str(cxx), "-std=c++17", "-O1", "-ffp-contract=off", "-I", str(ROOT / "tests" / "host_hip"),
                    "-I", str(ROOT / "include"), "-I", str(ROOT / "paper_1607_04245_amd" / "csrc"),
                    str(ROOT / "tests" / "p3_rounding.cpp"), "-o", str(exe), "-lm"], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    return {tuple(x.split()[:4]): [float(y) for y in x.split()[4:]] for x in lines}


@pytest.mark.parametrize("physics", ["laplace", "elasticity"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("field", ["independent", "offset", "linear", "smooth"])
def test_orbits_round_no_more_than_the_table(errors, physics, dtype, field):
    for coef in ("independent", "constant", "spike"):
        r_tab, r_orb, d_tab, d_orb = errors[physics, dtype, field, coef]
        assert 0 < r_orb <= r_tab, (coef, r_orb / r_tab)
        assert 0 < d_orb <= d_tab, (coef, d_orb / d_tab)
