"""Launch configurations on the CPU: tests/launch_shapes.cpp calls the library
with its own recorder in place of the runtime's launch function and prints
kernel, grid, workgroup and workgroup order (0 launch, 1 XCD by XCD, 2 runs)."""
import os
import pathlib
import re
import subprocess

import pytest

from paper_1607_04245_amd import _native as N
from paper_1607_04245_amd import meshgen as mg

ROOT = pathlib.Path(__file__).resolve().parents[1]
F32, F64 = N.F32, N.F64


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    exe = tmp_path_factory.mktemp("launch") / "launch_shapes"
    rocm = pathlib.Path(os.environ.get("ROCM_PATH", "/opt/rocm")) / "lib"
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "launch_shapes.cpp"), str(N.LIB_PATH), f"-Wl,-rpath,{N.LIB_PATH.parent}",
                    f"-Wl,-rpath,{rocm}", "-Wl,--allow-shlib-undefined", "-o", str(exe)], check=True)

    def run(*commands):
        """One dict per launch of the calls among the commands."""
        text = "".join(" ".join(map(str, c)) + "\n" for c in commands)
        env = {k: v for k, v in os.environ.items() if k != "FEM_TUNE_CACHE"}
        out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True, env=env).stdout
        res = []
        for line in out.splitlines():
            name, gx, gy, block, order = line.rsplit(" ", 4)
            kernel, args = re.fullmatch(r"(?:void)?femq::(\w+)<(.*)>", name).groups()
            res.append(dict(kernel=kernel, args=args.split(","), grid=(int(gx), int(gy)), block=int(block), order=int(order)))
        return res

    return run


def _lanes(n, vec):
    return -(-n // vec)


# a chosen configuration with the built-in one's values is used as it is, at odd
# words too, where the built-in one is refined
@pytest.mark.parametrize("call,op", [("residual", N.OP_RESIDUAL), ("backward", N.OP_BACKWARD)])
@pytest.mark.parametrize("dtype,wide", [(F32, 4), (F64, 2)])
@pytest.mark.parametrize("n,offset", [(1000001, 0), (1 << 20, 1)])
def test_chosen_shape_at_odd_words(launches, call, op, dtype, wide, n, offset):
    key = (3, mg.LAPLACE, mg.RULE_TET4)
    c = (call, *key, N.COEF_QUAD, dtype, n, offset)
    built_in, chosen = launches(c, ("set", op, *key, dtype, N.STRATEGY_LANE, 1, 4, 0), c)
    assert built_in["args"][4] == str(wide) and built_in["block"] == 64
    assert chosen["args"][4] == "1" and chosen["block"] == 256 and chosen["grid"] == (_lanes(n, 256), 1)


@pytest.mark.parametrize("order,op,rule", [(1, N.OP_JACOBIAN, mg.RULE_TET4), (2, N.OP_JACOBIAN_P2, mg.RULE_TET11),
                                           (3, N.OP_JACOBIAN_P3, mg.RULE_TET11)])
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("waves,per_cu", [(1, 0), (2, 8), (4, 1)])
@pytest.mark.parametrize("n", [2000, 70001, 1000000, 1000001])
def test_chosen_matrix_shape(launches, order, op, rule, dtype, waves, per_cu, n):
    """Element matrices: the waves that were chosen, and no more workgroups
    than the chosen persistent grid, however many share a tile's columns."""
    key = (3, mg.ELASTICITY, rule)
    got, = launches(("set", op, *key, dtype, N.STRATEGY_LANE, 1, waves, per_cu),
                    ("jacobian", *key, N.COEF_QUAD, dtype, n, 0, order))
    assert got["block"] == 64 * waves
    if per_cu:
        cap = 256 * per_cu
        assert got["grid"][0] * got["grid"][1] <= cap
        vec = int(got["args"][3]) if order < 3 else 1
        if _lanes(n, 64 * waves * vec) >= cap:   # a persistent grid is filled
            assert got["grid"] == (cap, 1)


def test_built_in_matrix_shapes(launches):
    """Small meshes deal a tile's columns out (48 waves of 2926 elements to 42
    of them); from two waves per SIMD on they do not."""
    key = (3, mg.ELASTICITY, mg.RULE_TET11)
    small, large = launches(("jacobian", *key, N.COEF_QUAD, F32, 2926, 0, 3), ("jacobian", *key, N.COEF_QUAD, F32, 131072, 0, 3))
    assert small["grid"] == (12, 42) and large["grid"] == (512, 1)
