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
@pytest.mark.parametrize("dtype,waves,odd", [(F32, 4, (4, 1)), (F64, 1, (1, 4))])
@pytest.mark.parametrize("n,offset", [((1 << 21) + 1, 0), (1 << 21, 1)])
def test_chosen_shape_at_odd_words(launches, call, op, dtype, waves, odd, n, offset):
    key = (3, mg.LAPLACE, mg.RULE_TET4)
    c = (call, *key, N.COEF_QUAD, dtype, n, offset)
    whole, built_in, chosen = launches((call, *key, N.COEF_QUAD, dtype, (1 << 21) - 32, 0), c,
                                       ("set", op, *key, dtype, N.STRATEGY_LANE, 1, waves, 0), c)
    assert (whole["args"][4], whole["block"]) == ("1", 64 * waves)
    assert (built_in["args"][4], built_in["block"]) == (str(odd[0]), 64 * odd[1])
    assert (chosen["args"][4], chosen["block"]) == ("1", 64 * waves) and chosen["grid"] == (_lanes(n, 64 * waves), 1)


# rows at odd words, the arrays on 16 bytes: 16 bytes per lane from 1280 waves and 32
# MiB of rows (22 of a tet's Laplacian) on
@pytest.mark.parametrize("call", ["residual", "backward"])
@pytest.mark.parametrize("dtype,n,vec", [(F32, 327676, 1), (F32, 400004, 4), (F32, 400002, 1),
                                         (F64, 163838, 1), (F64, 220002, 2), (F64, 220001, 1)])
def test_width_at_odd_words(launches, call, dtype, n, vec):
    got, = launches((call, 3, mg.LAPLACE, mg.RULE_TET4, N.COEF_QUAD, dtype, n, 0))
    assert (got["args"][4], got["block"]) == (str(vec), 64 if vec > 1 else 256)


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


# rows at whole lines: plain stores in runs of workgroups where the last-level cache
# can hold some of them, streaming stores in launch order above; at odd words plain
# stores in runs, but FP64 triangles stream when large
@pytest.mark.parametrize("dim,physics,dtype,n,offset,stream", [
    (3, mg.ELASTICITY, F32, 1 << 20, 0, 0), (3, mg.ELASTICITY, F32, 2796160, 0, 0), (3, mg.ELASTICITY, F32, 2796224, 0, 1),
    (3, mg.LAPLACE, F64, (1 << 20) - 32, 0, 1), (2, mg.LAPLACE, F64, (1 << 22) - 32, 0, 0), (3, mg.ELASTICITY, F32, 2796224, 1, 0),
    (3, mg.ELASTICITY, F64, 1 << 21, 1, 0), (2, mg.ELASTICITY, F64, 1 << 21, 1, 0), (2, mg.ELASTICITY, F64, 3100000, 1, 0),
    (2, mg.ELASTICITY, F64, 3100704, 1, 1)])
def test_row_stores(launches, dim, physics, dtype, n, offset, stream):
    rule = mg.RULE_TRI3 if dim == 2 else mg.RULE_TET4
    got, = launches(("residual", dim, physics, rule, N.COEF_QUAD, dtype, n, offset))
    assert got["args"][5] == ("true" if stream else "false") and got["order"] == (0 if stream else 2)


# rows a multiple of 8 MiB apart: XCD by XCD (an eighth of the workgroups each where
# they stream, from 512 MiB of rows on); 4 MiB and an odd multiple of 2 are not that
@pytest.mark.parametrize("dim,physics,dtype,n,stream,order", [
    (3, mg.LAPLACE, F64, 1 << 20, 0, 1), (2, mg.ELASTICITY, F32, 1 << 22, 0, 1), (3, mg.ELASTICITY, F64, 1 << 21, 1, None),
    (3, mg.ELASTICITY, F64, 3 << 20, 1, None), (3, mg.ELASTICITY, F32, 1 << 20, 0, 2), (3, mg.ELASTICITY, F32, 3 << 19, 0, 2)])
def test_rows_far_apart(launches, dim, physics, dtype, n, stream, order):
    rule = mg.RULE_TRI3 if dim == 2 else mg.RULE_TET4
    got, = launches(("residual", dim, physics, rule, N.COEF_QUAD, dtype, n, 0))
    assert got["args"][5] == ("true" if stream else "false") and got["block"] == 256
    assert got["order"] == (got["grid"][0] // 8 if order is None else order)


# shares of a tile's P1 and P2 matrices: no more than 640 waves, streaming at whole
# lines; one share from 640 waves of elements on
@pytest.mark.parametrize("n,share", [(1024, 10), (4096, 10), (10240, 4), (10243, 3), (20480, 2), (40960, 1), (163840, 1)])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_matrix_shares(launches, dtype, n, share):
    got, = launches(("jacobian", 3, mg.ELASTICITY, mg.RULE_TET11, N.COEF_QUAD, dtype, n, 0, 2))
    assert got["grid"] == (_lanes(n, 256), share)
    assert got["args"][4] == ("true" if n % 32 == 0 else "false")


@pytest.mark.parametrize("dim,n,waves", [(3, 1 << 20, 4), (3, 1000000, 1), (2, 1 << 20, 1), (2, 1 << 21, 4)])
def test_p2_matrix_waves(launches, dim, n, waves):
    rule = mg.RULE_TRI6 if dim == 2 else mg.RULE_TET11
    got, = launches(("jacobian", dim, mg.LAPLACE, rule, N.COEF_QUAD, F64, n, 0, 2))
    assert got["block"] == 64 * waves
