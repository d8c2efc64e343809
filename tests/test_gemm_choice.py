"""The list of launches that a GEMM is carried out by (csrc/gemm_choice.h, plain C++), checked on the CPU over the sizes:
the parts tile the matrix, and rows that share a column are summed over k in one order."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_30010_amd", "csrc")
IN_ORDER = {0, 1, 5, 6}          # one accumulator, k ascending; 2, 3 and 4 add up 4, 2 (of an odd number of k-tiles 4) and 2 shares of k

SHIM = """
#include "gemm_choice.h"
extern "C" int plan(int rows, int cols, int K, int cus, int rows_splittable, int one_tile, int residual, int *out) {
  const et::GemmPlan p = et::plan_gemm(et::GemmRules{K, cus, rows_splittable != 0, one_tile != 0, residual != 0}, rows, cols);
  for (int i = 0; i < p.n; ++i) {
    const et::GemmPart &t = p.part[i];
    const int v[5] = {t.row0, t.rows, t.col0, t.cols, t.cfg};
    for (int j = 0; j < 5; ++j) out[5 * i + j] = v[j];
  }
  return p.n;
}
extern "C" double cost(int cfg, int rows, int cols, int K) { return et::gemm_cost(cfg, rows, cols, K); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("gemm_choice")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    shim = C.CDLL(lib)
    shim.cost.restype = C.c_double
    return shim


@pytest.fixture(scope="module")
def plan(shim):
    fn = shim.plan
    buf = (C.c_int * 80)()

    def call(rows, cols, K, rows_splittable=True, one_tile=False, cus=256, residual=False):
        n = fn(rows, cols, K, cus, int(rows_splittable), int(one_tile), int(residual), buf)
        assert 1 <= n <= 16
        return [tuple(buf[5 * i:5 * i + 5]) for i in range(n)]
    return call


def _sizes():
    for tokens, mats in ((729, ((3456, 1152), (4352, 1152), (1152, 1152), (1152, 4352), (1152, 640))),
                         (196, ((2304, 768), (3072, 768), (768, 768), (768, 3072))), (64, ((192, 64), (256, 64), (64, 256)))):
        for frames in range(1, 65):
            for keep in (1.0, 0.5, 0.3):
                for cols, K in mats:
                    yield frames * max(1, int(tokens * keep)), cols, K
    rng = random.Random(4)
    for _ in range(4000):
        yield int(2 ** rng.uniform(0, 18)), 8 * int(2 ** rng.uniform(0, 13)), 64 * int(2 ** rng.uniform(0, 8))


@pytest.mark.parametrize("residual", [False, True])
def test_parts_tile_the_matrix_and_keep_one_order_over_its_rows(plan, residual):
    split = 0
    for rows, cols, K in _sizes():
        for rows_splittable in (True, False):
            parts = plan(rows, cols, K, rows_splittable, residual=residual)
            assert sum(n * c for _, n, _, c, _ in parts) == rows * cols, (rows, cols, K, parts)
            for i, (r0, n, c0, c, cfg) in enumerate(parts):
                assert n > 0 and c > 0 and 0 <= r0 and r0 + n <= rows and 0 <= c0 and c0 + c <= cols
                assert c0 % 64 == 0 and 0 <= cfg <= 6
                for r1, n1, c1, m1, _ in parts[:i]:
                    assert r1 + n1 <= r0 or r0 + n <= r1 or c1 + m1 <= c0 or c0 + c <= c1, (rows, cols, K, parts)
                assert n == rows or (rows_splittable and cfg in IN_ORDER), (rows, cols, K, parts)
                split += n < rows
    assert split > 300           # (the sizes do reach launches over some of the rows)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("cus", [32, 64, 128, 256])
def test_launches_with_row_statistics_walk_one_tile_per_workgroup(plan, cus, residual):
    """The persistent kernel takes row statistics only where each workgroup has one tile (one 256 x 256 or two 128 x 128
    per compute unit); it refuses the call otherwise, so on no device, whole or partitioned, may it be chosen there."""
    for rows, cols, K in _sizes():
        (_, _, _, _, cfg), = plan(rows, cols, K, one_tile=True, cus=cus, residual=residual)
        assert cfg != 0 or -(-rows // 256) * -(-cols // 256) <= cus, (rows, cols, K)
        assert cfg != 1 or -(-rows // 128) * -(-cols // 128) <= 2 * cus, (rows, cols, K)


def test_an_odd_number_of_k_tiles_is_rated_by_its_own_kernel(plan, shim):
    """128 x 64 tiles run another kernel where K / 64 is odd, which takes longer than the other one's next larger K (256
    workgroups, 5 to 19 k-tiles: 7.2, 6.8, 7.8, 7.2, .., 11.0, 10.1, 11.5 us)."""
    for kt in range(5, 18, 2):
        assert shim.cost(3, 2048, 1024, 64 * kt) > shim.cost(3, 2048, 1024, 64 * (kt + 1)), kt
    assert [p[4] for p in plan(1261, 3264, 1088)] == [5]              # 17.2 us; as 128 x 64 tiles 18.6
    assert [p[4] for p in plan(2787, 1472, 1472, residual=True)] == [5]   # 22.7; 23.9


def test_short_contractions_of_several_rounds_run_on_the_persistent_kernel(plan):
    """256 x 128 tiles fetch and finish anew in each round, which short k-loops do not hide (us per launch, that tiling / the
    persistent kernel): 23709 x 1344, 7 k-tiles, 43.4 / 34.3; 15395 x 1536, 8, 34.7 / 29.8; 13409 x 1152, 6, 21.1 / 17.8."""
    for rows, cols, K in ((23709, 1344, 448), (15395, 1536, 512), (13409, 1152, 384), (16057, 1344, 448)):
        assert {p[4] for p in plan(rows, cols, K)} <= {0, 1}, (rows, cols, K)
