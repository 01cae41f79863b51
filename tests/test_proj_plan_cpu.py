"""Which projection kernel a call runs and how its sums are cut, from shapes alone (256 compute units): the host code is
compiled by itself."""
import ctypes
import math
import os
import random
import subprocess

import pytest

from paper_2505_21487_amd.binding import GlaProjParams

from test_proj_placement_gpu import ABSORB as PLACED_ABSORB, OUTPUT_PROJ

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_21487_amd", "csrc")
SOURCE = r"""
#include "proj_plan.hpp"
extern "C" int plan(const gla_proj_params* p, int sum_groups, int small, int64_t out[6]) {
  gla::ProjPlan q;
  const int rc = gla::proj_plan(p, sum_groups, 256, small, &q);
  if (rc != GLA_OK) return rc;
  out[0] = q.mt; out[1] = q.nt; out[2] = q.ksplit; out[3] = q.k_per_split; out[4] = q.direct; out[5] = (int64_t)q.part_bytes;
  return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("proj_plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "plan.so"), str(d / "plan.cpp")])
    return ctypes.CDLL(str(d / "plan.so"))


def plan(lib, rows, groups, n, k, sum_groups, small=0):
    p = GlaProjParams()
    p.rows, p.groups, p.n, p.k = rows, groups, n, k
    p.a_row_stride, p.a_group_stride, p.c_row_stride, p.c_group_stride = groups * k, k, groups * n, n
    out = (ctypes.c_int64 * 6)()
    assert lib.plan(ctypes.byref(p), sum_groups, small, out) == 0
    return dict(zip(("mt", "nt", "ranges", "features", "direct", "bytes"), out))


def rows_computed(q, rows):
    tile = 32 * q["mt"]
    return (rows + tile - 1) // tile * tile


ABSORB = [(heads, n, k) for heads in (16, 32, 64, 128) for n in (128, 256, 512) for k in (64, 128, 192, 512)]


@pytest.mark.parametrize("heads,n,k", ABSORB)
def test_absorbed_query_computes_few_rows_for_padding(lib, heads, n, k):
    """Sums of one range: 128 rows per workgroup only where 64 would compute about as many, and up to 256 rows."""
    for rows in range(1, 600, 7):
        q = plan(lib, rows, heads, n, k, 0)
        assert q["ranges"] == 1 and q["direct"] and q["bytes"] == 0
        assert rows_computed(q, rows) <= 1.12 * max(32, (rows + 63) // 64 * 64) and (q["mt"] < 4 or 64 < rows <= 256)


# (rows, groups, output features, input features, summed over the groups) -> (32-row blocks, 32-feature blocks): the faster
# one of those measured
FASTER = {
    (100, 128, 256, 128, 0): (2, 2), (129, 128, 256, 128, 0): (2, 1), (200, 128, 256, 128, 0): (4, 2), (256, 128, 256, 128, 0): (4, 2),
    (100, 128, 512, 128, 0): (4, 2), (129, 128, 512, 128, 0): (2, 1), (100, 64, 512, 128, 0): (2, 1), (129, 64, 512, 128, 0): (2, 1),
    (256, 64, 512, 128, 0): (4, 2), (300, 32, 512, 128, 0): (2, 1), (100, 64, 256, 128, 0): (2, 1), (200, 128, 128, 128, 0): (2, 1),
    (64, 2, 5120, 16384, 1): (2, 2), (100, 2, 5120, 16384, 1): (4, 2), (65, 2, 5120, 4096, 1): (4, 2), (100, 2, 2048, 8192, 1): (2, 2),
    (65, 3, 1024, 10752, 1): (4, 2), (100, 1, 2048, 8192, 1): (2, 1), (129, 1, 5120, 4096, 1): (2, 1), (256, 1, 5120, 4096, 1): (2, 2),
    (129, 2, 5120, 8192, 1): (2, 2), (256, 2, 5120, 8192, 1): (4, 2), (129, 2, 8192, 8192, 1): (4, 2), (167, 4, 5120, 8192, 1): (2, 1),
    (129, 2, 2048, 8192, 1): (2, 2), (384, 1, 2048, 8192, 1): (2, 2),
}


@pytest.mark.parametrize("shape", sorted(FASTER))
def test_the_faster_kernel(lib, shape):
    q = plan(lib, *shape)
    assert (q["mt"], q["nt"]) == FASTER[shape], q


def test_ranges_cover_the_sum(lib):
    for rows in (1, 33, 65, 100, 129, 200, 300, 500):
        for groups, n, k in ((1, 32, 64), (2, 5120, 16384), (1, 5120, 4160), (3, 1056, 12352), (4, 4096, 8192), (1, 96, 65536), (128, 512, 128)):
            for sum_groups in (0, 1):
                for small in (0, 1, 2):
                    q = plan(lib, rows, groups, n, k, sum_groups, small)
                    assert (q["ranges"] - 1) * q["features"] < k <= q["ranges"] * q["features"] and q["features"] % 64 == 0
                    assert small == 0 or q["mt"] <= 2


def test_a_list_of_workgroups_fits_one_dimension_of_a_launch(lib):
    """The projections' grids have one dimension: fewer than 2^32 threads, 2^24 workgroups.  Sums of 2^30 features and more
    than 2^20 rows or output features are no calls anyone makes, but the plan takes them."""
    rng = random.Random(5)
    longest = 0
    for i in range(60000):
        rows = min(17 + int(2 ** rng.uniform(0, 20)), 64 * 65535)
        n, k = 32 * int(2 ** rng.uniform(0, 20)), 64 * int(2 ** rng.uniform(0, 24))
        most = min(0x7fffffff // (rows * n), 65535)
        if most < 1:
            continue
        groups = most if i % 2 else int(2 ** rng.uniform(0, math.log2(most)))
        q = plan(lib, rows, groups, n, k, i % 3 % 2)
        blocks, tiles, slices = -(-n // (128 * q["nt"])), -(-rows // (32 * q["mt"])), groups * q["ranges"]
        if q["mt"] * q["nt"] > 1 and tiles <= 65535 and slices <= 65535:
            longest = max(longest, blocks * tiles * slices)
    assert 2 ** 20 < longest < 2 ** 24, longest


@pytest.mark.parametrize("sum_groups,cases", [(1, OUTPUT_PROJ), (0, PLACED_ABSORB)])
def test_the_placement_tests_reach_what_they_are_for(lib, sum_groups, cases):
    for shape, (mt, nt, ranges, steps, last) in cases.items():
        q = plan(lib, *shape, sum_groups)
        assert (q["mt"], q["nt"], q["ranges"], q["features"] // 64) == (mt, nt, ranges, steps), (shape, q)
        assert shape[3] // 64 - (ranges - 1) * steps == last, shape
