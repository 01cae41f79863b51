"""Which projection kernel a call runs and how its sums are cut, from shapes alone (256 compute units): the host code is
compiled by itself."""
import ctypes
import itertools
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
extern "C" int plan(const gla_proj_params* p, int sum_groups, int small, int64_t out[8]) {
  gla::ProjPlan q;
  const int rc = gla::proj_plan(p, sum_groups, 256, small, &q);
  if (rc != GLA_OK) return rc;
  out[0] = q.mt; out[1] = q.nt; out[2] = q.ksplit; out[3] = q.k_per_split; out[4] = q.direct; out[5] = (int64_t)q.part_bytes;
  out[6] = q.placed; out[7] = q.rotated;
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
    out = (ctypes.c_int64 * 8)()
    assert lib.plan(ctypes.byref(p), sum_groups, small, out) == 0
    return dict(zip(("mt", "nt", "ranges", "features", "direct", "bytes", "placed", "rotated"), out))


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
# one of those measured when workgroups had the plain order.  (In the present one 64 rows are faster on 2 x 5120 x 4096 and 3 x
# 1024 x 10752, 32 features per wave with 100 rows of 128 heads x 256 x 128, both by 2 to 14 %, and 64 features per wave with 167 rows
# of 4 x 5120 x 8192 by 4 %.)
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


# ... -> (placed on the XCDs, blocks of features start at different steps): the faster order of those measured
ORDER = {
    # 64 features per wave, long ranges; rows of weights that lie close together
    (64, 2, 5120, 16384, 1): (1, 1), (128, 2, 5120, 8192, 1): (1, 1), (32, 2, 8192, 8192, 1): (1, 1), (16, 1, 5120, 16384, 1): (0, 1),
    (1, 8, 4096, 2048, 0): (1, 1), (16, 1, 16384, 1536, 0): (0, 1), (1, 64, 1024, 1024, 0): (1, 1), (1, 16, 4096, 512, 0): (1, 0),
    (65, 8, 4096, 1024, 1): (1, 0), (17, 64, 1024, 4096, 0): (1, 1), (17, 32, 2048, 8192, 0): (0, 0), (1, 4, 5120, 8192, 1): (0, 1),
    # 32 features per wave and short ranges: more weights than the last-level cache holds
    (64, 1, 128256, 8192, 1): (1, 1), (64, 32, 8192, 2048, 0): (1, 1), (300, 2, 20480, 8192, 1): (1, 1), (1, 1, 128256, 8192, 1): (0, 0),
    (32, 16, 7168, 7168, 0): (0, 0), (64, 16, 8192, 1024, 0): (0, 0),
    # ... than the L2s do between two row tiles
    (129, 1, 128256, 1024, 1): (1, 0), (300, 2, 28672, 1536, 1): (1, 0), (300, 8, 5120, 2048, 0): (0, 0), (65, 64, 16384, 64, 0): (0, 0),
    # ... one row tile, few blocks of features, many, too few workgroups
    (64, 128, 256, 128, 0): (0, 0), (32, 128, 512, 128, 0): (0, 0), (65, 128, 256, 128, 0): (1, 0), (256, 128, 256, 1024, 0): (1, 0),
    (65, 32, 7168, 64, 0): (0, 0), (256, 4, 1024, 2048, 1): (0, 0), (200, 128, 1536, 64, 0): (0, 0), (200, 16, 5120, 128, 0): (0, 0),
    (200, 16, 512, 128, 0): (0, 0), (129, 32, 256, 128, 0): (1, 0), (128, 32, 256, 128, 0): (0, 0), (129, 64, 128, 1024, 0): (1, 0),
    # ... one round of long ranges, few weights, several rounds
    (64, 1, 1024, 16384, 1): (1, 0), (33, 64, 256, 1024, 0): (1, 0), (64, 2, 4096, 1024, 1): (0, 0), (33, 8, 5120, 2048, 0): (0, 0),
}


@pytest.mark.parametrize("shape", sorted(ORDER))
def test_the_faster_order(lib, shape):
    q = plan(lib, *shape)
    assert (q["placed"], q["rotated"]) == ORDER[shape], q


def test_the_kernel_of_one_block_has_the_plain_order(lib):
    """proj_kernel<1, 1> has neither the placement nor the offsets."""
    found = 0
    for rows, groups, n, k in itertools.product((1, 16, 17, 32, 33, 64, 65, 129), (1, 2, 8, 32, 128), (32, 160, 512, 2048, 16384), (64, 192, 512, 1024, 2048, 16384)):
        for sum_groups, small in itertools.product((0, 1), (0, 1, 2)):
            q = plan(lib, rows, groups, n, k, sum_groups, small)
            if (q["mt"], q["nt"]) == (1, 1):
                found += 1
                assert (q["placed"], q["rotated"]) == (0, 0), (rows, groups, n, k, sum_groups, small)
    assert found > 100


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
    for shape, (mt, nt, ranges, steps, last, placed, rotated) in cases.items():
        q = plan(lib, *shape, sum_groups)
        assert (q["mt"], q["nt"], q["ranges"], q["features"] // 64) == (mt, nt, ranges, steps), (shape, q)
        assert shape[3] // 64 - (ranges - 1) * steps == last, shape
        assert (q["placed"], q["rotated"]) == (placed, rotated), (shape, q)
