"""The merge of partial results against the oracle: lists of one chunk to hundreds, every way a unit's blocks are spread over
workgroups (by the mean length of the lists, and further by windows of chunks inside a long one), empty sequences and
chunks without a visible key among them.  Chunks of one tile: the lists are as long as the sequences have tiles."""
import pytest

import paper_2505_21487_amd as gla
from workloads import make_problem

from gpu_util import check_problem

pytestmark = pytest.mark.gpu

SHAPES = {"gla2": ("gla", 128, 2, 256), "gla2_h16": ("gla", 16, 2, 256), "gla1": ("gla", 20, 1, 256), "mla": ("gla", 72, 1, 512),
          "gta4": ("gta", 32, 4, 128), "gta1": ("gta", 8, 1, 128)}
LISTS = {  # tiles per sequence
    "one_of_130": [130],                          # sixteen sets; sixteen waves per block
    "one_of_20": [20],
    "mixed": [40, 0, 17, 8, 3, 1, 9, 2],          # windows inside the longer lists
    "long_among_short": [2] * 30 + [97] + [1] * 10,
    "many": [5, 1, 0, 3] * 40,
}


@pytest.mark.parametrize("T", [1, 4])
@pytest.mark.parametrize("lists", sorted(LISTS))
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_merge(shape, lists, T):
    kind, h, g, d_v = SHAPES[shape]
    lens = [max(0, 32 * n - (5 * i) % 32) for i, n in enumerate(LISTS[lists])]
    p = make_problem(f"merge_{shape}_{lists}", kind=kind, seq_lens=lens, T=T, h_q=h, h_c=g, d_v=d_v, seed=8500 + len(lens) + T,
                     num_pages=sum((n + 63) // 64 for n in lens) + 64, poison_tail=True)
    for splits in (2 * p.max_pages, 0):
        check_problem(p, impl=gla.GLA_IMPL_TUNED, num_splits=splits, what=f"{shape} {lists} splits={splits}")
