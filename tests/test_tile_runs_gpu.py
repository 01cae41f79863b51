"""Runs of tiles on the four-wave kernel: tile loads are prepared in runs that end with the unit, the chunk or the 64 page ids
at hand.  Sequences of several times 64 pages, cut so that a run ends inside a chunk, together with it, in a group block behind
which the next one begins at tile 0 again, and with chunks that begin in the middle of the ids requested on a guess."""
import pytest
import torch

import gpu_util
import oracle
import paper_2505_21487_amd as gla
from paper_2505_21487_amd.harness import DeviceProblem
from workloads import make_problem

pytestmark = pytest.mark.gpu

# kind, heads, groups, d_v, query positions (gla2: one unit per sequence; the others: two)
KERNELS = {
    "gla2": ("gla", 128, 2, 256, 1), "gla4": ("gla", 64, 4, 256, 2), "gla2_T2": ("gla", 96, 2, 256, 2), "mla2": ("gla", 64, 2, 512, 1),
    "gta8": ("gta", 64, 8, 128, 1),
}


@pytest.mark.parametrize("page", [16, 32, 64])
@pytest.mark.parametrize("kernel", sorted(KERNELS))
def test_runs(kernel, page):
    kind, h, g, d_v, T = KERNELS[kernel]
    w = 64 * page  # tokens behind 64 page ids
    # chunks of the longest sequence's tiles, of exactly 64 pages (equal splits), and of neither
    for name, lens, splits in (("ragged", [3 * w, 2 * w + 100, w, w - 31, 5, 0, w + 33], (1, 3, 5)), ("equal", [3 * w] * 3, (1, 3, 4))):
        p = make_problem(f"runs_{kernel}_{name}", kind=kind, seq_lens=lens, T=T, h_q=h, h_c=g, d_v=d_v, page_size=page, seed=8300 + page + h,
                         num_pages=sum((n + page - 1) // page for n in lens) + 64, poison_tail=True)
        assert p.max_pages == 3 * 64
        dp = DeviceProblem(p, poison_unused=True)
        out = torch.empty(p.B, T, h, d_v, dtype=torch.float32, device="cuda")
        prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=torch.empty(p.B, T, h, device="cuda"), workspace=None)
        # a few rows of every group: all of them read the same tiles
        sel = [(b, t, i) for b in range(p.B) for t in range(T) for i in range(b, h, h // g // 2 - 1)]
        ref = oracle.decode_problem(p, sel=sel)
        idx = tuple(zip(*sel))
        for n in splits:
            prm.num_splits = n
            assert gla.gla_decode_kernel_name(prm, kind == "gta", lens) == "four-wave kernel"
            res = gpu_util.run_gpu(p, dp=dp, out_dtype=torch.float32, num_splits=n, impl=gla.GLA_IMPL_TUNED)
            gpu_util.compare(res[0][idx], res[1][idx], *ref, what=f"{kernel}, pages of {page}, {name}, {n} splits", bf16_out_allowance=False)
