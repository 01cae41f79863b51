"""What a call does with the workspace it is given: one sized for a larger batch serves every smaller one, and one that
is too small for the plan a call would get still serves the plan with fewer chunks."""
import pytest
import torch

import paper_2505_21487_amd as gla
from paper_2505_21487_amd.harness import DeviceProblem
from workloads import make_problem

from gpu_util import check_problem

pytestmark = pytest.mark.gpu

SHAPES = {
    "gla2": dict(kind="gla", h_q=32, h_c=2, d_v=256), "mla": dict(kind="gla", h_q=64, h_c=1, d_v=512),
    "gta4_d128": dict(kind="gta", h_q=32, h_c=4, d_v=128), "gta4_d64": dict(kind="gta", h_q=32, h_c=4, d_v=64, d_r=32),
    "generic": dict(kind="gla", h_q=32, h_c=2, d_v=256, page_size=128),
}
LENS = [250, 1, 64, 200, 131, 0, 33, 256]


def problem(shape, batch):
    return make_problem(f"ws_{shape}_{batch}", seq_lens=LENS[:batch], num_pages=64, seed=9000 + batch, poison_tail=True,
                        extra_table_cols=4 - (max(LENS[:batch]) + 63) // 64 if shape != "generic" else 0, **SHAPES[shape])


def need_of(p):
    dp = DeviceProblem(p)
    out = torch.empty(p.B, p.T, p.h_q, p.d_v, dtype=torch.float32, device="cuda")
    lse = torch.empty(p.B, p.T, p.h_q, dtype=torch.float32, device="cuda")
    return gla.gla_decode_workspace_size(gla.make_params(*dp.args()[:6], p.scale, out=out, lse=lse, workspace=None), p.kind == "gta")


@pytest.mark.parametrize("shape", [s for s in sorted(SHAPES) if s != "generic"])
def test_workspace_of_the_largest_batch(shape):
    ws = torch.full((need_of(problem(shape, len(LENS))),), 0xFF, dtype=torch.uint8, device="cuda")
    for batch in range(len(LENS), 0, -1):
        check_problem(problem(shape, batch), workspace=ws, what=f"{shape} batch {batch}")


@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_smaller_workspace(shape):
    p = problem(shape, 2)
    need = need_of(p)
    for size in (need // 2, need // 2 + 256):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        check_problem(p, workspace=ws, what=f"{shape} with {size} of {need} bytes")
    with pytest.raises(gla.GlaError) as e:
        check_problem(p, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == gla.GLA_ERR_WORKSPACE_TOO_SMALL
