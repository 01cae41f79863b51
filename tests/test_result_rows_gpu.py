"""Results as the four-wave kernel stores them: sequences that one chunk holds (written in place, bf16 in 16-byte pieces
or fp32) and such that several share (partials, without the rows that pad a slab of 32), into rows that start on any
multiple of four elements.  What lies between the rows stays as it was."""
import pytest
import torch

import oracle
import paper_2505_21487_amd as gla
from paper_2505_21487_amd.harness import DeviceProblem
from workloads import make_problem

from gpu_util import compare

pytestmark = pytest.mark.gpu

SHAPES = {
    "rows_8_of_32": ("gla", 16, 2, 256, 1), "rows_96_of_128": ("gla", 64, 2, 256, 3), "rows_full": ("gla", 128, 2, 256, 1),
    "mla_rows_40": ("gla", 40, 1, 512, 1), "mla_rows_33": ("gla", 11, 1, 512, 3), "gta": ("gta", 32, 4, 128, 1), "gta_rows_full": ("gta", 32, 4, 128, 4),
}


@pytest.mark.parametrize("pad", [4, 8])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_rows_of_the_result(shape, pad):
    kind, h, g, d_v, T = SHAPES[shape]
    p = make_problem(f"rows_{shape}", kind=kind, seq_lens=[20, 1500, 0, 64, 3, 333], T=T, h_q=h, h_c=g, d_v=d_v, seed=8300 + len(shape),
                     num_pages=128, poison_tail=True)
    ref_out, ref_lse = oracle.decode_problem(p)
    dp = DeviceProblem(p, poison_unused=True)
    fn = gla.gta_decode if kind == "gta" else gla.gla_decode
    for dt in (torch.bfloat16, torch.float32):
        for splits in (0, 1, 5):
            wide = torch.full((p.B, p.T, p.h_q, d_v + pad), 7.0, dtype=dt, device="cuda")
            out, lse = fn(*dp.args(), out=wide[..., :d_v], impl=gla.GLA_IMPL_TUNED, num_splits=splits)
            torch.cuda.synchronize()
            assert (wide[..., d_v:] == 7.0).all()
            compare(out.double().cpu().numpy(), lse.double().cpu().numpy(), ref_out, ref_lse, what=f"{shape} {dt} splits={splits}",
                    bf16_out_allowance=dt == torch.bfloat16)
