"""The eight-wave kernel against the oracle at the sizes where it can go wrong: remainders of its 64-token tiles,
many sequences inside one chunk, more than 64 sequences, page-id windows crossed (64 tiles at pages of 8 tokens or
more, 8 tiles below), row blocks that are not full, RoPE keys of fewer than 64 dims, moved references and heavy
weights (peaky softmax).  Tables are long enough that the plan takes that kernel."""
import numpy as np
import pytest
import torch

import paper_2505_21487_amd as gla
from paper_2505_21487_amd.harness import DeviceProblem
from workloads import make_problem

from gpu_util import check_problem

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 63, 64, 65, 127, 129, 700, 2, 4]
CASES = {
    # name: (shape, lengths, T, page, other)
    "mla_edges": ("mla", EDGES, 1, 64, {}),
    "mla_peaky": ("mla", EDGES + [1500], 1, 16, dict(q_gain=6.0)),
    "mla_rows33": ("mla", [300, 65, 31, 0, 128], 3, 32, dict(h_q=11)),
    "mla_windows_page8": ("mla", [5000, 4097, 64], 1, 8, {}),
    "mla_windows_page1": ("mla", [1100, 513, 70], 2, 1, {}),
    "mla_page4_rope32": ("mla", [700, 130, 9], 1, 4, dict(d_r=32)),
    "mla_many": ("mla", [17] * 70 + [0, 200, 64], 1, 64, {}),
    "gla_edges_page8": ("gla", EDGES, 4, 8, {}),
    "gla_peaky_page2": ("gla", [900, 77, 300], 3, 2, dict(q_gain=6.0)),
    "gla_long": ("gla", [9000, 4100], 4, 64, {}),
    "gla_rope48_page1": ("gla", [640, 1, 63], 4, 1, dict(d_r=48)),
    "gla_many_page4": ("gla", [5] * 66 + [129, 0, 3], 3, 4, {}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_eight_wave_kernel(name):
    shape, lens, T, page, kw = CASES[name]
    kw = dict(kw)
    h_q = kw.pop("h_q", 128)
    # (a row length for which the plan picks the kernel: chunks of at least 24 / 192 / 64 tiles if every row were full)
    want_tokens = ((24 if page < 16 else 192) if shape == "mla" else 64) * 64 * 256 // len(lens) + 64
    pages = max((n + page - 1) // page for n in lens)
    p = make_problem(name, seq_lens=lens, T=T, h_q=h_q, h_c=1 if shape == "mla" else 2, d_v=512 if shape == "mla" else 256,
                     page_size=page, seed=7000 + len(name), num_pages=sum((n + page - 1) // page for n in lens) + 64,
                     poison_tail=True, extra_table_cols=max(1, want_tokens // page - pages), **kw)
    for splits in (0, 3):
        check_problem(p, impl=gla.GLA_IMPL_TUNED, num_splits=splits, what=f"{name} splits={splits}")
    check_problem(p, impl=gla.GLA_IMPL_TUNED, num_splits=p.max_pages, what=f"{name} one tile per chunk or little more")


def test_eight_wave_kernel_repeats_bit_for_bit():
    """Many segments, moved references and residual passes: the same call gives the same bits."""
    p = make_problem("repeat", seq_lens=[70, 300, 64, 1, 513] * 8, T=1, h_q=128, h_c=1, d_v=512, page_size=64, seed=71,
                     num_pages=4096, q_gain=3.0, poison_tail=True, extra_table_cols=1300)
    dp = DeviceProblem(p, poison_unused=True)
    first = None
    for _ in range(20):
        out, lse = gla.gla_decode(*dp.args(), out_dtype=torch.float32)
        torch.cuda.synchronize()
        if first is None:
            first = (out.clone(), lse.clone())
        assert torch.equal(out, first[0]) and torch.equal(lse, first[1])
    assert np.isfinite(out.cpu().numpy()).all()
