"""The eight-wave kernel against the oracle at the sizes where it can go wrong: remainders of its 64-token tiles,
many sequences inside one chunk, more than 64 sequences, page-id windows crossed (64 tiles at pages of 8 tokens or
more, 8 tiles below), row blocks that are not full, RoPE keys of fewer than 64 dims, moved references and heavy
weights (peaky softmax).  Every batch holds one sequence long enough for the library to take that kernel."""
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
    "mla_edges": ("mla", EDGES + [17000], 1, 64, {}),
    "mla_peaky": ("mla", EDGES + [18001], 1, 16, dict(q_gain=6.0)),
    "mla_rows33": ("mla", [300, 65, 31, 0, 128, 9100], 3, 32, dict(h_q=11)),
    "mla_windows_page8": ("mla", [5000, 4097, 64], 1, 8, {}),
    "mla_windows_page1": ("mla", [1100, 2513, 70], 2, 1, {}),
    "mla_page4_rope32": ("mla", [700, 1930, 9], 1, 4, dict(d_r=32)),
    "mla_many": ("mla", [17] * 12 + [0, 200, 64, 23000], 1, 64, {}),
    "mla_many_page8": ("mla", [17] * 70 + [0, 20100, 64], 1, 8, dict(h_q=64)),
    "gla_edges_page8": ("gla", EDGES + [10000], 4, 8, {}),
    "gla_edges": ("gla", EDGES + [32100], 3, 64, dict(h_q=96)),
    "gla_peaky_page2": ("gla", [900, 77, 4300], 3, 2, dict(q_gain=6.0)),
    "gla_long": ("gla", [19000, 8100], 4, 64, {}),
    "gla_rope48_page1": ("gla", [640, 1, 63, 5000], 4, 1, dict(d_r=48)),
    "gla_many_page4": ("gla", [5] * 66 + [129, 0, 3, 32000], 3, 4, dict(h_q=96)),
}


def _problem(name, lens, **kw):
    page = kw["page_size"]
    return make_problem(name, seq_lens=lens, num_pages=sum((n + page - 1) // page for n in lens) + 64, poison_tail=True, **kw)


def _kernel(p, num_splits=0):
    dp = DeviceProblem(p)
    out = torch.empty(p.B, p.T, p.h_q, p.d_v, dtype=torch.float32, device="cuda")
    prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=torch.empty(p.B, p.T, p.h_q, device="cuda"), workspace=None, num_splits=num_splits)
    return gla.gla_decode_kernel_name(prm, 0, p.seq_lens)


@pytest.mark.parametrize("name", sorted(CASES))
def test_eight_wave_kernel(name):
    shape, lens, T, page, kw = CASES[name]
    kw = dict(kw)
    p = _problem(name, lens, T=T, h_q=kw.pop("h_q", 128), h_c=1 if shape == "mla" else 2, d_v=512 if shape == "mla" else 256,
                 page_size=page, seed=7000 + len(name), **kw)
    # few chunks per sequence: several sequences in one, and sequences over several
    for splits in (1, 2):
        assert _kernel(p, splits) == "eight-wave kernel"
        check_problem(p, impl=gla.GLA_IMPL_TUNED, num_splits=splits, what=f"{name} splits={splits}")
    # short chunks: the four-wave kernel, launched alone
    assert _kernel(p, p.max_pages if page > 1 else 400) == "four-wave kernel"


@pytest.mark.parametrize("shape,lens,T,page,h_q", [("mla", [4000, 3900, 2100] * 20 + [0, 77], 1, 64, 128), ("mla", [2600] * 16 + [0, 77], 1, 4, 128),
                                                  ("gla", [2900] * 32 + [0, 77], 3, 8, 96)])
def test_automatic_chunks(shape, lens, T, page, h_q):
    """The library's own cut, on lists on either side of the line between the two kernels (all rows of some sequences)."""
    for keep, want in ((len(lens), "eight-wave kernel"), (4, "four-wave kernel")):
        p = _problem("auto", lens[-keep:], T=T, h_q=h_q, h_c=1 if shape == "mla" else 2, d_v=512 if shape == "mla" else 256, page_size=page,
                     seed=7100 + page, extra_table_cols=131072 // page)
        assert _kernel(p) == want
        sel = [(b, t, h) for b in (0, p.B // 2, p.B - 3, p.B - 2, p.B - 1) for t in range(T) for h in range(0, h_q, 3)]
        check_problem(p, sel=sel, impl=gla.GLA_IMPL_TUNED, what=f"{shape} {want}")


def test_captured_call_chooses_again_for_other_lengths():
    """Replays of one captured call, the lengths changed in place between them: each takes the kernel of its lengths."""
    p = _problem("graph", [4000, 3900, 2100] * 20 + [0, 77], T=1, h_q=128, h_c=1, d_v=512, page_size=64, seed=72)
    dp = DeviceProblem(p, poison_unused=True)
    out = torch.empty(p.B, p.T, p.h_q, p.d_v, dtype=torch.float32, device="cuda")
    lse = torch.empty(p.B, p.T, p.h_q, device="cuda")
    prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=lse, workspace=None)
    ws = torch.full((gla.gla_decode_workspace_size(prm),), 0xFF, dtype=torch.uint8, device="cuda")
    prm.workspace, prm.workspace_bytes = ws.data_ptr(), ws.numel()
    gla.decode_prepared(prm)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        prm.stream = torch.cuda.current_stream().cuda_stream
        gla.decode_prepared(prm)
    full = dp.seq_lens.clone()
    for lens, kernel in ((full, "eight-wave kernel"), (full.clamp(max=150), "four-wave kernel"), (full, "eight-wave kernel"), (full // 7, "four-wave kernel")):
        assert gla.gla_decode_kernel_name(prm, 0, lens.tolist()) == kernel
        dp.seq_lens.copy_(lens)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone(), lse.clone()
        want = gla.gla_decode(*dp.args(), out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_eight_wave_kernel_repeats_bit_for_bit():
    """Many segments, moved references and residual passes: the same call gives the same bits."""
    p = _problem("repeat", [70, 300, 64, 1, 513] * 4 + [30000], T=1, h_q=128, h_c=1, d_v=512, page_size=64, seed=71, q_gain=3.0)
    assert _kernel(p, 1) == "eight-wave kernel"
    dp = DeviceProblem(p, poison_unused=True)
    first = None
    for _ in range(20):
        out, lse = gla.gla_decode(*dp.args(), out_dtype=torch.float32, num_splits=1)
        torch.cuda.synchronize()
        if first is None:
            first = (out.clone(), lse.clone())
        assert torch.equal(out, first[0]) and torch.equal(lse, first[1])
    assert np.isfinite(out.cpu().numpy()).all()
