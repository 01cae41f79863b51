"""Which workgroup of the projections works on what: the order of the steps of a range, which starts elsewhere for every block
of output features, and the placement of workgroups on the XCDs.  Which calls have which: proj_plan."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_21487_amd as gla
from workloads import bf16_bits, projection_weights

from test_proj_gpu import check_projection

pytestmark = pytest.mark.gpu


# What a call's plan makes of it at 256 compute units, held on the CPU in test_proj_plan_cpu.py.
# (rows, groups, output features, input features) -> 32-row and 32-feature blocks, ranges, steps of a range and of the last one,
# placed, blocks start at different steps
OUTPUT_PROJ = {
    # few blocks of features, grids that do not divide by eight, ranges of an odd number of steps, a last block of 32 features
    (16, 1, 10400, 3136): (1, 2, 6, 9, 4, 0, 1), (17, 1, 10400, 3136): (1, 2, 6, 9, 4, 1, 1), (65, 1, 10400, 3136): (4, 2, 6, 9, 4, 1, 1),
    (16, 3, 1312, 6208): (1, 2, 11, 9, 7, 0, 1), (17, 3, 1312, 6208): (1, 2, 11, 9, 7, 1, 1), (65, 3, 1312, 6208): (4, 2, 11, 9, 7, 1, 1),
    # variants and shapes without either
    (16, 2, 4128, 1600): (1, 1, 1, 25, 25, 0, 0), (17, 2, 4128, 1600): (1, 1, 1, 25, 25, 0, 0), (65, 2, 4128, 1600): (2, 1, 1, 25, 25, 0, 0),
    # a last range of fewer steps than the ring has stages (three with 64 features per wave)
    (16, 3, 1088, 6976): (1, 2, 13, 9, 1, 0, 1), (17, 3, 832, 9280): (1, 2, 17, 9, 1, 1, 1), (33, 3, 1312, 5824): (2, 2, 11, 9, 1, 1, 1),
    (65, 2, 1088, 8512): (2, 2, 12, 12, 1, 1, 1), (100, 2, 1152, 8576): (2, 2, 12, 12, 2, 1, 1), (100, 3, 1056, 6976): (4, 2, 13, 9, 1, 1, 1),
    # placed, in plain order: more weights between two row tiles than the L2s hold
    (200, 1, 33056, 1024): (2, 1, 1, 16, 16, 1, 0),
}
ABSORB = {
    (33, 77, 160, 64): (2, 1, 1, 1, 1, 0, 0), (65, 13, 544, 192): (2, 1, 1, 3, 3, 0, 0), (17, 21, 288, 2048): (1, 1, 4, 8, 8, 0, 0),
    (33, 77, 160, 128): (2, 1, 1, 2, 2, 0, 0), (66, 33000, 32, 64): (2, 1, 1, 1, 1, 1, 0), (34, 33000, 160, 128): (2, 1, 1, 2, 2, 0, 0),
    # placed, in plain order
    (40, 13, 3872, 576): (2, 2, 1, 9, 9, 1, 0), (65, 11, 2592, 1024): (4, 2, 2, 8, 8, 1, 0), (40, 64, 256, 1024): (2, 1, 2, 8, 8, 1, 0),
    (65, 67, 160, 1024): (2, 1, 2, 8, 8, 1, 0),
    (130, 33, 288, 128): (2, 1, 1, 2, 2, 1, 0), (65, 33000, 160, 64): (2, 1, 1, 1, 1, 1, 0),
    # both, groups that keep their own results; few rows, two ranges; 32 features per wave
    (5, 11, 2080, 2112): (1, 2, 2, 17, 16, 1, 1), (70, 36, 1856, 2112): (2, 1, 1, 33, 33, 1, 1),
}


@pytest.mark.parametrize("M,G,N,K", sorted(OUTPUT_PROJ))
def test_output_proj(M, G, N, K):
    g = torch.Generator().manual_seed(840 + M + G)
    a = (torch.randn(M, G, K, generator=g) * 0.05).to(torch.bfloat16)
    w = projection_weights(G, N, K, seed=841 + M)
    ref = oracle.project(bf16_bits(a), bf16_bits(w), sum_groups=True)
    abs_prod = sum(np.abs(a[:, i].double().numpy()) @ np.abs(w[i].double().numpy()).T for i in range(G))
    c = gla.gla_output_proj(a.cuda(), w.cuda(), out_dtype=torch.float32)
    torch.cuda.synchronize()
    check_projection(c.double().cpu().numpy(), ref, abs_prod, bf16_out=False, what=f"out-proj {M}x{G}x{N}x{K}")


@pytest.mark.parametrize("M,G,N,K", sorted(ABSORB))
def test_absorb_query(M, G, N, K):
    """33000 groups: more than 2^16 workgroups, with one block of features and with two, where the kernel divides by both."""
    gen = torch.Generator(device="cuda").manual_seed(850 + M)
    a = torch.randn(M, G, K, generator=gen, device="cuda", dtype=torch.bfloat16)
    w = (torch.randn(G, N, K, generator=gen, device="cuda", dtype=torch.bfloat16) / K ** 0.5).to(torch.bfloat16)
    c = torch.full((M, G, N), float("nan"), device="cuda")  # (a result that no workgroup wrote shows)
    gla.gla_absorb_query(a, w, out=c)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(c).all())
    some = sorted({0, 1, G // 3, G // 2, G - 2, G - 1, *range(0, G, max(1, G // 50))})
    a, w, c = a[:, some].cpu(), w[some].cpu(), c[:, some].double().cpu().numpy()
    ref = oracle.project(bf16_bits(a), bf16_bits(w), sum_groups=False)
    abs_prod = np.einsum("mgk,gnk->mgn", np.abs(a.double().numpy()), np.abs(w.double().numpy()))
    check_projection(c, ref, abs_prod, bf16_out=False, what=f"absorb {M}x{G}x{N}x{K}")


def test_on_the_current_stream():
    """On a stream of its own, behind work that takes a while, and captured: the input is what that stream has made of it."""
    gen = torch.Generator(device="cuda").manual_seed(860)
    a = torch.randn(24, 16, 128, generator=gen, device="cuda", dtype=torch.bfloat16)
    w = torch.randn(16, 256, 128, generator=gen, device="cuda", dtype=torch.bfloat16)
    want = gla.gla_absorb_query(a, w)
    other, ws = torch.zeros_like(a), torch.empty(256, dtype=torch.uint8, device="cuda")
    got = torch.empty_like(want)
    big = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(4):
            big = big @ big * 1e-4
        other.copy_(a)
        gla.gla_absorb_query(other, w, out=got, workspace=ws)
    side.synchronize()
    assert torch.equal(got, want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gla.gla_absorb_query(other, w, out=got, workspace=ws)
    for scale in (1.0, 2.0):  # (a power of two: exact)
        other.copy_(a * scale)
        got.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got.float(), want.float() * scale)
