"""Which workgroup of the projections works on what: the order of the steps of a range, which starts elsewhere for every block
of output features, and the placement of workgroups on the XCDs, which begins at 17 rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_21487_amd as gla
from workloads import bf16_bits, projection_weights

from test_proj_gpu import check_projection

pytestmark = pytest.mark.gpu


# (rows, groups, output features, input features): 41 blocks or fewer of features, grids that do not divide by eight, ranges of
# fewer steps than the ring has stages and of an odd number of them, a last block of 32 features
@pytest.mark.parametrize("M", [16, 17, 65])
@pytest.mark.parametrize("G,N,K", [(1, 10400, 3136), (3, 1312, 6208), (2, 4128, 1600)])
def test_output_proj(M, G, N, K):
    g = torch.Generator().manual_seed(840 + M + G)
    a = (torch.randn(M, G, K, generator=g) * 0.05).to(torch.bfloat16)
    w = projection_weights(G, N, K, seed=841 + M)
    ref = oracle.project(bf16_bits(a), bf16_bits(w), sum_groups=True)
    abs_prod = sum(np.abs(a[:, i].double().numpy()) @ np.abs(w[i].double().numpy()).T for i in range(G))
    c = gla.gla_output_proj(a.cuda(), w.cuda(), out_dtype=torch.float32)
    torch.cuda.synchronize()
    check_projection(c.double().cpu().numpy(), ref, abs_prod, bf16_out=False, what=f"out-proj {M}x{G}x{N}x{K}")


@pytest.mark.parametrize("M,G,N,K", [(33, 77, 160, 64), (65, 13, 544, 192), (17, 21, 288, 2048), (66, 33000, 32, 64)])
def test_absorb_query(M, G, N, K):
    """The last has more than 2^16 workgroups."""
    gen = torch.Generator(device="cuda").manual_seed(850 + M)
    a = torch.randn(M, G, K, generator=gen, device="cuda", dtype=torch.bfloat16)
    w = (torch.randn(G, N, K, generator=gen, device="cuda", dtype=torch.bfloat16) / K ** 0.5).to(torch.bfloat16)
    c = gla.gla_absorb_query(a, w, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(c).all())
    some = sorted({0, 1, G // 3, G // 2, G - 2, G - 1})
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
