"""Workspace sizes (host only): a program may size its workspace once, for its largest batch, and keep it as requests
come and go."""
import pytest

import paper_2505_21487_amd as gla

# mode, heads, groups, d_v, d_rope: every shape with an MFMA kernel of its own
SHAPES = {
    "gla2": (0, 128, 2, 256, 64), "gla2_h16": (0, 16, 2, 256, 64), "mla": (0, 128, 1, 512, 64), "mla_h40": (0, 40, 1, 512, 64),
    "gla4_d128": (0, 32, 4, 128, 32), "gta4_d128": (1, 32, 4, 128, 64), "gta4_d96": (1, 24, 4, 96, 48),
    "gta4_d64": (1, 32, 4, 64, 32), "gqa4_d128": (2, 32, 4, 128, 0), "gqa8_d64": (2, 16, 8, 64, 0),
}


def params(shape, *, batch, q_len, page, tokens, impl=gla.GLA_IMPL_AUTO):
    mode, h, g, d_v, d_r = SHAPES[shape] if isinstance(shape, str) else shape
    d_n = d_v // 2 if mode == 1 else d_v
    p = gla.shape_params(batch=batch, q_len=q_len, num_q_heads=h, num_groups=g, d_v=d_v, d_nope=d_n, d_rope=d_r, page_size=page,
                         max_pages_per_seq=max(1, tokens // page), num_pages=10**6, impl=impl)
    p.state_stride[:] = (g * page * d_v, page * d_v, d_v)
    p.rope_stride[:] = (page * d_r, d_r)
    p.q_nope_stride[:] = (q_len * h * d_n, h * d_n, d_n)
    p.q_rope_stride[:] = (q_len * h * d_r, h * d_r, d_r)
    p.out_stride[:] = (q_len * h * d_v, h * d_v, d_v)
    p.softmax_scale = 0.05
    return p, mode


@pytest.mark.parametrize("q_len", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_a_larger_batch_never_needs_less(shape, q_len):
    for page in (64, 16, 1):
        for tokens in (64, 200, 256, 1000, 4096, 16384, 131072):
            last = 0
            for batch in (1, 2, 3, 4, 5, 6, 8, 12, 16, 24, 32, 33, 48, 64, 96, 128, 300):
                p, mode = params(shape, batch=batch, q_len=q_len, page=page, tokens=tokens)
                assert gla.gla_decode_select_impl(p, mode) == gla.GLA_IMPL_TUNED
                need = gla.gla_decode_workspace_size(p, mode)
                assert need >= last, (page, tokens, batch)
                last = need
