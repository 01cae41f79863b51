"""What the host decides from shapes alone.  Workspace sizes: a program may size its workspace once, for its largest
batch, and keep it as requests come and go.  The eight-wave kernel: taken by the real lengths, not by how long the page
table's rows are."""
import ctypes

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


def kernel(shape, lens, *, q_len, page, tokens, num_splits=0, num_pages=10**6):
    p, mode = params(shape, batch=len(lens), q_len=q_len, page=page, tokens=tokens)
    p.num_splits, p.num_pages = num_splits, num_pages
    return gla.gla_decode_kernel_name(p, mode, lens)


@pytest.mark.parametrize("shape,q_len,page", [("mla", 1, 64), ("mla", 1, 16), ("mla", 2, 1), ("mla_h40", 1, 8), ("gla2", 4, 64), ("gla2", 3, 1)])
def test_short_sequences_in_a_long_table_stay_with_the_four_wave_kernel(shape, q_len, page):
    for batch, length in ((1, 4096), (16, 200), (64, 200), (64, 400), (1024, 50)):
        assert kernel(shape, [length] * batch, q_len=q_len, page=page, tokens=131072) == "four-wave kernel"
    for batch, length in ((64, 16384), (128, 8192), (32, 16384)):
        assert kernel(shape, [length] * batch, q_len=q_len, page=page, tokens=131072) == "eight-wave kernel"
    # one line between them, the same however long the table
    lines = []
    for tokens in (16384, 131072):
        names = [kernel(shape, [n] * 64, q_len=q_len, page=page, tokens=tokens) for n in range(32, 16385, 32)]
        line = names.index("eight-wave kernel")
        assert names == ["four-wave kernel"] * line + ["eight-wave kernel"] * (len(names) - line)
        lines.append(line)
    assert lines[0] == lines[1]
    # not launched at all where the pool cannot hold such a batch, nor in chunks too short for it
    assert kernel(shape, [16384] * 64, q_len=q_len, page=page, tokens=131072, num_pages=4096 // page) == "four-wave kernel"
    assert kernel(shape, [16384] * 64, q_len=q_len, page=page, tokens=16384, num_splits=100) == "four-wave kernel"
    assert kernel(shape, [16384] * 64, q_len=q_len, page=page, tokens=16384, num_splits=1) == "eight-wave kernel"


def test_kernel_names():
    assert kernel("gla2", [100000] * 64, q_len=2, page=64, tokens=131072) == "four-wave kernel"   # 128 rows per group
    assert kernel("gta4_d128", [100000] * 64, q_len=4, page=64, tokens=131072) == "four-wave kernel"
    assert kernel("gta4_d64", [10], q_len=1, page=64, tokens=64) == kernel("gqa4_d128", [10], q_len=1, page=64, tokens=64) == "second MFMA kernel"
    assert kernel("gla2", [10], q_len=1, page=128, tokens=128) == "generic MFMA kernel"
    p, _ = params("gla2", batch=1, q_len=1, page=128, tokens=128)
    p.q_nope_stride[2] += 1
    assert gla.gla_decode_kernel_name(p, 0, [10]) == "scalar kernel"
    p.q_len = 5
    assert gla.gla_decode_kernel_name(p, 0, [10]) == ""


@pytest.mark.parametrize("groups,n,k", [(2, 5120, 16384), (1, 5120, 4096), (2, 2048, 8192), (1, 4096, 32768), (3, 1056, 12352), (4, 512, 8192), (2, 96, 1024)])
@pytest.mark.parametrize("sum_groups", [0, 1])
def test_more_rows_never_need_less(groups, n, k, sum_groups):
    """Projections: a workspace sized for the most rows serves every call with fewer."""
    last = 0
    for rows in range(1, 700):
        p = gla.GlaProjParams()
        p.rows, p.groups, p.n, p.k = rows, groups, n, k
        need = gla.binding.load_library().gla_proj_workspace_size(ctypes.byref(p), sum_groups)
        assert need >= last, rows
        last = need
