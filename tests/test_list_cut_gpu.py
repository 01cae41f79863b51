"""The cut of a batch's tile list into chunks against the oracle, where it can go wrong: sequences on either side of the
64 that are counted at once, empty ones first, last and between, chunks that begin in front of a sequence or hold several,
several units per sequence, equal lengths that end with a chunk and such that do not."""
import pytest
import torch

import paper_2505_21487_amd as gla
from paper_2505_21487_amd.harness import DeviceProblem
from workloads import make_problem

from gpu_util import check_problem

pytestmark = pytest.mark.gpu

# kind, heads, groups, d_v, RoPE dims, query positions: the four-wave kernel (gla2_units: two units per sequence, each of
# two row blocks; gla4_units: two units) and the second MFMA kernel; the eight-wave kernel below
KERNELS = {
    "gla2_h16": ("gla", 16, 2, 256, 64, 1), "gla2_units": ("gla", 96, 2, 256, 64, 3), "gla4_units": ("gla", 64, 4, 256, 64, 2),
    "mla": ("gla", 40, 1, 512, 64, 1), "gta4_d128": ("gta", 32, 4, 128, 64, 1), "gta4_d64": ("gta", 32, 4, 64, 32, 1),
    "gqa4": ("gqa", 16, 4, 128, 0, 2),
}
LENGTHS = {
    "ragged": [0, 33, 700, 1, 0, 0, 95, 64, 2100, 5, 31, 32, 400, 0],
    "empty_first_64": [0] * 64 + [70, 0, 1300, 3],
    "around_64": [40] * 62 + [900, 0, 0, 800, 33] + [7] * 60 + [0, 500],
    "equal_aligned": [256] * 16,
    "equal_not_aligned": [352] * 19,
    "one_long": [64] * 9 + [5000],
}


@pytest.mark.parametrize("lengths", sorted(LENGTHS))
@pytest.mark.parametrize("kernel", sorted(KERNELS))
def test_cut_list(kernel, lengths):
    kind, h, g, d_v, d_r, T = KERNELS[kernel]
    lens = LENGTHS[lengths]
    p = make_problem(f"{kernel}_{lengths}", kind=kind, seq_lens=lens, T=T, h_q=h, h_c=g, d_v=d_v, **({"d_r": d_r} if d_r else {}), seed=8100 + len(kernel) + len(lengths),
                     num_pages=sum((n + 63) // 64 for n in lens) + 64, poison_tail=True)
    check_problem(p, impl=gla.GLA_IMPL_TUNED, what=f"{kernel} {lengths}")


@pytest.mark.parametrize("shape", ["mla", "gla2"])
def test_cut_list_of_the_eight_wave_kernel(shape):
    """The library's own cut, with set-ups: more than 64 sequences, empty ones first, between and around the 64th, many short
    ones per chunk, long ones over many.  Some rows of every sequence."""
    lens = [0, 0, 3] + [17, 65, 0, 129] * 14 + [0, 5000, 0, 0, 900, 0, 33] + [1, 64, 40] * 14 + [30000, 0, 21000, 7, 26000, 0]
    h, d_v, T = (128, 512, 1) if shape == "mla" else (96, 256, 3)
    if shape == "gla2":
        lens = lens + [60000]
    p = make_problem(f"cut_{shape}", seq_lens=lens, T=T, h_q=h, h_c=1 if shape == "mla" else 2, d_v=d_v, page_size=8, seed=8150,
                     num_pages=sum((n + 7) // 8 for n in lens) + 64, poison_tail=True)
    dp = DeviceProblem(p, poison_unused=True)
    out = torch.empty(p.B, T, h, d_v, dtype=torch.float32, device="cuda")
    prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=torch.empty(p.B, T, h, device="cuda"), workspace=None)
    assert gla.gla_decode_kernel_name(prm, 0, lens) == "eight-wave kernel"
    sel = [(b, t, i) for b in range(p.B) for t in range(T) for i in range(b % 7, h, 31)]
    check_problem(p, dp=dp, sel=sel, impl=gla.GLA_IMPL_TUNED, what=f"eight-wave kernel, {shape}")


# kind, heads, groups, d_v, RoPE dims, tokens per page, lengths, unused table columns, splits whose chunks are the library's own.  Lists that no chunk
# boundary has to make allowances for are cut into equal chunks in tiles, as the caller's own number of splits is: one
# sequence alone (63 tiles over 32 chunks, 7 over 3); chunks of one tile, short sequences of about one length; on the second MFMA
# kernel one long sequence in chunks of eight tiles, so that the merge does not get too many pieces
EQUAL_TILES = {
    "gla2_h16_one": ("gla", 16, 2, 256, 64, 64, [2010], 0, 32),
    "gta4_d64_one": ("gta", 32, 4, 64, 32, 32, [216], 0, 3),
    "gla2_h16_short": ("gla", 16, 2, 256, 64, 64, [190, 150, 170, 130, 185], 0, 6),
    "gta4_d64_short": ("gta", 32, 4, 64, 32, 32, [190, 150, 170, 130, 185], 6, 12),
    "gta4_d96_long": ("gta", 24, 4, 96, 48, 64, [900 * 32], 0, 113), "gqa4_d128_long_wide_table": ("gqa", 16, 4, 128, 0, 64, [700 * 32], 4 * 350, 438),
}


@pytest.mark.parametrize("name", sorted(EQUAL_TILES))
def test_chunks_without_crossings_are_equal_in_tiles(name):
    """Bit for bit what the same chunks give when the caller asks for them."""
    kind, h, g, d_v, d_r, page, lens, extra, splits = EQUAL_TILES[name]
    p = make_problem(name, kind=kind, seq_lens=lens, T=1, h_q=h, h_c=g, d_v=d_v, **({"d_r": d_r} if d_r else {}), page_size=page, seed=8200 + len(name),
                     num_pages=sum((n + page - 1) // page for n in lens) + 9, extra_table_cols=extra)
    dp = DeviceProblem(p, poison_unused=True)

    def run(n):
        kw = dict(out_dtype=torch.float32, impl=gla.GLA_IMPL_TUNED, num_splits=n)
        if kind == "gqa":
            return gla.gqa_decode(dp.q_nope, dp.key_cache, dp.state_cache, dp.page_table, dp.seq_lens, p.scale, **kw)
        return (gla.gta_decode if kind == "gta" else gla.gla_decode)(*dp.args(), **kw)

    own, asked = run(0), run(splits)
    torch.cuda.synchronize()
    assert torch.equal(own[0], asked[0]) and torch.equal(own[1], asked[1])
