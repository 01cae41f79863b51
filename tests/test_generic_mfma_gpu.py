"""The generic route against the oracle.  Its MFMA kernel where general indexing can go wrong: page sizes that are
not powers of two or larger than 64, dims that are no multiple of a contraction step, an odd number of 16-byte chunks
per cache row, row counts around its 16-row waves, ranges that end inside a tile, strided tensors, separate key caches.
Its scalar kernel at every instantiation (value dims up to 128, 256, 512, 1024): odd dims, dims beyond 512, misaligned
tensors.  Both where the cache holds what it is not meant to.

fp32 results are held to 2e-5: products of bf16 are exact, weights keep 24 bits, and the largest term left is the
rounding of a score before its exponential, |score| 2^-24 relative to a weight (scores here stay below 20 in base 2,
values below 5: 20 * 0.7 * 6e-8 * 2 * 5 < 1e-5), beside sums of at most 1300 terms of total weight one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_21487_amd as gla
from paper_2505_21487_amd.harness import DeviceProblem
from workloads import make_problem

from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

LENS = [0, 1, 31, 32, 33, 300, 1, 1300]
CASES = {
    # name: (kind, h_q, h_c, d_v, d_r, T, page, splits)
    "gla2_page128": ("gla", 128, 2, 256, 64, 1, 128, 0),
    "gla2_page256_q4": ("gla", 32, 2, 256, 64, 4, 256, 3),
    "mla_page128": ("gla", 40, 1, 512, 64, 2, 128, 0),
    "page48_rope40": ("gla", 12, 3, 96, 40, 3, 48, 5),
    "page3_dv80": ("gla", 4, 1, 80, 24, 1, 3, 1),
    "page100_rope0": ("gla", 17, 1, 128, 0, 1, 100, 2),
    "gta_page7": ("gta", 18, 2, 112, 56, 1, 7, 0),
    "gqa_page24": ("gqa", 10, 2, 80, 0, 4, 24, 0),
    "gqa_dv256": ("gqa", 33, 1, 256, 0, 1, 5, 4),
    "gqa_dv512_rows1": ("gqa", 1, 1, 512, 0, 1, 64, 2),
    "rope128": ("gla", 16, 1, 64, 128, 1, 16, 0),
}


def _close(p, dp, **kw):
    _compare(*run_gpu(p, dp=dp, impl=gla.GLA_IMPL_GENERIC, out_dtype=torch.float32, **kw), *oracle.decode_problem(p))


def _compare(out, lse, ref_out, ref_lse):
    none = np.isneginf(ref_lse)
    assert np.array_equal(np.isneginf(lse), none) and (out[none] == 0).all()
    assert np.abs(out - ref_out).max() <= 2e-5
    assert np.abs(lse[~none] - ref_lse[~none]).max() <= 2e-5


@pytest.mark.parametrize("name", sorted(CASES))
def test_generic_mfma(name):
    kind, h_q, h_c, d_v, d_r, T, page, splits = CASES[name]
    p = make_problem(name, kind=kind, seq_lens=LENS, T=T, h_q=h_q, h_c=h_c, d_v=d_v, d_r=d_r, page_size=page, seed=8100 + len(name),
                     num_pages=sum(n // page + 1 for n in LENS) + 9, poison_tail=True, extra_table_cols=2, causal=0 if page == 7 else 1)
    dp = DeviceProblem(p, poison_unused=True)
    assert _name(p, dp) == "generic MFMA kernel"
    _close(p, dp, num_splits=splits)


RING = {
    # name: (kind, h_q, h_c, d_v, d_r, T, page): one range over many tiles for every number of waves and stages
    "dv128_two_slabs_page1": ("gla", 24, 1, 128, 32, 1, 1), "dv96_one_slab_page2": ("gla", 16, 2, 96, 48, 1, 2), "dv128_four_slabs": ("gla", 61, 1, 128, 64, 1, 72),
    "dv256_four_slabs_page1": ("gla", 128, 2, 256, 64, 1, 1), "dv256_two_slabs_rope128": ("gla", 20, 1, 256, 128, 1, 65), "dv208_five_blocks": ("gla", 70, 1, 208, 24, 4, 96),
    "dv512_four_slabs": ("gla", 64, 1, 512, 64, 1, 130), "dv464_two_slabs": ("gla", 10, 1, 464, 120, 3, 33), "gta_one_slab": ("gta", 16, 2, 256, 64, 1, 128),
    "gqa256_four_slabs": ("gqa", 64, 1, 256, 0, 1, 200), "gqa512_two_slabs": ("gqa", 20, 1, 512, 0, 1, 96), "gqa128_one_slab_page3": ("gqa", 9, 1, 128, 0, 1, 3),
}


@pytest.mark.parametrize("name", sorted(RING))
def test_generic_mfma_ring(name):
    """A sequence as one range: tiles of 32 to 128 tokens through every stage of the ring, page ids across the 64 or 128 a
    wave holds, last tiles that end inside or before a wave's 32 tokens; and as ranges of a few tiles."""
    kind, h_q, h_c, d_v, d_r, T, page = RING[name]
    lens = [0, 1, 129, 64, 97, 1030, 33]
    p = make_problem(name, kind=kind, seq_lens=lens, T=T, h_q=h_q, h_c=h_c, d_v=d_v, d_r=d_r, page_size=page, seed=8900 + len(name),
                     num_pages=sum(n // page + 1 for n in lens) + 9, poison_tail=True, extra_table_cols=1)
    dp = DeviceProblem(p, poison_unused=True)
    assert _name(p, dp) == "generic MFMA kernel"
    for splits in (1, 4):
        _close(p, dp, num_splits=splits)


GRIDS = {
    # name: (kind, h_q, h_c, d_v, T, page, lengths, unused table columns): automatic ranges on grids that fill the chip.  Short
    # sequences in short tables (half the waves), ranges that run in one round or in two by the lengths, two workgroups per
    # compute unit, last tiles that end in every block of 32 tokens
    "gta_short": ("gta", 16, 4, 64, 1, 33, [1 + (7 * i) % 70 for i in range(66)], 0),
    "gla256_short": ("gla", 32, 2, 256, 1, 48, [(11 * i) % 97 for i in range(130)], 1), "gqa128_short_three_positions": ("gqa", 8, 4, 128, 3, 3, [3 + (5 * i) % 131 for i in range(64)], 2),
    "gqa256_short_two_slabs": ("gqa", 12, 2, 256, 4, 128, [4 + (13 * i) % 120 for i in range(128)], 2), "gta128_two_slabs": ("gta", 48, 2, 128, 1, 96, [(9 * i) % 333 for i in range(130)], 0),
    "gla256_alike": ("gla", 64, 1, 256, 1, 128, [1300] * 61 + [0, 700, 1299], 0), "gla256_one_long": ("gla", 64, 1, 256, 1, 128, [40] * 60 + [0, 1300, 5, 1290], 0),
    "mla_16_heads": ("gla", 16, 1, 512, 1, 128, [1500, 33, 0, 1217, 640] * 8, 2), "more_than_64_sequences": ("gla", 40, 1, 256, 1, 80, [900] * 70, 0),
}


@pytest.mark.parametrize("name", sorted(GRIDS))
def test_generic_mfma_full_grids(name):
    kind, h_q, h_c, d_v, T, page, lens, extra = GRIDS[name]
    p = make_problem(name, kind=kind, seq_lens=lens, T=T, h_q=h_q, h_c=h_c, d_v=d_v, page_size=page, seed=9100 + len(name),
                     num_pages=sum(n // page + 1 for n in lens) + 9, poison_tail=True, extra_table_cols=extra)
    dp = DeviceProblem(p, poison_unused=True)
    assert _name(p, dp) == "generic MFMA kernel"
    some = sorted({0, 1, 2, p.B // 3, p.B // 2, p.B - 4, p.B - 3, p.B - 2, p.B - 1})
    sel = [(b, t, h) for b in (range(p.B) if max(lens) < 400 else some) for t in range(T) for h in range(0, h_q, 5)]
    out, lse = run_gpu(p, dp=dp, impl=gla.GLA_IMPL_GENERIC, out_dtype=torch.float32)
    at = tuple(np.asarray(sel).T)
    _compare(out[at], lse[at], *oracle.decode_problem(p, sel=sel))


def _shifted(t, by):
    """The same values in a wider buffer, each row `by` elements in."""
    wide = torch.zeros(*t.shape[:-1], t.shape[-1] + 40, dtype=t.dtype, device=t.device)
    wide[..., by:by + t.shape[-1]] = t
    return wide[..., by:by + t.shape[-1]]


def _name(p, dp):
    out = torch.empty(p.B, p.T, p.h_q, p.d_v, dtype=torch.float32, device="cuda")
    prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=torch.empty(p.B, p.T, p.h_q, device="cuda"), workspace=None, impl=gla.GLA_IMPL_GENERIC)
    return gla.gla_decode_kernel_name(prm, {"gla": 0, "gta": 1, "gqa": 2}[p.kind], p.seq_lens)


SCALAR = {
    # name: (kind, h_q, h_c, d_v, d_r, T, page, what is shifted by one element)
    "odd_dims_90": ("gla", 6, 2, 90, 32, 2, 48, None),
    "odd_dims_201": ("gla", 3, 1, 201, 40, 1, 3, None),
    "dims_328_misaligned": ("gla", 4, 1, 328, 64, 1, 128, "q_nope"),
    "dims_520": ("gla", 4, 2, 520, 24, 3, 64, None),
    "dims_1024": ("gla", 2, 1, 1024, 128, 1, 100, None),
    "gta_68": ("gta", 8, 4, 68, 34, 1, 7, None),
    "gta_256_misaligned": ("gta", 4, 2, 256, 128, 4, 64, "q_rope"),
    "gqa_80_misaligned_keys": ("gqa", 6, 3, 80, 0, 2, 24, "key_cache"),
    "gqa_256_misaligned_values": ("gqa", 2, 2, 256, 0, 1, 128, "state_cache"),
}


@pytest.mark.parametrize("splits", [0, 1, 3, 70])
@pytest.mark.parametrize("name", sorted(SCALAR))
def test_scalar_kernel(name, splits):
    kind, h_q, h_c, d_v, d_r, T, page, shifted = SCALAR[name]
    p = make_problem(name, kind=kind, seq_lens=[0, 1, 33, 300], T=T, h_q=h_q, h_c=h_c, d_v=d_v, d_r=d_r, page_size=page, seed=8250 + len(name),
                     num_pages=200, poison_tail=True, extra_table_cols=2)
    dp = DeviceProblem(p, poison_unused=True)
    if shifted is not None:
        setattr(dp, shifted, _shifted(getattr(dp, shifted), 1))
    if shifted != "key_cache":  # (not among what the query sees)
        assert _name(p, dp) == "scalar kernel"
    _close(p, dp, num_splits=splits)


@pytest.mark.parametrize("offset", [8, 4, 1])
def test_generic_strided_queries(offset):
    """Queries inside a wider buffer: 16-byte aligned (MFMA variant), 8-byte and 2-byte aligned (scalar variant)."""
    p = make_problem("strided", seq_lens=LENS, T=2, h_q=6, h_c=3, d_v=96, d_r=32, page_size=48, seed=8200, num_pages=64, poison_tail=True)
    dp = DeviceProblem(p, poison_unused=True)
    dp.q_nope = _shifted(dp.q_nope, offset)
    assert _name(p, dp) == ("generic MFMA kernel" if offset == 8 else "scalar kernel")
    _close(p, dp)


def test_merge_of_more_ranges_than_lanes():
    p = make_problem("many_ranges", seq_lens=[1300, 0, 70], T=1, h_q=5, h_c=1, d_v=112, d_r=40, page_size=5, seed=8300, num_pages=512)
    for splits in (63, 64, 65, 200):
        _close(p, DeviceProblem(p, poison_unused=True), num_splits=splits)


# ---- values a cache is not meant to hold.  A row's result depends on the keys it sees and on nothing else, and is what
# the definition gives for them (the oracle reads visible keys alone): NaN where it sees a NaN, infinite where the
# only such value it sees is an infinity of one sign.
def _set_tokens(p, b, tokens, value, dims=slice(None)):
    """Write `value` into cached tokens of sequence b: state (or value) rows, and keys where they are kept apart."""
    for tok in tokens:
        page = int(p.table_compact[b, tok // p.page_size])
        p.state_pages[page, :, tok % p.page_size, dims] = value
        if p.key_pages is not None and dims == slice(None):
            p.key_pages[page, :, tok % p.page_size] = value


def _same_with_special_values(p, **kw):
    out, lse = run_gpu(p, impl=gla.GLA_IMPL_GENERIC, out_dtype=torch.float32, **kw)
    ref_out, ref_lse = oracle.decode_problem(p)
    for got, ref in ((out, ref_out), (lse, ref_lse)):
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(ref), ref, 0))
        fin = np.isfinite(ref)
        assert (np.abs(got[fin] - ref[fin]) <= 2e-5).all()


HIDDEN_LENS = [1, 2, 4, 32, 33, 34, 35, 36, 63, 66, 300]


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("kind,d_v,T,splits", [("gla", 256, 4, 1), ("gla", 96, 2, 0), ("gta", 128, 3, 4), ("gqa", 80, 4, 3), ("gla", 512, 3, 2)])
def test_causally_hidden_keys_do_not_reach_earlier_rows(kind, d_v, T, splits, value):
    """The last T - 1 tokens are hidden from the first row and seen by later ones: on tile and range boundaries too."""
    for hidden in sorted({1, T - 1}):
        p = make_problem("hidden", kind=kind, seq_lens=HIDDEN_LENS, T=T, h_q=24, h_c=2, d_v=d_v, d_r=32 if kind == "gla" else d_v // 2,
                         page_size=128, seed=8400 + T, num_pages=40, poison_tail=True)
        for b, n in enumerate(HIDDEN_LENS):
            _set_tokens(p, b, range(max(0, n - hidden), n), value)
        ref_out, _ = oracle.decode_problem(p)
        assert np.isfinite(ref_out[:, :T - hidden]).all() and np.isnan(ref_out).any()
        _same_with_special_values(p, num_splits=splits)


@pytest.mark.parametrize("d_v,splits,aligned", [(80, 1, True), (256, 3, True), (512, 0, True), (80, 3, False), (256, 2, False)])
def test_infinite_values(d_v, splits, aligned):
    """Infinities in values whose keys, kept apart, are ordinary numbers.  (Misaligned queries: the scalar kernel.)"""
    p = make_problem("infinite", kind="gqa", seq_lens=[33, 300, 64], T=2, h_q=12, h_c=2, d_v=d_v, page_size=128, seed=8500, num_pages=16)
    inf = float("inf")
    _set_tokens(p, 0, [5], inf, d_v - 1)
    _set_tokens(p, 1, [0, 299], inf, d_v - 2)
    _set_tokens(p, 1, [140], -inf, d_v - 3)
    _set_tokens(p, 2, [63], -inf, d_v - 4)
    ref_out, _ = oracle.decode_problem(p)
    assert np.isposinf(ref_out).any() and np.isneginf(ref_out).any() and not np.isnan(ref_out).any()
    dp = DeviceProblem(p, poison_unused=True)
    if not aligned:
        dp.q_nope = _shifted(dp.q_nope, 1)
    _same_with_special_values(p, dp=dp, num_splits=splits)


def _partial_lse(p, **kw):
    """Log-sum-exps [range][batch, position, head] a call leaves in its workspace (NaN: not written), after the check of
    its result."""
    dp = DeviceProblem(p, poison_unused=True)
    out = torch.empty(p.B, p.T, p.h_q, p.d_v, dtype=torch.float32, device="cuda")
    lse = torch.empty(p.B, p.T, p.h_q, dtype=torch.float32, device="cuda")
    prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=lse, workspace=None, impl=gla.GLA_IMPL_GENERIC, **kw)
    need = gla.gla_decode_workspace_size(prm, p.kind == "gta")
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    _close(p, dp, workspace=ws, **kw)
    rows = p.B * p.T * p.h_q
    up = lambda n: (n + 255) // 256 * 256
    splits = next(s for s in range(1, 4097) if up(s * rows * p.d_v * 4) + up(s * rows * 4) == need)
    part = ws[up(splits * rows * p.d_v * 4):][:splits * rows * 4].view(torch.float32)
    return part.view(splits, p.B, p.T, p.h_q).cpu().numpy()


@pytest.mark.parametrize("extra_cols", [0, 1000])
def test_ranges_go_by_the_longest_sequence(extra_cols):
    """However wide the page table: the longest sequence is cut into ranges of 256 tokens or a little more."""
    lens = [4500, 300, 1, 0, 2100]
    p = make_problem("ranges", seq_lens=lens, T=1, h_q=128, h_c=2, d_v=256, page_size=128, seed=8700, num_pages=64, poison_tail=True,
                     extra_table_cols=extra_cols)
    used = np.isfinite(_partial_lse(p)).sum(axis=0)[:, 0]
    for b, n in enumerate(lens):
        assert (used[b] == used[b, 0]).all() and -(-n // 320) <= used[b, 0] <= -(-n // 256), (b, used[b, 0])


@pytest.mark.parametrize("page", [128, 3])
def test_small_batches_are_not_cut_too_finely(page):
    """A few output rows: no more ranges than the merge takes in one go (the scalar kernel's rule alone would cut the
    first of these into 235, the second into 256), so the rest of the workspace is left alone."""
    p = make_problem("fine", seq_lens=[30000 if page == 128 else 2600], T=1, h_q=16, h_c=1, d_v=96, d_r=32, page_size=page, seed=8800, num_pages=1200)
    dp = DeviceProblem(p, poison_unused=True)
    out = torch.empty(1, 1, 16, 96, dtype=torch.float32, device="cuda")
    prm = gla.make_params(*dp.args()[:6], p.scale, out=out, lse=torch.empty(1, 1, 16, device="cuda"), workspace=None)
    ws = torch.full((gla.gla_decode_workspace_size(prm),), 0xFF, dtype=torch.uint8, device="cuda")
    _close(p, dp, workspace=ws)
    assert (ws[64 * 16 * (96 + 1) * 4:] == 0xFF).all() and (ws[:4] != 0xFF).any()
