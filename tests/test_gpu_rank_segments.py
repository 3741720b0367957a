"""The key pass of relevance ranking (bf16, head_dim 128) where it can go wrong: shots that begin, end or lie inside a block
of 32 keys, many of them in one, shots cut by a split, partial row tiles of both widths, and score ranges that move the rows'
references."""
import numpy as np
import pytest
import torch

from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


LENGTHS = {
    "ones": [1] * 700,
    "tiny": [1, 2, 3, 4, 5, 31, 32, 33, 1, 1, 63, 64, 65, 96, 7] * 6,
    "whole_blocks": [32, 64, 96, 256, 512] * 2,
    "one_long": [1500],
    "mixed": [700, 1, 48, 160, 33, 290, 2, 2, 2, 129],
    # few keys a segment: the form that sums a block's segments by matrix instructions
    "short": [1, 2, 3, 4, 5, 31, 1, 1, 2, 7, 33, 1] * 19,
    "fours": [4] * 300,
    "tens": [10] * 150,
    "long_then_ones": [300] + [1] * 70 + [65] + [1, 1, 2] * 30,
}
# factor of key u's length, of n keys: the usual range; a range that grows or shrinks by hundreds of log2 units inside a
# split; scores that lie far from 0 from the first key on
SCALES = {
    "plain": lambda u, n: np.ones(n),
    "growing": lambda u, n: 0.2 + 40.0 * (u % 256) / 256.0,
    "falling": lambda u, n: 0.2 + 40.0 * (255 - u % 256) / 256.0,
    "far": lambda u, n: np.full(n, 60.0),
    "late_peak": lambda u, n: np.where(u % 256 > 200, 60.0, 0.01),
}


@pytest.mark.parametrize("g", [3, 64, 300])
@pytest.mark.parametrize("scale", list(SCALES))
@pytest.mark.parametrize("lengths", list(LENGTHS))
def test_rank_segments_against_float64(ad, lengths, scale, g):
    """One query token at position 0 over keys used as stored: the rounded, scaled query is known exactly, so a float64
    softmax is the reference.  Bound: a score of sum |q k| = S (log2 units) carries fp32 accumulation errors below
    8 * 2^-24 * S (128 products, summed in pieces), and 2^x turns that into ln(2) times as much; S is at most 2500 here,
    which gives 8.3e-4; the sums of up to 1500 positive terms and the exponential add less than 1e-4."""
    hkv = 2
    lens = np.array(LENGTHS[lengths])
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    gen = torch.Generator().manual_seed(len(lens) * 100 + g)
    u = np.arange(n)
    k = torch.randn(1, n, hkv, 128, generator=gen) * torch.from_numpy(SCALES[scale](u, n)).float()[None, :, None, None]
    k = k.bfloat16()
    q = torch.randn(1, hkv * g, 128, generator=gen).bfloat16()
    ctx = ad.Context(1, hkv * g, hkv, 128, 1.0e4, ad.BF16, key_state=ad.KEYS_ROTATED_LOCAL, max_position=1 << 12)
    kd = k.cuda()
    ctx.pool_register(kd, kd.clone(), off)
    got = ctx.rank_shots(0, q.cuda()).cpu().numpy().astype(np.float64)
    again = ctx.rank_shots(0, q.cuda()).cpu().numpy().astype(np.float64)
    assert np.array_equal(got, again)
    qs = (q.float() * np.float32(1.4426950408889634 / np.sqrt(128.0))).bfloat16().double()[0].view(hkv, g, 128)
    s = torch.einsum("hgd,uhd->hgu", qs, k[0].double())
    largest = float(torch.einsum("hgd,uhd->hgu", qs.abs(), k[0].double().abs()).max())
    assert largest < 2500.0
    p = torch.softmax(s * np.log(2.0), dim=-1).mean(dim=(0, 1)).numpy()
    want = np.array([p[a:b].sum() / (b - a) for a, b in zip(off[:-1], off[1:])])
    bound = np.log(2.0) * 8 * 2.0 ** -24 * largest + 1e-4
    err = np.abs(got - want)
    assert float(np.max(err - bound * want)) <= 1e-7 * want.max(), float(np.max(err / np.maximum(want, 1e-30)))
    ctx.close()


@pytest.mark.parametrize("key_state", [0, 1])
@pytest.mark.parametrize("t_q,h_q,h_kv", [(70, 32, 8), (150, 28, 4), (1, 5, 1)])
def test_rank_wide_row_tiles_against_oracle(ad, oracle_mod, key_state, t_q, h_q, h_kv):
    """More than 256 rows per kv head (two row blocks per wavefront, a second row tile), and five rows in all; a pool whose
    first shot does not start at token 0."""
    rng = np.random.default_rng(t_q)
    off = (np.concatenate([[0], np.cumsum(rng.integers(20, 130, 30))]) + 17).astype(np.int64)
    g = torch.Generator(device="cuda"); g.manual_seed(t_q)
    k = torch.randn(1, int(off[-1]), h_kv, 128, device="cuda", generator=g).bfloat16()
    q = torch.randn(t_q, h_q, 128, device="cuda", generator=g).bfloat16()
    ctx = ad.Context(1, h_q, h_kv, 128, 5.0e5, ad.BF16, key_state=key_state, max_position=1 << 12)
    ctx.pool_register(k, k.clone(), off)
    got = ctx.rank_shots(0, q, q_pos0=9).cpu().numpy().astype(np.float64)
    want = oracle_mod.rank_scores(H.to_storage(k[:, 17:].contiguous())[0], "bf16", off - 17, H.to_storage(q), 5.0e5, key_state,
                                  q_pos0=9)
    err = np.abs(got - want)   # the rotated query is rounded to bf16 on the GPU, not in the oracle
    assert float(err.max()) <= 2e-2 * want.max() and float((err / want).mean()) < 5e-3
    assert abs(float((got * np.diff(off)).sum()) - 1.0) < 1e-5   # fp32 sums: all attention mass is accounted for
    ctx.close()


@pytest.mark.parametrize("t_q", [3, 80])
def test_rank_short_shots_in_a_pool_that_begins_late(ad, oracle_mod, t_q):
    """Shots of one to five tokens, un-rotated keys, the first shot at token 5, one and two row blocks per wavefront."""
    rng = np.random.default_rng(t_q)
    off = (np.concatenate([[0], np.cumsum(rng.integers(1, 6, 700))]) + 5).astype(np.int64)
    g = torch.Generator(device="cuda"); g.manual_seed(t_q)
    k = torch.randn(1, int(off[-1]), 4, 128, device="cuda", generator=g).bfloat16()
    q = torch.randn(t_q, 28, 128, device="cuda", generator=g).bfloat16()
    ctx = ad.Context(1, 28, 4, 128, 5.0e5, ad.BF16, key_state=ad.KEYS_UNROTATED, max_position=1 << 12)
    ctx.pool_register(k, k.clone(), off)
    got = ctx.rank_shots(0, q, q_pos0=9).cpu().numpy().astype(np.float64)
    want = oracle_mod.rank_scores(H.to_storage(k[:, 5:].contiguous())[0], "bf16", off - 5, H.to_storage(q), 5.0e5,
                                  ad.KEYS_UNROTATED, q_pos0=9)
    err = np.abs(got - want)   # the bars of the wide-tile test above, for the same reason
    assert float(err.max()) <= 2e-2 * want.max() and float((err / want).mean()) < 5e-3
    assert abs(float((got * np.diff(off)).sum()) - 1.0) < 1e-5
    ctx.close()
