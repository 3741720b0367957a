"""A single key far above all others (an attention sink), at every position of a 64-key tile: whatever lane and register its
score lands in, the reference maximum has to see it, or 2^(s - m) overflows."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("tile", [0, 1, 4])
@pytest.mark.parametrize("n_split", [1, 2])
def test_attention_sees_a_sink_at_every_key_position(ad, tile, n_split):
    """The query and the sink live in columns 63 and 127, whose frequency (5e5^(-126/128) = 2.5e-6 per position) turns them
    by less than 1e-3 here.  The sink's score exceeds the others by more than 2 * 128 in log2 units, so its softmax weight
    is 1 and the output is its value row exactly (one product, one fp16 partial scaled by its own largest element: both
    bf16 roundings leave a difference of at most 2^-8 relative to the row's largest element)."""
    h, d, t_q, n = 4, 128, 160, 448
    ctx = ad.Context(1, h, h, d, 5.0e5, ad.BF16, max_position=1 << 12)
    ctx.set_attn_splits(n_split)
    cache = ad.Cache(ctx, n, with_index=False)
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    noise = (0.01 * torch.randn(1, n, h, d, device="cuda", generator=g)).bfloat16()
    cache.v.copy_(torch.randn(1, n, h, d, device="cuda", generator=g).bfloat16())
    cache.c.len = n
    q = torch.zeros(t_q, h, d, device="cuda", dtype=torch.bfloat16)
    q[:, :, 63] = q[:, :, 127] = 11.0
    ks = (0.01 * torch.randn(t_q, h, d, device="cuda", generator=g)).bfloat16()
    vs = torch.randn(t_q, h, d, device="cuda", generator=g).bfloat16()
    for pos in range(64):
        at = 64 * tile + pos
        cache.k.copy_(noise)
        cache.k[0, at, :, 63] = cache.k[0, at, :, 127] = 100.0
        out = ctx.query_attn(cache, 0, n, q, ks, vs, 0).float()
        want = cache.v[0, at].float().expand(t_q, h, d)
        err = (out - want).abs() / want.abs().amax(-1, keepdim=True)
        assert not torch.isnan(out).any(), pos
        assert float(err.max()) <= 2.0 ** -8, (pos, float(err.max()))
    ctx.close()
