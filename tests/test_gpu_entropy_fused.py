"""Entropy in one launch: rows of one chunk, of two, of more chunks than a wavefront has lanes; row counts at which the
arrival counters move closer together, and beyond which the merge has a launch of its own; ragged strides; calls one after the other on the same counters."""
import numpy as np
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


def _want(z, tokens):
    z = z.double()
    lp = torch.log_softmax(z, dim=-1)
    if tokens:
        lp = lp[:, tokens]
    return (-lp.exp() * lp).sum(-1)


@pytest.mark.parametrize("rows,vocab,stride", [(1, 1, 1), (1, 1025, 1028), (3, 2047, 2047), (1, 128256, 128256), (17, 70001, 70001),
                                               (127, 9000, 9000), (129, 9000, 9001), (255, 20480, 20480), (1024, 8193, 8196), (1025, 8193, 8193), (4096, 8193, 8196),
                                               (4097, 8193, 8196)])
@pytest.mark.parametrize("tokens", [None, [0, 5]])
def test_entropy_one_launch(ad, rows, vocab, stride, tokens):
    """1e-4 absolute, the bar of every entropy test: exponent errors of 2^-24 |x| and fp32 sums give about 2e-6."""
    if tokens and vocab < 6:
        tokens = [0]
    ctx = ad.Context(1, 4, 2, 64, 1.0e4, ad.F32, max_position=1 << 12)
    g = torch.Generator(device="cuda"); g.manual_seed(rows + vocab)
    buf = torch.randn(rows, stride, device="cuda", generator=g) * 2.0 ** 0.5
    z = buf[:, :vocab]
    for rep in range(3):   # the counters are back at zero every time
        h = torch.full((rows,), -7.0, device="cuda")
        if tokens:
            ctx.probe_entropy_tokens(z, tokens, out=h)
        else:
            ctx.probe_entropy(z, out=h)
        if rep == 0:
            first = h.clone()
        assert torch.equal(h, first)
    assert float((first.double() - _want(z, tokens)).abs().max()) <= 1e-4
    ctx.close()


@pytest.mark.parametrize("rows,vocab,launches", [(1024, 10000, 1), (1025, 10000, 2), (9000, 10000, 2), (9000, 3000, 1), (300, 20000, 1)])
@pytest.mark.parametrize("tokens", [None, [1, 7]])
def test_many_rows_of_several_chunks_merge_in_a_second_launch(ad, rows, vocab, launches, tokens):
    """Beyond 1024 rows of several chunks arrivals cost what a launch does."""
    ctx = ad.Context(1, 4, 2, 64, 1.0e4, ad.F32, max_position=1 << 12)
    z = torch.randn(rows, vocab, device="cuda")
    ctx.profile_enable(True)
    h = ctx.probe_entropy_tokens(z, tokens) if tokens else ctx.probe_entropy(z)
    torch.cuda.synchronize()
    got = ctx.profile_read()
    assert (got["entropy_chunk"][1], got["entropy_finish"][1]) == (1, launches - 1)
    assert float((h.double() - _want(z, tokens)).abs().max()) <= 1e-4
    ctx.close()
