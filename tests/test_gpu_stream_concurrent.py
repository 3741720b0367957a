"""Attention calls of contexts on streams of their own, side by side: the bits of the same calls one after the other, in no more time.  (A
workgroup that waits for others inside a kernel holds what the other streams' workgroups need: with such a merge four streams took 1.4
times as long as one.)"""
import pytest
import torch

from paper_2605_03644_amd import workloads as wl

pytestmark = pytest.mark.gpu
CALLS, REPLAYS = 10, 6


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


class Caller:
    def __init__(self, ad, hq, hkv, d, dtype, t_q, n_ctx, seed):
        td = torch.float32 if dtype == ad.F32 else torch.bfloat16
        rnd = lambda i, *s: wl.normal_tensor(s, td, "cuda", seed * 8 + i)  # noqa: E731
        self.ctx = ad.Context(1, hq, hkv, d, 1.0e4, dtype, max_position=1 << 16)
        self.cache, self.n = ad.Cache(self.ctx, n_ctx, with_index=False), n_ctx
        self.cache.k.copy_(rnd(0, *self.cache.k.shape))
        self.cache.v.copy_(rnd(1, *self.cache.v.shape))
        self.cache.c.len = n_ctx
        self.qkv = rnd(2, t_q, hq, d), rnd(3, t_q, hkv, d), rnd(4, t_q, hkv, d)
        self.out = [torch.empty_like(self.qkv[0]) for _ in range(CALLS)]
        self.stream, self.graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(self.stream):
            self.call(0)  # workspaces
        torch.cuda.synchronize()
        with torch.cuda.graph(self.graph, stream=self.stream):
            for i in range(CALLS):
                self.call(i)

    def call(self, i):
        self.ctx.query_attn(self.cache, 0, self.n, *self.qkv, self.n, out=self.out[i])


def _us_a_call(callers, streams):
    """All callers' graphs, on one stream or each on its own."""
    main, best = torch.cuda.current_stream(), float("inf")
    for _ in range(7):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        torch.cuda.synchronize()
        a.record()
        for s in streams:
            s.wait_stream(main)
        for _ in range(REPLAYS):
            for c, s in zip(callers, streams):
                with torch.cuda.stream(s):
                    c.graph.replay()
        for s in streams:
            main.wait_stream(s)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / (REPLAYS * CALLS * len(callers)))
    return best


@pytest.mark.parametrize("hq,hkv,d,f32,t_q,n_ctx", [(28, 4, 128, False, 1, 16000), (32, 8, 128, False, 1, 6800), (28, 4, 128, False, 16, 5000),
                                                    (32, 8, 128, False, 24, 830), (8, 2, 128, True, 32, 2300), (32, 8, 64, False, 64, 6400)])
def test_streams_side_by_side(ad, hq, hkv, d, f32, t_q, n_ctx):
    callers = [Caller(ad, hq, hkv, d, ad.F32 if f32 else ad.BF16, t_q, n_ctx, i) for i in range(4)]
    one = _us_a_call(callers, [callers[0].stream] * 4)
    alone = [c.out[-1].clone() for c in callers]
    four = _us_a_call(callers, [c.stream for c in callers])
    print(f"one stream {one:.1f}, four {four:.1f} us a call")
    for c, want in zip(callers, alone):
        assert all(torch.equal(o, want) for o in c.out)
    assert four < 1.1 * one
