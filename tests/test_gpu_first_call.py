"""The first calls on a new context, issued at once on a stream that is not ordered behind the null stream: what
adapshot_create uploads (rotation tables, arrival counters at zero) is there by then, and the counters are at zero after."""
import pytest
import torch

from paper_2605_03644_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


def test_first_calls_on_a_non_blocking_stream(ad):
    n, stream = 2000, torch.cuda.Stream()               # torch's streams are non-blocking
    k, v = (wl.normal_tensor((1, n, 2, 64), torch.float32, "cuda", s) for s in (1, 2))
    q, ks, vs = (wl.normal_tensor((8, h, 64), torch.float32, "cuda", 5 + h) for h in (4, 2, 3))
    vs = vs[:, :2].contiguous()
    z = torch.randn(3, 20000, device="cuda")
    out, h = torch.zeros_like(q), torch.zeros(3, device="cuda")
    torch.cuda.synchronize()
    results = []
    for first in ("attention", "entropy"):
        for _ in range(4):
            ctx = ad.Context(1, 4, 2, 64, 1.0e4, ad.F32, max_position=1 << 12)
            caches = ad.CacheStruct(k.data_ptr(), v.data_ptr(), n, n, None, None, None)
            cache = type("C", (), {"c": caches})()      # (ad.Cache would fill its buffers on the default stream first)
            ctx.set_attn_splits(8)
            for _ in range(2):
                if first == "entropy":
                    ctx.probe_entropy(z, out=h, stream=stream)
                ctx.query_attn(cache, 0, n, q, ks, vs, n, out=out, stream=stream)
                ctx.probe_entropy(z, out=h, stream=stream)
                stream.synchronize()
                results.append((out.clone(), h.clone()))
                torch.cuda.synchronize()
                out.fill_(7.0)
                h.fill_(7.0)
                torch.cuda.synchronize()
            ctx.close()
    for o, e in results:
        assert torch.equal(o, results[0][0]) and torch.equal(e, results[0][1])
    assert torch.isfinite(results[0][0]).all()
    lp = torch.log_softmax(z.double(), dim=-1)
    assert float((results[0][1].double() + (lp.exp() * lp).sum(-1)).abs().max()) <= 1e-4
