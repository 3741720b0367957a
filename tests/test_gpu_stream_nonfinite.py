"""Values that are not finite, in the streaming attention kernel: row j attends to its own tokens 0..j, so what later tokens
hold must not reach it (a caller may leave them unwritten), and an infinite value counts as such whatever its weight."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (dtype, head_dim, query tokens): with 2 query heads per kv head 12 tokens are two 16-row blocks; bf16 models with
# head_dim 128 run this kernel for decode steps alone
SHAPES = [("f32", 8, 12), ("f32", 32, 12), ("f32", 64, 12), ("f32", 128, 12), ("bf16", 16, 12), ("bf16", 64, 12), ("bf16", 128, 4),
          ("bf16", 256, 12)]
BAR = {"f32": 1e-4, "bf16": 2e-2}  # the bars of the kernel's other tests: the same sums in another order


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


class _Setup:
    def __init__(self, ad, dtype, d, n, form):
        w = dataclasses.replace(wl.WORKLOADS["tiny_fp32"], n_q_heads=4, n_kv_heads=2, head_dim=d, dtype=dtype, rope_theta=1.0e4)
        self.form, self.n, self.td = form, n, w.torch_dtype
        self.ctx = ad.Context.for_workload(w, n_layers=1, max_position=1 << 12)
        room = max(n, 50)
        self.k, self.v = (wl.normal_tensor((1, room, 2, d), w.torch_dtype, "cuda", s) for s in (1, 2))
        self.ctx.pool_register(self.k, self.v, np.arange(0, room + 1, 50).astype(np.int64))
        self.cache = ad.Cache(self.ctx, room, with_index=False)
        self.cache.k.copy_(self.k)
        self.cache.v = self.v                      # one buffer: a value planted in it is seen by every form
        self.cache.c.v = self.v.data_ptr()
        self.cache.c.len = n

    def run(self, q, ks, vs):
        if self.form == "pool":
            return self.ctx.query_attn_pool(0, np.arange(self.n // 50, dtype=np.int32), None, q, ks, vs, self.n).float()
        if self.form == "batch":
            outs = [torch.empty_like(q) for _ in range(2)]
            self.ctx.query_attn_batched([self.cache, self.cache], 0,
                                        [(i, self.n, q, ks, vs, self.n, outs[i]) for i in range(2)])
            torch.cuda.synchronize()
            assert torch.equal(outs[0].nan_to_num(), outs[1].nan_to_num())
            return outs[0].float()
        return self.ctx.query_attn(self.cache, 0, self.n, q, ks, vs, self.n).float()


def _forms(dtype, d):
    return ["cache", "batch"] if (dtype, d) == ("bf16", 128) else ["cache", "batch", "pool"]  # (its pool form is the tile kernel's)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("n", [0, 50, 900])
@pytest.mark.parametrize("dtype,d,t_q", SHAPES)
def test_later_own_tokens_do_not_reach_earlier_rows(ad, dtype, d, t_q, n, bad):
    for form in _forms(dtype, d):
        s = _Setup(ad, dtype, d, n, form)
        q, ks, vs = (wl.normal_tensor((t_q, h, d), s.td, "cuda", 5 + h) for h in (4, 2, 3))
        vs = vs[:, :2].contiguous()
        first = t_q // 2 - 1                        # tokens first.. hold nothing a result may use
        clean = s.run(q, ks, vs)
        vs[first:, :, : d // 2] = bad
        ks[first + 1:] = float("nan")
        got = s.run(q, ks, vs)
        assert torch.isfinite(got[:first]).all(), form
        assert float((got[:first] - clean[:first]).abs().max()) <= BAR[dtype], form
        hit = got[first, :, : d // 2]               # the row of the first bad token sees that value
        assert (torch.isnan(hit) if bad != bad else hit == bad).all(), form
        assert torch.isfinite(got[first, :, d // 2:]).all(), form
        s.ctx.close()


@pytest.mark.parametrize("dtype,d,t_q", SHAPES)
def test_infinite_value_of_weight_one(ad, dtype, d, t_q):
    """A row that sees one token returns its value, and a context key that takes the whole weight passes its infinity on."""
    for form in _forms(dtype, d):
        s = _Setup(ad, dtype, d, 0, form)
        q, ks = (wl.normal_tensor((1, h, d), s.td, "cuda", 5 + h) for h in (4, 2))
        vs = wl.normal_tensor((1, 2, d), s.td, "cuda", 9)
        vs[0, 0, 3], vs[0, 1, 0] = float("inf"), -float("inf")
        assert torch.equal(s.run(q, ks, vs).view(2, 2, d), vs.float().view(2, 1, d).expand(2, 2, d)), form
        s.ctx.close()
        s = _Setup(ad, dtype, d, 100, form)
        q, ks, vs = (wl.normal_tensor((t_q, h, d), s.td, "cuda", 5 + h) for h in (4, 2, 3))
        vs = vs[:, :2].contiguous()
        clean = s.run(q, ks, vs)
        s.v[0, 37, 0, 5] = float("inf")
        got = s.run(q, ks, vs)
        assert (got[:, :2, 5] == float("inf")).all(), form
        got[:, :2, 5] = clean[:, :2, 5]
        assert torch.isfinite(got).all() and float((got - clean).abs().max()) <= BAR[dtype], form
        s.ctx.close()
