"""What the binding hands to the library: attention items packed in one piece, and the stream of a call."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2605_03644_amd import binding as ad


@pytest.mark.parametrize("n", [0, 1, 3, 48])
def test_packed_items_are_the_structures(n):
    items = [(i - 1 if i else -1, 10 ** 12 + i, torch.empty(2 + i, 4, 8), torch.empty(2 + i, 2, 8), torch.empty(2 + i, 2, 8), 7 * i - 3,
              torch.empty(2 + i, 4, 8)) for i in range(n)]
    arr = ad.Context.pack_attn_items(items)
    assert isinstance(arr, ctypes.Array) and arr._type_ is ad.AttnItem and len(arr) == n
    for got, (ci, n_ctx, q, ks, vs, pos, out) in zip(arr, items):
        want = ad.AttnItem(q.data_ptr(), ks.data_ptr(), vs.data_ptr(), out.data_ptr(), n_ctx, pos, q.shape[0], ci)
        assert bytes(got) == bytes(want)


def test_a_strided_item_is_refused():
    x = torch.empty(4, 4, 16)
    with pytest.raises(AssertionError):
        ad.Context.pack_attn_items([(0, 1, x[..., :8], x, x, 0, x)])


@pytest.mark.parametrize("n", [0, 1, 7])
@pytest.mark.parametrize("writable", [True, False])
def test_the_address_of_an_array(n, writable):
    base = np.arange(n + 3, dtype=np.int32)
    a = base[2:2 + n]
    a.flags.writeable = writable
    assert n == 0 or ad._host_addr(a) == a.ctypes.data == base.ctypes.data + 8
    assert isinstance(ad._host_addr(a), int)


@pytest.mark.gpu
def test_the_stream_of_a_call_is_the_current_one():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    side = torch.cuda.Stream()
    assert ad._stream_ptr() == torch.cuda.current_stream().cuda_stream
    assert ad._stream_ptr(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert ad._stream_ptr() == torch.cuda.current_stream().cuda_stream == side.cuda_stream
    assert ad._stream_ptr() == torch.cuda.current_stream().cuda_stream
