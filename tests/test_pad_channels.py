"""Padding and cutting of channel counts the kernels do not take (``scram_pad_channels``)."""
import ctypes

import pytest
import torch

from paper_1905_10308_amd import binding


def _call(L, count=1, src=64, dst=4096, rows=2, width_short=3, width=16, elem=4, unpad=0):
    P = ctypes.c_void_p * max(count, 1)
    a = [(x + 1024 * i if x else None) for x in (src, dst) for i in range(max(count, 1))]
    n = max(count, 1)
    return L.scram_pad_channels(count, P(*a[:n]), P(*a[n:]), (ctypes.c_int64 * n)(*([rows] * n)),
                                (ctypes.c_int * n)(*([width_short] * n)), width, elem, unpad, None)


def test_bad_arguments_are_rejected_on_the_host():
    L = binding.lib()
    assert L.scram_pad_channels(1, None, None, None, None, 16, 4, 0, None) == -1
    assert _call(L, src=None) == -1
    assert _call(L, count=0) == -2
    assert _call(L, rows=0) == -2
    assert _call(L, rows=1 << 40) == -2
    assert _call(L, width_short=17) == -2
    assert _call(L, width=24) == -3
    assert _call(L, elem=8) == -3
    assert _call(L, dst=4100) == -4  # the wide side is 16-byte aligned
    assert _call(L, src=66) == -4
    assert _call(L, src=4096 + 16) == -5


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,n,width", [(1, 1, 16), (7, 3, 16), (1031, 3, 16), (65, 17, 32), (300, 63, 64), (33, 100, 128)])
def test_pad_and_cut(scram, dtype, rows, n, width):
    gen = torch.Generator(device="cuda").manual_seed(rows)
    # a source that starts off a 16-byte boundary, and one that is as wide already
    flat = torch.randn(rows * n + 1, device="cuda", generator=gen).to(dtype)
    x = flat[1:].view(1, 1, rows, n)
    y = torch.randn(1, 1, rows, width, device="cuda", generator=gen).to(dtype)
    px, py = binding._pad_channels(width, x, y)
    assert py is y
    assert torch.equal(px, torch.nn.functional.pad(x, (0, width - n)))
    cx, cy = binding._unpad(width, (px, n), (y, width))
    assert cy is y and torch.equal(cx, x)
    assert torch.equal(binding._unpad_into(y, n), y[..., :n])
