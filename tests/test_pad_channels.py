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


def test_tensors_without_elements():
    """No channels pad to zeros, no rows to no rows, and zero channels of a wide tensor are an empty one: nothing of
    it needs the library."""
    none, row = torch.empty(2, 3, 4, 0), torch.empty(0, 3, 4, 5)
    a, b = binding._pad_channels(16, none, row)
    assert a.shape == (2, 3, 4, 16) and not a.any() and b.shape == (0, 3, 4, 16)
    wide = torch.ones(2, 3, 4, 16)
    assert binding._unpad_into(wide, 0).shape == (2, 3, 4, 0)
    out = torch.empty(2, 3, 4, 0)
    assert binding._unpad_into(wide, 0, out) is out
    c, d = binding._unpad(16, (wide, 0), (wide, 16))
    assert c.shape == (2, 3, 4, 0) and d is wide


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_calls_without_channels(scram, dtype):
    """Queries and keys of no channels score 0 everywhere, values of none give rows of none."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    Q, K, V = (torch.randn(2, 9, 11, 3, device="cuda", generator=gen).to(dtype) for _ in range(3))
    none = Q[..., :0].contiguous()
    J, s = scram.patchmatch(none, none, 2, 7, return_score=True)
    assert not s.any() and ((J >= 0) & (J < 99)).all()
    assert torch.equal(scram.patchmatch_kappa(none, none, 1, 2, 7)[0], J)
    # every key of the window has the same weight
    got, want = (scram.sparse_attend(q, k, V, J, 3, 1.0) for q, k in ((none, none), (Q * 0, K)))
    assert torch.equal(got, want)
    assert scram.sparse_attend(Q, K, none, J, 3).shape == (2, 9, 11, 0)
    assert scram.snis_attend(Q, K, none, J, 8).shape == (2, 9, 11, 0)
    dQ, dK, dV = scram.sparse_attend_backward(Q, K, none, J, none, 3)
    assert not dQ.any() and not dK.any() and dV.shape == (2, 9, 11, 0)
    dQ, dK, dV = scram.sparse_attend_backward(none, none, V, J, V, 3, 1.0)
    assert dQ.shape == dK.shape == (2, 9, 11, 0) and dV.shape == V.shape and dV.any()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float16, torch.int32])
def test_other_types_are_refused_as_such(scram, dtype):
    """Also where rows of 8-byte elements would have to be padded first: a TypeError, as for widths that need none."""
    Q = torch.zeros(1, 4, 5, 3, device="cuda", dtype=dtype)
    J = torch.zeros(1, 4, 5, device="cuda", dtype=torch.int32)
    for call in (lambda: scram.patchmatch(Q, Q, 1, 0), lambda: scram.patchmatch_kappa(Q, Q, 2, 1, 0),
                 lambda: scram.patchmatch_noalloc(Q, Q, 1, 0), lambda: scram.sparse_attend(Q, Q, Q, J, 3),
                 lambda: scram.sparse_attend_backward(Q, Q, Q, J, Q, 3), lambda: scram.snis_attend(Q, Q, Q, J, 4),
                 lambda: scram.forward(Q, Q, Q, 1, 0, 3)):
        with pytest.raises(TypeError):
            call()
