"""The native marshalling of the per-layer calls (csrc/py_call.cpp) against what the arguments mean, through a
callback in place of the C entry point: arrays of any integer type, order and stride, lists, a flat block
table, tensors, addresses, None, streams.  No GPU needed."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2601_08743_amd import _py_call
from paper_2601_08743_amd import binding  # noqa: F401  (installs the converter)

_I, _P = ctypes.c_int32, ctypes.c_void_p
_FN = ctypes.CFUNCTYPE(_I, _P, _I, _P, _P, _P, _P, _P, _P, _I, _P, _P, _I, ctypes.c_float, _P)


def _call(cu, bt, pl, sl, stream=None, q=0x1000, layer=3, scale=0.25):
    seen = {}

    def ints(addr, n):
        return list((ctypes.c_int32 * n).from_address(addr)) if n else []

    def fn(ctx, layer, q, k, v, out, cu, bt, max_blocks, pl, sl, B, scale, stream):
        seen.update(ctx=ctx, layer=layer, q=q, k=k, v=v, out=out, max_blocks=max_blocks, B=B, scale=scale, stream=stream,
                    cu=ints(cu, B + 1), bt=ints(bt, B * max_blocks), pl=ints(pl, B), sl=ints(sl, B))
        return -5

    cb = _FN(fn)
    rc = _py_call.prefill(ctypes.cast(cb, _P).value, 0x77, layer, q, 0x2000, None, 0x3000, cu, bt, pl, sl, scale, stream)
    assert rc == -5
    return seen


WANT = dict(cu=[0, 4, 9], bt=[1, 2, 3, 4, 5, 6], pl=[16, 33], sl=[4, 5])


@pytest.mark.parametrize("make", [
    lambda x: np.array(x, dtype=np.int32), lambda x: np.array(x, dtype=np.int64), lambda x: np.array(x, dtype=np.uint8),
    lambda x: np.array(x, dtype=">i4"), lambda x: np.repeat(np.array(x, dtype=np.int32), 2, axis=-1)[..., ::2],
    lambda x: np.asfortranarray(np.array(x, dtype=np.int32)), lambda x: x, lambda x: torch.tensor(x)])
def test_integer_arguments(make):
    got = _call(make(WANT["cu"]), make([WANT["bt"][:3], WANT["bt"][3:]]), make(WANT["pl"]), make(WANT["sl"]))
    assert {k: got[k] for k in WANT} == WANT and got["max_blocks"] == 3 and got["B"] == 2
    assert (got["ctx"], got["layer"], got["q"], got["k"], got["v"], got["out"]) == (0x77, 3, 0x1000, 0x2000, None, 0x3000)
    assert got["scale"] == 0.25 and got["stream"] is None


def test_flat_block_table_and_empty_batch():
    assert _call(WANT["cu"], np.array(WANT["bt"], dtype=np.int32), WANT["pl"], WANT["sl"])["max_blocks"] == 3
    assert _call([0], np.zeros((0, 5), dtype=np.int32), [], [])["B"] == 0


def test_addresses_and_streams():
    t, a = torch.zeros(8), np.zeros(8, dtype=np.float32)

    class Stream:
        cuda_stream = 0x55

    assert _call(**WANT, q=t, stream=Stream())["q"] == t.data_ptr()
    got = _call(**WANT, q=a, stream=Stream())
    assert got["q"] == a.ctypes.data and got["stream"] == 0x55
    assert _call(**WANT, stream=0x66)["stream"] == 0x66


def test_what_is_no_argument_raises():
    with pytest.raises((TypeError, AttributeError)):
        _call(**WANT, q=object())
    with pytest.raises((TypeError, ValueError)):
        _call(**dict(WANT, pl=["x", "y"]))
    with pytest.raises(TypeError):
        _call(**WANT, scale="1")
    with pytest.raises(TypeError):
        _py_call.prefill(1, 2, 3)
