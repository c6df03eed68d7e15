"""GPU parity of the head product at the edges between its tiles: 32, 64 and 128 token
columns, 64, 128 and 192 vocabulary rows (vocabularies above and below a block per CU),
one K-tile, fewer K-tiles than stages and a ragged width, 16-byte and scalar stores, with
guard values behind the logits."""

import ctypes

import pytest
import torch

from paper_2608_09703_amd import api as D
from paper_2608_09703_amd import binding as B

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _tile(T, V):
    """(vocabulary rows, token columns) of the tile that the library takes for bf16."""
    f = B.lib()._ZN3mls9head_tileEbllPiS0_  # mls::head_tile(bool, long, long, int*, int*)
    f.restype = None
    f.argtypes = [ctypes.c_bool, ctypes.c_long, ctypes.c_long, ctypes.POINTER(ctypes.c_int),
                  ctypes.POINTER(ctypes.c_int)]
    rows, cols = ctypes.c_int(), ctypes.c_int()
    f(True, T, V, ctypes.byref(rows), ctypes.byref(cols))
    return rows.value, cols.value


def _check(T, V, d):
    g = torch.Generator(device=DEV).manual_seed(T * 1000 + d + V)
    o = (torch.randn(T, d, generator=g, device=DEV) * 3).bfloat16()
    W = (torch.randn(V, d, generator=g, device=DEV) * 0.05).bfloat16()
    flat = torch.full((T * V + 256,), 7.0, device=DEV)
    got = D.head_logits(o, W, out=flat[:T * V].view(T, V))
    on, Wn = o.double(), W.double()
    bound = 1e-5 * (on.abs() @ Wn.abs().t()) + 1e-6
    assert torch.all((got.double() - on @ Wn.t()).abs() <= bound), (T, V, d)
    assert torch.all(flat[T * V:] == 7.0)


@pytest.mark.parametrize("d", [64, 192, 200, 640])
@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 65, 129, 384, 385])
def test_head_tiles(T, d):
    for V in (63, 1031, 32769 if T in (65, 385) else 4100):
        _check(T, V, d)


@pytest.mark.parametrize("d", [192, 200])
@pytest.mark.parametrize("T,tile", [(65, (128, 128)), (129, (128, 128)), (385, (192, 128))])
def test_large_head_tiles_with_16_byte_stores(T, tile, d):
    """Whole vocabulary tiles and a rest of four rows, with and without a K tail."""
    for V in (32768, 32772):
        assert _tile(T, V) == tile
        _check(T, V, d)


def test_every_tile_is_reached():
    """The sizes above run each tile that the rule has."""
    seen = {_tile(T, V) for T in (1, 31, 32, 33, 64, 65, 129, 384, 385) for V in (63, 1031, 4100, 32769)}
    assert seen == {(64, 32), (64, 64), (64, 128), (128, 128), (192, 128)}
