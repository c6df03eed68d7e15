"""GPU parity of the head product at the edges between its tiles: 32, 64 and 128 token
columns, 64, 128 and 192 vocabulary rows (vocabularies above and below a block per CU),
one K-tile, fewer K-tiles than stages and a ragged width, with guard values behind the
logits."""

import pytest
import torch

from paper_2608_09703_amd import api as D

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("d", [64, 192, 200, 640])
@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 65, 129, 384, 385])
def test_head_tiles(T, d):
    for V in (63, 1031, 32769 if T in (65, 385) else 4100):
        g = torch.Generator(device=DEV).manual_seed(T * 1000 + d + V)
        o = (torch.randn(T, d, generator=g, device=DEV) * 3).bfloat16()
        W = (torch.randn(V, d, generator=g, device=DEV) * 0.05).bfloat16()
        flat = torch.full((T * V + 256,), 7.0, device=DEV)
        got = D.head_logits(o, W, out=flat[:T * V].view(T, V))
        on, Wn = o.double(), W.double()
        bound = 1e-5 * (on.abs() @ Wn.abs().t()) + 1e-6
        assert torch.all((got.double() - on @ Wn.t()).abs() <= bound), (T, V, d)
        assert torch.all(flat[T * V:] == 7.0)
