"""GPU parity of bf16 widths that are multiples of 8 but not of the MFMA core's
64-wide K-tile: the last K-tile of the logit products is filled up with zeros and
the gradient products' last column block is masked per column. Widths below one
K-tile, one chunk short of and one chunk past a K-tile, and past a 256-wide output
tile, with ragged tokens, one vocabulary chunk and several."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_09703_amd import api as D
from paper_2608_09703_amd import binding as B
from paper_2608_09703_amd import workloads as WL
from tests.gpu_helpers import assert_losses, assert_rows, run_fused, run_gpu, to_np
from tests.test_parity_gpu import check_head_grads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # name, workload, vocab_chunk
    ("one_chunk_width", WL.custom(1, 140, (8,), 300, w_std=0.3, seed=41), 512),
    ("below_a_k_tile", WL.custom(2, 257, (24, 56), 700, tau=1.5, w_std=0.2, ignore_frac=0.1, seed=42), 256),
    ("around_k_tiles", WL.custom(4, 130, (72, 120, 128, 136), 520, w_std=0.1, seed=43), 256),
    ("past_an_output_tile", WL.custom(3, 300, (200, 264, 408), 900, tau=2.0, w_std=0.06,
                                      ignore_frac=0.1, seed=44), 0),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_ragged_widths(case):
    name, wl, chunk = case
    print(f"[wide tail] {name} M={wl.M} T={wl.T} V={wl.V} dims={wl.dims}", flush=True)
    h, W, y = WL.make_inputs(wl, device=DEV)
    hn, Wn, yn = to_np(h), to_np(W), y.cpu().numpy()
    g_ce, g_kl = oracle.coeffs(wl.M, -1, alpha=0.4, tau=wl.tau)
    gpu = run_gpu(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk)
    ref = oracle.forward(hn, Wn, yn, tau=wl.tau)
    assert gpu["flags"] == 0
    assert_losses(gpu, ref, name)
    assert_rows(gpu, ref, what=name)
    gh, gW = oracle.backward(hn, Wn, yn, g_ce, g_kl, tau=wl.tau)
    check_head_grads(gpu, gh, gW, yn, wl.V, name)
    # the same products with a bf16 grad_h and, accumulated onto ones, with both outputs read back
    f = run_fused(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk, grad_h_dtype=torch.bfloat16)
    for i in range(wl.M):
        assert np.array_equal(torch.from_numpy(gpu["grad_h"][i]).bfloat16().float().numpy(), f["grad_h"][i])
        assert np.array_equal(gpu["grad_W"][i], f["grad_W"][i])


def test_ragged_widths_accumulate_and_leave_neighbours_alone():
    """Accumulation reads and writes exactly the outputs: columns past the width are the
    next row's, and the guard bytes behind the last row stay as they were."""
    wl = WL.custom(2, 150, (40, 296), 333, w_std=0.1, seed=45)
    h, W, y = WL.make_inputs(wl, device=DEV)
    base = run_gpu(h, W, y, g_ce=[1.0, 1.0], g_kl=[0.5, 0.0])
    p = D.make_problem(h, W, y, flags=B.MLS_ACCUMULATE_GRAD_W | B.MLS_ACCUMULATE_GRAD_H)
    buf = D.Buffers(p, torch.device(DEV))
    D.forward(p, buf, torch.device(DEV))
    flat = [torch.full((x.numel() + 64,), 2.0, device=DEV) for x in h + W]
    outs = [f[:x.numel()].view(x.shape) for f, x in zip(flat, h + W)]
    c1 = torch.tensor([1.0, 1.0], device=DEV)
    c2 = torch.tensor([0.5, 0.0], device=DEV)
    D.backward(p, buf, torch.device(DEV), c1, c2, outs[:2], outs[2:])
    torch.cuda.synchronize()
    for f, o, r in zip(flat, outs, base["grad_h"] + base["grad_W"]):
        # one rounding of values near 2 per accumulated chunk (two at most here), 2^-23 each
        assert np.abs(o.cpu().numpy() - (2.0 + r)).max() <= 4 * 2.0 ** -22 * 2
        assert torch.all(f[o.numel():] == 2.0)


@pytest.mark.parametrize("T", [3, 600])
@pytest.mark.parametrize("d", [8, 72, 120])
def test_ragged_head_logits(T, d):
    """One column tile of 32 and several of 128 tokens, 64 vocabulary rows, less than a K-tile and
    a K-tile with a rest (the larger tiles: test_head_tiles_gpu.py)."""
    g = torch.Generator(device=DEV).manual_seed(T + d)
    o = torch.randn(T, d, generator=g, device=DEV).bfloat16()
    W = torch.randn(391, d, generator=g, device=DEV).bfloat16()
    got = D.head_logits(o, W).cpu().numpy().astype(np.float64)
    on, Wn = o.double().cpu().numpy(), W.double().cpu().numpy()
    assert np.all(np.abs(got - on @ Wn.T) <= 1e-5 * (np.abs(on) @ np.abs(Wn).T) + 1e-6)
