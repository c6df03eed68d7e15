"""GPU parity of the fp32 path at the edges of its tiles: 64 x 64 logit tiles whose
records are grouped by 128 tokens, and the gradient GEMM's two output tiles (64 x 64;
32 x 32 with K split over the block's waves where the larger ones would leave CUs
idle). Widths that are multiples of 4, ragged tokens and vocabularies, one chunk and
several, against the float64 oracle with fp32 bounds."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_09703_amd import workloads as WL
from tests.gpu_helpers import assert_losses, assert_rows, rel_fro, run_fused, run_gpu, to_np

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # name, workload, vocab_chunk
    ("one_of_each_tile", WL.custom(1, 64, (32,), 256, dtype="f32", w_std=0.2, seed=51), 256),
    ("ragged_small", WL.custom(2, 65, (4, 36), 259, dtype="f32", tau=1.5, w_std=0.2, ignore_frac=0.1, seed=52), 256),
    ("split_k_remainders", WL.custom(3, 193, (28, 100, 132), 1021, dtype="f32", w_std=0.1, seed=53), 512),
    ("large_tile", WL.custom(2, 700, (132, 260), 9001, dtype="f32", tau=2.0, w_std=0.05, ignore_frac=0.1,
                             seed=54), 0),
    ("v2", WL.custom(2, 130, (8, 16), 2, dtype="f32", w_std=0.5, seed=55), 0),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_f32_edges(case):
    name, wl, chunk = case
    print(f"[f32] {name} M={wl.M} T={wl.T} V={wl.V} dims={wl.dims}", flush=True)
    h, W, y = WL.make_inputs(wl, device=DEV)
    hn, Wn, yn = to_np(h), to_np(W), y.cpu().numpy()
    g_ce, g_kl = oracle.coeffs(wl.M, -1, alpha=0.4, tau=wl.tau)
    gpu = run_gpu(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk)
    ref = oracle.forward(hn, Wn, yn, tau=wl.tau)
    assert gpu["flags"] == 0
    assert_losses(gpu, ref, name)
    assert_rows(gpu, ref, what=name)
    gh, gW = oracle.backward(hn, Wn, yn, g_ce, g_kl, tau=wl.tau)
    for i in range(wl.M):
        # fp32 sums and the hardware exp2 (about 2^-22 relative), with cancellation in p - q: 1e-5 is 40 ulps
        assert rel_fro(gpu["grad_h"][i], gh[i]) <= 1e-5, (name, i)
        assert rel_fro(gpu["grad_W"][i], gW[i]) <= 1e-5, (name, i)
    # a bf16 grad_h is the fp32 one rounded once, also over several chunks
    f = run_fused(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk, grad_h_dtype=torch.bfloat16)
    for i in range(wl.M):
        assert np.array_equal(torch.from_numpy(gpu["grad_h"][i]).bfloat16().float().numpy(), f["grad_h"][i])
        assert np.array_equal(gpu["grad_W"][i], f["grad_W"][i])
