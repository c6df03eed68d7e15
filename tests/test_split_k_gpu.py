"""GPU parity of grad_h products taken in K parts (few tokens against the vocabulary):
both plans, a shorter last vocabulary chunk with fewer parts, fp32 and bf16 outputs,
accumulation, a skipped output, and the same bits on every run."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_09703_amd import api as D
from paper_2608_09703_amd import binding as B
from paper_2608_09703_amd import workloads as WL
from tests.gpu_helpers import run_fused, run_gpu, to_np
from tests.test_parity_gpu import check_head_grads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # name, workload, vocab_chunk
    ("one_chunk", WL.custom(2, 140, (64, 192), 9000, w_std=0.08, ignore_frac=0.1, seed=61), 9216),
    ("short_last_chunk", WL.custom(3, 257, (64, 128, 320), 9000, tau=1.5, w_std=0.08, seed=62), 4096),
    ("ragged_width", WL.custom(1, 200, (72,), 20011, w_std=0.1, seed=63), 0),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_k_parts(case):
    name, wl, chunk = case
    print(f"[k parts] {name} M={wl.M} T={wl.T} V={wl.V} dims={wl.dims}", flush=True)
    h, W, y = WL.make_inputs(wl, device=DEV)
    hn, Wn, yn = to_np(h), to_np(W), y.cpu().numpy()
    g_ce, g_kl = oracle.coeffs(wl.M, -1, alpha=0.4, tau=wl.tau)
    gh, gW = oracle.backward(hn, Wn, yn, g_ce, g_kl, tau=wl.tau)
    sep = run_gpu(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk)
    check_head_grads(sep, gh, gW, yn, wl.V, name)
    fus = run_fused(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk)
    check_head_grads(fus, gh, gW, yn, wl.V, name + " fused")
    again = run_gpu(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk)
    fus16 = run_fused(h, W, y, tau=wl.tau, g_ce=g_ce, g_kl=g_kl, vocab_chunk=chunk,
                      grad_h_dtype=torch.bfloat16)
    for i in range(wl.M):
        assert np.array_equal(sep["grad_h"][i], again["grad_h"][i])
        # a bf16 grad_h is the fp32 one rounded once
        assert np.array_equal(torch.from_numpy(fus["grad_h"][i]).bfloat16().float().numpy(), fus16["grad_h"][i])


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_k_parts_accumulate_and_skip(dt):
    """MLS_ACCUMULATE_GRAD_H adds the sum of the parts to the output once; a NULL output is skipped."""
    wl = WL.custom(2, 150, (64, 128), 9000, w_std=0.1, seed=64)
    h, W, y = WL.make_inputs(wl, device=DEV)
    base = run_gpu(h, W, y, g_ce=[1.0, 1.0], g_kl=[0.5, 0.0])
    dev = torch.device(DEV)
    p = D.make_problem(h, W, y, flags=B.MLS_ACCUMULATE_GRAD_H, grad_h_dtype=dt)
    buf = D.Buffers(p, dev)
    D.forward(p, buf, dev)
    out = torch.full(h[1].shape, 0.5, device=DEV, dtype=dt)
    c = [torch.tensor(v, device=DEV) for v in ([1.0, 1.0], [0.5, 0.0])]
    D.backward(p, buf, dev, c[0], c[1], [None, out], [None, None])
    want = (torch.tensor(base["grad_h"][1], device=DEV) + 0.5).to(dt)
    assert torch.equal(out, want)


def test_no_sum_without_a_hidden_state_gradient():
    """The sum over the parts is launched with the gradients it is for, in both plans, and only then;
    the head gradients are the same bits either way."""
    wl = WL.custom(2, 150, (64, 128), 9000, w_std=0.1, seed=65)
    h, W, y = WL.make_inputs(wl, device=DEV)
    dev = torch.device(DEV)
    p = D.make_problem(h, W, y)
    buf = D.Buffers(p, dev)
    c = [torch.tensor(v, device=DEV) for v in ([1.0, 1.0], [0.5, 0.0])]
    ws = torch.empty(B.query_fwd_bwd_workspace(p), dtype=torch.uint8, device=DEV)
    gh = [torch.empty(x.shape, device=DEV) for x in h]
    D.forward(p, buf, dev)
    for fused in (False, True):
        got = {}
        for want_h in (True, False):
            gW = [torch.empty(x.shape, device=DEV) for x in W]
            outs = gh if want_h else [None, None]
            B.profile_enable(True)
            try:
                if fused:
                    B.distill_fwd_bwd(p, buf.stats.data_ptr(), buf.ce.data_ptr(), buf.kl.data_ptr(), None,
                                      c[0].data_ptr(), c[1].data_ptr(),
                                      [x.data_ptr() if x is not None else None for x in outs],
                                      [x.data_ptr() for x in gW], ws.data_ptr(), ws.numel(), D._stream(dev))
                else:
                    D.backward(p, buf, dev, c[0], c[1], outs, gW)
                assert ("split_sum" in B.profile_report()) == want_h, (fused, want_h)
            finally:
                B.profile_enable(False)
            got[want_h] = gW
        assert all(torch.equal(a, b) for a, b in zip(got[True], got[False]))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dims", [(64, 192), (72, 296)])
def test_any_workspace_from_the_slab_on_is_taken(dims, dt):
    """A call takes as many parts as its workspace holds: none, some, all of them, and the same ones in
    any larger workspace; the gradients agree with the oracle and nothing past the workspace is written."""
    wl = WL.custom(2, 140, dims, 20011, w_std=0.08, seed=66)
    h, W, y = WL.make_inputs(wl, device=DEV)
    hn, Wn, yn = to_np(h), to_np(W), y.cpu().numpy()
    g_ce, g_kl = oracle.coeffs(2, -1, alpha=0.4, tau=1.0)
    gh, gW = oracle.backward(hn, Wn, yn, g_ce, g_kl)
    dev = torch.device(DEV)
    p = D.make_problem(h, W, y, grad_h_dtype=dt)
    buf = D.Buffers(p, dev)
    D.forward(p, buf, dev)
    c = [torch.tensor(v, device=DEV, dtype=torch.float32) for v in (g_ce, g_kl)]
    part = 140 * sum(dims) * 4
    for fused in (False, True):
        size = B.query_fwd_bwd_workspace(p) if fused else buf.ws_bytes
        with pytest.raises(B.MlsError, match=r"needs \d+ workspace") as e:
            _call(p, buf, dev, c, h, W, dt, fused, 16)
        need = int(str(e.value).split("needs ")[1].split()[0])
        assert need < size
        seen = {}
        for nbytes in (need, need + 256, need + 2 * part, need + 3 * part + 256, size, size + 4096):
            gpu = _call(p, buf, dev, c, h, W, dt, fused, nbytes)
            check_head_grads(gpu, gh, gW, yn, wl.V, f"{dims} fused={fused} {nbytes} bytes")
            seen[nbytes] = gpu
        assert all(np.array_equal(a, b) for a, b in zip(seen[size]["grad_h"], seen[size + 4096]["grad_h"]))
        assert all(np.array_equal(a, b) for a, b in zip(seen[need]["grad_W"], seen[size]["grad_W"]))


def _call(p, buf, dev, c, h, W, dt, fused, nbytes):
    """Gradients of one backward (or fused call) in a workspace of exactly nbytes, guard bytes behind it."""
    ws = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    gh = [torch.full(x.shape, float("nan"), dtype=dt, device=DEV) for x in h]
    gW = [torch.full(x.shape, float("nan"), device=DEV) for x in W]
    ptrs = [x.data_ptr() for x in gh], [x.data_ptr() for x in gW]
    cp = c[0].data_ptr(), c[1].data_ptr()
    if fused:
        B.distill_fwd_bwd(p, buf.stats.data_ptr(), buf.ce.data_ptr(), buf.kl.data_ptr(), None, *cp, *ptrs,
                          ws.data_ptr(), nbytes, D._stream(dev))
    else:
        B.distill_bwd(p, buf.stats.data_ptr(), *cp, *ptrs, ws.data_ptr(), nbytes, D._stream(dev))
    torch.cuda.synchronize()
    assert torch.all(ws[nbytes:] == 0xA5)
    return {"grad_h": to_np(gh), "grad_W": to_np(gW)}
