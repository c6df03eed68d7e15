"""The front end's cached descriptors and raw stream handles: settings that hash by
identity are taken by value, descriptors are not mixed up between calls, and every
form of device that names a stream still does."""

from types import SimpleNamespace

import pytest
import torch

from paper_2608_09703_amd import api as D
from paper_2608_09703_amd import binding as B


def test_cached_descriptors_carry_their_own_values():
    a = D._make_sampling(1000, 0.4, 0.9, False)
    b = D._make_sampling(1000, 0.5, 0.9, False)
    c = D._make_sampling(1000, 0.4, 0.9, True)
    assert (a.temperature, b.temperature, c.greedy) == (pytest.approx(0.4), 0.5, 1)
    assert D._make_sampling(1000, 0.4, 0.9, False) is a and a.greedy == 0
    j = D._make_junction(5, 64, 128, B.MLS_BF16, B.MLS_F32, B.MLS_JUNCTION_FRESH_FIRST, 0)
    k = D._make_junction(5, 64, 128, B.MLS_F32, B.MLS_F32, B.MLS_JUNCTION_FRESH_FIRST, 0)
    assert (j.T, j.d_prev, j.d_fresh, j.act_dtype, k.act_dtype) == (5, 64, 128, B.MLS_BF16, B.MLS_F32)
    assert D._make_junction.cache_info().maxsize == D._make_sampling.cache_info().maxsize == 256


def test_settings_are_converted_as_the_descriptor_does():
    import numpy as np
    t = torch.tensor(0.25)
    assert D._sampling(1000, t, np.float32(0.5), 1).temperature == 0.25
    t.fill_(4)
    assert D._sampling(1000, t, 1, False).temperature == 4.0
    for bad in ("0.5", b"0.5", None, 1j):
        with pytest.raises(TypeError):
            B.make_sampling(1000, bad, 0.9, False)
        with pytest.raises(TypeError):
            D._sampling(1000, bad, 0.9, False)
        with pytest.raises(TypeError):
            D._sampling(1000, 0.5, bad, False)


@pytest.mark.gpu
def test_settings_as_tensors_are_read_on_every_call():
    g = torch.Generator(device="cuda:0").manual_seed(3)
    logits = torch.randn(64, 500, generator=g, device="cuda:0")
    u = torch.rand(64, generator=g, device="cuda:0")
    t = torch.tensor(0.4)
    first = D.sample(logits, u, temperature=t)
    t.fill_(2.0)
    second = D.sample(logits, u, temperature=t)
    assert torch.equal(first, D.sample(logits, u, temperature=0.4))
    assert torch.equal(second, D.sample(logits, u, temperature=2.0)) and not torch.equal(first, second)


def test_stream_without_the_raw_handle(monkeypatch):
    """A torch build without the raw handle's name: the stream object's."""
    monkeypatch.setattr(D, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev: SimpleNamespace(cuda_stream=(77, dev)))
    assert D._stream(torch.device("cuda:1")) == (77, torch.device("cuda:1"))


@pytest.mark.gpu
@pytest.mark.parametrize("raw", [True, False], ids=["raw_handle", "stream_object"])
def test_stream_handles(raw, monkeypatch):
    if not raw:
        monkeypatch.setattr(D, "_raw_stream", None)
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            for dev in (torch.device("cuda:0"), torch.device("cuda"), "cuda:0", 0, None):
                assert D._stream(dev) == stream.cuda_stream


@pytest.mark.gpu
def test_losses_are_outputs_of_their_own():
    """The losses of two calls do not share memory, and dropping them frees the context."""
    import gc
    h = [torch.randn(130, 64, device="cuda:0").bfloat16().requires_grad_(True)]
    W = [torch.randn(300, 64, device="cuda:0").bfloat16().requires_grad_(True)]
    y = torch.randint(0, 300, (130,), device="cuda:0")
    a = D.distill(h, W, y)
    b = D.distill(h, W, y)
    assert all(p.data_ptr() != q.data_ptr() and torch.equal(p, q) for p, q in zip(a, b))
    a[0].sum().backward()
    del a, b
    h[0].grad = W[0].grad = None
    gc.collect()
    gc.disable()  # no cycle: the graph goes with its last reference
    try:
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        for _ in range(3):
            D.distill(h, W, y)
        assert torch.cuda.memory_allocated() == before
    finally:
        gc.enable()


def test_backward_takes_the_addresses_of_the_saved_tensors(monkeypatch):
    """Saved-tensor hooks may hand the backward other tensors than the forward saw."""
    old = [torch.zeros(4, 8) for _ in range(4)]
    p = B.make_problem(2, 4, 4, [8, 8], [x.data_ptr() for x in old[:2]], [x.data_ptr() for x in old[2:]],
                       torch.zeros(4, dtype=torch.int64).data_ptr(), dtype=B.MLS_F32, tau=1.5)
    y = torch.ones(4, dtype=torch.int64)
    new = [torch.ones(8, 4).t() if i == 1 else torch.ones(4, 8) for i in range(4)]  # one of other strides
    seen = []
    monkeypatch.setattr(D, "backward", lambda q, buf, dev, gc, gk, gh, gW: seen.append((q, gh, gW)))
    ctx = SimpleNamespace(saved_tensors=(y, *new), M=2, p=p, buf=None, needs_input_grad=[False, False] + [True] * 4)
    before = bytes(p)
    D._Distill.backward(ctx, None, None, None)
    (q, gh, gW), = seen
    assert q.labels == y.data_ptr() and q.h[0] == new[0].data_ptr()
    assert [q.W[0], q.W[1]] == [x.data_ptr() for x in new[2:]]
    assert q.h[1] not in (old[1].data_ptr(), new[1].data_ptr())  # a contiguous copy
    assert q.tau == 1.5 and bytes(p) == before
    assert all(g.is_contiguous() and g.shape == (4, 8) for g in gh + gW)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_gradients_with_saved_tensors_kept_on_the_host(dt):
    """The hidden states of the forward are given back and written over before the backward."""
    g = torch.Generator(device="cuda:0").manual_seed(5)
    W = [(torch.randn(700, d, generator=g, device="cuda:0") * 0.1).to(dt) for d in (64, 128)]
    h0 = [torch.randn(300, d, generator=g, device="cuda:0").to(dt) for d in (64, 128)]
    y = torch.randint(0, 700, (300,), generator=g, device="cuda:0")

    def grads(offload):
        leaves = [x.clone().requires_grad_(True) for x in h0 + W]
        mids = [x * 1.0 for x in leaves]  # not leaves: only the graph keeps them
        if offload:
            with torch.autograd.graph.save_on_cpu():
                ce, kl, _ = D.distill(mids[:2], mids[2:], y, tau=1.5)
        else:
            ce, kl, _ = D.distill(mids[:2], mids[2:], y, tau=1.5)
        loss = (ce + 0.5 * kl).sum()
        if offload:
            shapes = [x.shape for x in mids]
            del mids, ce, kl
            junk = [torch.full(s, float("nan"), device="cuda:0", dtype=dt) for s in shapes]
        loss.backward()
        return [x.grad for x in leaves]

    for a, b in zip(grads(False), grads(True)):
        assert torch.equal(a, b)
