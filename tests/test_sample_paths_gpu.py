"""GPU parity of the sampler's threshold search where its paths meet: nuclei at the
sizes of the list wave's runs and of the list, concentrated in one wave's range, made
of exact ties, and rows that are mostly impossible tokens; and of the verification
with more drafts than a wave has lanes. Against the float64 oracle, as in
test_decode_gpu."""

import numpy as np
import pytest
import torch

from oracle import decode as OD
from paper_2608_09703_amd import api as D
from tests.decode_checks import check_samples

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _sample(rows, u, temperature, top_p):
    logits = torch.tensor(np.asarray(rows, dtype=np.float32), device=DEV)
    ut = torch.tensor(u, dtype=torch.float32, device=DEV)
    tok = D.sample(logits, ut, temperature=temperature, top_p=top_p).cpu().numpy().astype(np.int64)
    return logits.double().cpu().numpy(), ut.double().cpu().numpy(), tok


@pytest.mark.parametrize("V", [3000, 16384, 49152, 65536])
def test_nucleus_sizes(V):
    """Leaders about 8 above the rest, their number around 64, 256 and 1,024, spread over
    the row or side by side (one wave's range of 1,024 to 4,096 tokens)."""
    rng = np.random.default_rng(V)
    rows = []
    for n in (1, 2, 63, 64, 65, 255, 257, 300, 1000, 1023, 1025, 1500):
        for side_by_side in (False, True):
            at = (rng.integers(0, V - n) + np.arange(n)) if side_by_side else rng.permutation(V)[:n]
            row = rng.standard_normal(V) - 12.0
            row[at] = rng.standard_normal(n) * 0.7
            rows.append(row)
    print(f"[decode] nucleus sizes V={V} rows={len(rows)}", flush=True)
    for top_p in (0.9, 0.99):
        u = rng.random(len(rows))
        check_samples(*_sample(rows, u, 1.0, top_p), 1.0, top_p)


@pytest.mark.parametrize("n", [40, 700, 2000])
def test_ties_and_impossible_tokens(n):
    """n exactly tied leaders cut by the nucleus (lower indices kept), every other token
    impossible or far below; the kept number is exact in both precisions."""
    V = 5000
    rng = np.random.default_rng(n)
    at = np.sort(rng.permutation(V)[:n])
    for fill in (-np.inf, -40.0):
        row = np.full(V, fill)
        row[at] = 1.5
        for top_p in (0.25 + 0.3 / n, 0.75 + 0.3 / n):
            u = np.array([0.0, 0.1, 0.37, 0.62, 0.99])
            lg, uu, tok = _sample(np.tile(row, (len(u), 1)), u, 1.0, top_p)
            keep = at[:int(np.ceil(top_p * n))]
            assert set(tok) <= set(keep)
            want = keep[np.minimum((uu * len(keep)).astype(np.int64), len(keep) - 1)]
            # a draw within fp32 rounding of a token's edge may fall to its neighbour
            edge = np.abs(uu * len(keep) - np.round(uu * len(keep))) < 1e-3
            assert np.array_equal(tok[~edge], want[~edge])


def test_verify_more_drafts_than_lanes():
    """70 drafts; equal distributions keep every draft until the step where the
    verifier finds the drafted token impossible."""
    G, V = 70, 200
    steps = [0, 1, 63, 64, 65, 69, 70]
    B = len(steps)
    rng = np.random.default_rng(7)
    dl = rng.standard_normal((G, B, V)).astype(np.float32)
    drafts = dl.argmax(axis=2).astype(np.int32)
    tl = np.concatenate([dl.transpose(1, 0, 2), rng.standard_normal((B, 1, V)).astype(np.float32)], axis=1)
    for b, r in enumerate(steps):
        if r < G:
            tl[b, r, drafts[r, b]] = -60.0
    ua = rng.random((G, B)).astype(np.float32) * 0.99
    us = rng.random(B).astype(np.float32)
    t = lambda x: torch.tensor(np.ascontiguousarray(x), device=DEV)
    n, nxt = D.spec_verify(t(dl), t(tl), t(drafts), t(ua), t(us), temperature=1.0, top_p=0.9)
    rn, rx = OD.verify(dl.transpose(1, 0, 2).astype(np.float64), tl.astype(np.float64), drafts.T,
                       ua.T.astype(np.float64), us.astype(np.float64), 1.0, 0.9)
    assert np.array_equal(n.cpu().numpy(), steps) and np.array_equal(rn, steps)
    assert np.array_equal(nxt.cpu().numpy(), rx)
