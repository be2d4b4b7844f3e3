"""Selection by histograms of the key range: score distributions that take every exit (one bin kept whole, equal keys in the last bin, the
window alone, scores of -inf among the kept), any bits as scores, run ends inside a wave, in the many-unit and the few-unit kernel."""
import numpy as np
import pytest
import torch

import oracle
from tests import gpu_util as G
from tests.util import random_problem

pytestmark = pytest.mark.gpu


def scores_of(kind, rng, shape):
    if kind == "bits":                                            # every pattern, NaN and infinities among them
        return rng.integers(0, 1 << 32, size=shape, dtype=np.uint64).astype(np.uint32).view(np.float32)
    if kind == "narrow":                                          # neighbours in the last bits
        return (np.float32(1.0).view(np.uint32) + rng.integers(0, 300, size=shape)).astype(np.uint32).view(np.float32)
    if kind == "clustered":                                       # a cluster of near ties far below a few outliers: three rounds and more
        s = (np.float32(1e-3).view(np.uint32) + rng.integers(0, 70000, size=shape)).astype(np.uint32).view(np.float32)
        s[rng.random(shape) < 0.01] = 1e30
        s[rng.random(shape) < 0.01] = -1e30
        return s
    if kind == "few":                                             # finite scores fewer than the keep count asks for
        s = np.full(shape, -np.inf, dtype=np.float32)
        s[rng.random(shape) < 0.05] = 0.25
        return s
    if kind == "denormal":
        return rng.integers(0, 5000, size=shape).astype(np.uint32).view(np.float32) * rng.choice([-1, 1], size=shape).astype(np.float32)
    return np.exp(rng.standard_normal(shape)).astype(np.float32)


@pytest.mark.parametrize("B", [8, 200])                           # one selecting workgroup of sixteen waves per unit, and of four
@pytest.mark.parametrize("kind", ["bits", "narrow", "clustered", "few", "denormal", "plain"])
@pytest.mark.parametrize("b,N_max,extra", [(4, 9, 2), (16, 64, 1), (24, 43, 3)])
def test_selection_rounds(kind, b, N_max, extra, B):
    w = 5
    p = random_problem(B + b, B=B, d=8, b=b, N_max=N_max, w=w, extra_blocks=extra)
    rng = np.random.default_rng(b + N_max)
    shape = (B, 1, 1)
    p.valid_len = rng.integers(w, (N_max + extra - 1) * b + 1, size=shape).astype(np.int32)
    p.valid_len[0] = (N_max + extra - 1) * b
    cap = np.minimum((N_max - 1) * b, p.valid_len + b)
    p.keep = rng.integers(w, cap + 1).astype(np.int32)
    p.keep[1], p.keep[2], p.keep[0] = w, cap[2], cap[0]           # the window alone, as many as there are
    S = scores_of(kind, rng, (B, 1, 1, (N_max + extra) * b))
    want_idx, want_len = oracle.select(p, S)
    pool, batch = G.to_device(p)
    _, idx, ln = G.alloc_outputs(pool, batch)
    G.ctx().zp_select_topk(torch.from_numpy(S).cuda(), pool, batch, idx, ln)
    G.ctx().zp_sync_status()
    assert np.array_equal(ln.cpu().numpy(), want_len) and np.array_equal(idx.cpu().numpy(), want_idx)
