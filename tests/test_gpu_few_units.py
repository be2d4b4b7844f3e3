"""Calls of few units, which take three launches with several workgroups per unit: around the segment and tile edges of the split,
every wave geometry, stale gaps and shared workspaces; bit for bit what one launch gives."""
import numpy as np
import pytest
import torch

from paper_2603_08743_amd import binding
from tests import gpu_util as G
from tests.test_gpu_extras import pick_threshold, plant_similar_keys, run_extras_protocol
from tests.util import random_problem

pytestmark = pytest.mark.gpu


def problem(seed, bf16, d, Gq, w, b, N_max, extra=1, gaps=True, B=2, L=1):
    p = random_problem(seed, B=B, L=L, h_kv=2, G=Gq, d=d, b=b, N_max=N_max, w=w, extra_blocks=extra, bf16=bf16, heavy=4)
    rng = np.random.default_rng(seed)
    N, budget = N_max + extra, (N_max - 1) * b
    vl = np.full((B, L, 2), (N - 1) * b, dtype=np.int32)
    if gaps:
        vl = rng.integers(max(w - b, 0), (N - 1) * b + 1, size=vl.shape).astype(np.int32)
        vl[0, 0, 0] = (N - 1) * b
        vl[-1, 0, 1] = max(w - b, 0)                              # a single segment, whatever the others have
    cap = np.minimum(budget, vl + b)
    p.valid_len, p.keep = vl, (w + (rng.random(vl.shape) * (cap - w + 1)).astype(np.int32)).clip(w, cap).astype(np.int32)
    return p


def captured_scores(pool, batch):
    """The same call in a graph: one launch does the scoring."""
    ref, _, _ = G.alloc_outputs(pool, batch)
    G.ctx().zp_score(pool, batch, ref)                            # eager first, as a program calls it (several launches)
    torch.cuda.synchronize()
    ref.fill_(float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        G.ctx().zp_score(pool, batch, ref)
        assert G.ctx().zp_last_launches() == 1
    graph.replay()
    torch.cuda.synchronize()
    return ref


@pytest.mark.parametrize("bf16,d,Gq,w,b,N_max,split", [
    (True, 128, 4, 64, 16, 31, False), (True, 128, 4, 64, 16, 39, True), (True, 128, 4, 64, 16, 127, True),   # 512, 640 and 2048 positions: the line of eight waves
    (True, 128, 4, 64, 16, 128, True), (True, 128, 4, 8, 16, 31, True), (True, 128, 4, 8, 16, 30, False), (True, 128, 4, 8, 16, 63, True),
    (True, 128, 2, 16, 16, 40, True), (True, 128, 7, 32, 24, 30, True), (True, 128, 5, 128, 16, 66, True), (True, 128, 8, 128, 32, 20, True),  # 1, 8, 22 and 32 query blocks
    (True, 64, 4, 33, 16, 64, True), (True, 64, 5, 17, 8, 65, False), (True, 64, 5, 17, 8, 81, True),
    (True, 96, 3, 20, 24, 42, True), (True, 192, 4, 16, 16, 34, True), (False, 128, 4, 32, 16, 64, True), (False, 64, 1, 3, 16, 33, True),
    (False, 256, 2, 9, 12, 45, True),
])
def test_split_gives_the_bits_of_one_launch(bf16, d, Gq, w, b, N_max, split):
    p = problem(300 + d + w, bf16, d, Gq, w, b, N_max)
    pool, batch = G.to_device(p)
    scores, _, ln = G.alloc_outputs(pool, batch)
    G.ctx().zp_compress(G.clone_pool(pool), batch, ln)
    assert G.ctx().zp_last_launches() == (3 if split else 1)
    G.ctx().zp_score(pool, batch, scores)
    assert G.ctx().zp_last_launches() == (2 if split else 1)
    assert torch.equal(scores.view(torch.int32), captured_scores(pool, batch).view(torch.int32))
    rep = G.full_protocol(p, pool, batch)
    assert rep["worst_rel"] < 1e-3


@pytest.mark.parametrize("units", [63, 64, 65, 96, 127, 128, 129, 192, 193])
@pytest.mark.parametrize("d,w", [(128, 4), (64, 4)])
def test_unit_counts_around_the_rounds_of_row_moving_workgroups(units, d, w):
    """One, two or four row-moving workgroups per unit, up to the last split count and past it, against one launch (a captured call)."""
    p = random_problem(units + d, B=units, h_kv=1, G=4, d=d, b=16, N_max=33, w=w, bf16=True)
    rng = np.random.default_rng(units)
    p.valid_len = rng.integers(w, 32 * 16 + 1, size=(units, 1, 1)).astype(np.int32)
    p.keep = rng.integers(w, np.minimum(512, p.valid_len + 16) + 1).astype(np.int32)
    pool, batch = G.to_device(p)
    one, ln, one_ln = G.clone_pool(pool), *(torch.full((units, 1, 1), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        G.ctx().zp_compress(one, batch, one_ln)
        assert G.ctx().zp_last_launches() == 1
    graph.replay()
    G.ctx().zp_compress(pool, batch, ln)
    assert G.ctx().zp_last_launches() == (3 if units <= 192 else 1)
    torch.cuda.synchronize()
    assert torch.equal(ln, one_ln) and torch.equal(ln, batch.keep)
    assert torch.equal(pool.k.view(torch.int16), one.k.view(torch.int16)) and torch.equal(pool.v.view(torch.int16), one.v.view(torch.int16))


def test_more_streams_than_workspaces():
    """Six streams, each held back by a kernel of a few milliseconds, so that all their calls wait at once and share four workspaces."""
    c = G.ctx()
    jobs = []
    for i in range(6):
        pool, batch = G.to_device(problem(900 + i, True, 128, 4, 32, 16, 80 + 7 * i, B=8, L=2))
        expect = G.clone_pool(pool)
        elen = torch.empty((8, 2, 2), dtype=torch.int32, device="cuda")
        c.zp_compress(expect, batch, elen)
        jobs.append((pool, batch, torch.cuda.Stream(), torch.full_like(elen, -7), expect, elen))
    torch.cuda.synchronize()
    for _, _, stream, _, _, _ in jobs:
        with torch.cuda.stream(stream):
            torch.cuda._sleep(5_000_000)
    for pool, batch, stream, ln, _, _ in jobs:
        with torch.cuda.stream(stream):
            c.zp_compress(pool, batch, ln)
            assert c.zp_last_launches() == 3
    torch.cuda.synchronize()
    for pool, _, _, ln, expect, elen in jobs:
        assert torch.equal(ln, elen)
        assert torch.equal(pool.k.view(torch.int16), expect.k.view(torch.int16)) and torch.equal(pool.v.view(torch.int16), expect.v.view(torch.int16))


@pytest.mark.parametrize("what", ["slot", "block", "keep"])
def test_bad_unit_is_skipped_by_every_launch(what):
    p = problem(77, True, 128, 4, 32, 16, 40, gaps=False)
    pool, batch = G.to_device(p)
    before = G.clone_pool(pool)
    if what == "slot":
        batch.q_slot[0] = pool.q.shape[1]
    elif what == "block":
        batch.block_table[0, 3] = pool.k.shape[1]
    else:
        batch.keep[0] = 1
    ln = torch.full((2, 1, 2), -7, dtype=torch.int32, device="cuda")
    G.ctx().zp_compress(pool, batch, ln)
    assert G.ctx().zp_last_launches() == 3
    with pytest.raises(binding.ZpError):
        G.ctx().zp_sync_status()
    assert (ln[0] == -1).all() and torch.equal(ln[1], batch.keep[1])
    own = torch.from_numpy(p.block_table[0].astype(np.int64)).cuda()
    assert torch.equal(pool.k[:, own].view(torch.int16), before.k[:, own].view(torch.int16))
    assert torch.equal(pool.v[:, own].view(torch.int16), before.v[:, own].view(torch.int16))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Gq,w", [(3, 64), (4, 64), (5, 40), (7, 32), (8, 32)])
def test_redundancy_over_all_segments(Gq, w, d):
    """One launch with the similarity tiles from sweep 2 (eight waves) sums the same segments as the split calls it is checked against."""
    p = random_problem(40 + Gq + d, B=1, L=1, h_kv=2, G=Gq, d=d, b=16, N_max=130, w=w, bf16=True, heavy=4)
    plant_similar_keys(p, np.random.default_rng(Gq), 60, noise=0.1)
    thr = pick_threshold(p, [0.4, 0.41, 0.42, 0.43] if d == 128 else [0.6, 0.61, 0.62, 0.63])
    rep = run_extras_protocol(p, dict(alpha=0.8, pool_kernel=3, lam=0.3, tau=2e-3, p=thr), seed=Gq)
    assert rep["worst"] < 1e-3


@pytest.mark.parametrize("into", ["valid_len", "keep"])
def test_lengths_may_replace_valid_len_or_keep(into):
    """128 units: more row-moving workgroups than run at once, so late ones start after the first has written its unit's length."""
    p = problem(55, True, 128, 4, 32, 16, 64, B=16, L=4)
    pool, batch = G.to_device(p)
    expect = G.clone_pool(pool)
    elen = torch.empty((16, 4, 2), dtype=torch.int32, device="cuda")
    G.ctx().zp_compress(expect, batch, elen)
    G.ctx().zp_compress(pool, batch, getattr(batch, into))
    assert G.ctx().zp_last_launches() == 3
    G.ctx().zp_sync_status()
    assert torch.equal(getattr(batch, into), elen)
    assert torch.equal(pool.k.view(torch.int16), expect.k.view(torch.int16)) and torch.equal(pool.v.view(torch.int16), expect.v.view(torch.int16))


@pytest.mark.parametrize("bf16,d,Gq,w,b", [(False, 64, 2, 9, 16), (False, 128, 4, 32, 16), (True, 96, 3, 20, 24), (True, 192, 4, 64, 16)])
def test_refined_padded_rows_over_all_segments(bf16, d, Gq, w, b):
    """Padded rows: the refined call in one launch sums the segments of the split plain call it is checked against."""
    p = random_problem(60 + d + w, B=1, L=1, h_kv=2, G=Gq, d=d, b=b, N_max=2080 // b, w=w, bf16=bf16, heavy=4)
    plant_similar_keys(p, np.random.default_rng(d), 60, noise=0.1)
    thr = pick_threshold(p, [0.5, 0.51, 0.52, 0.53, 0.54, 0.55])
    rep = run_extras_protocol(p, dict(alpha=0.8, pool_kernel=3, lam=0.3, tau=2e-3, p=thr), seed=d)
    assert rep["worst"] < 1e-3
