"""Lightning redundancy in blocks that do not divide 32: around the 32-row tiles and the 64-row passes, whole and partly live, both
element types, rows whose fragments fit the registers and longer ones, one to eight waves, many zeroed entries per row."""
import numpy as np
import pytest

from tests.test_gpu_extras import pick_threshold, plant_similar_keys, run_extras_protocol
from tests.util import random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,d,Gq,w,b,N_max", [
    (True, 128, 4, 8, 24, 5), (True, 128, 4, 16, 33, 4), (True, 128, 4, 64, 48, 4), (True, 64, 2, 8, 31, 5), (True, 128, 2, 5, 65, 3),
    (True, 128, 5, 100, 96, 4), (True, 128, 4, 16, 256, 3), (True, 64, 8, 40, 127, 3), (True, 96, 3, 9, 40, 4), (True, 512, 2, 6, 40, 3),
    (False, 64, 2, 9, 24, 4), (False, 16, 1, 3, 5, 4), (False, 128, 3, 12, 70, 3),
])
def test_redundancy_of_other_block_sizes(bf16, d, Gq, w, b, N_max):
    p = random_problem(1200 + b + d, B=2, L=1, h_kv=2, G=Gq, d=d, b=b, N_max=N_max, w=w, extra_blocks=1, bf16=bf16, heavy=4)
    rng = np.random.default_rng(b)
    N, budget = N_max + 1, (N_max - 1) * b
    vl = rng.integers(max(w - b, 0), (N - 1) * b + 1, size=(2, 1, 2)).astype(np.int32)
    vl[0, 0, 0] = (N - 1) * b
    cap = np.minimum(budget, vl + b)
    p.valid_len, p.keep = vl, (w + (rng.random(vl.shape) * (cap - w + 1)).astype(np.int32)).clip(w, cap).astype(np.int32)
    plant_similar_keys(p, rng, 60 + 4 * b, noise=0.1)
    thr = pick_threshold(p, [0.4, 0.41, 0.42, 0.43, 0.44, 0.45])
    rep = run_extras_protocol(p, dict(alpha=0.8, pool_kernel=5, lam=0.3, tau=0.02, p=thr), seed=b)
    assert rep["worst"] < 1e-3


@pytest.mark.parametrize("p_thr", [-0.5, 0.0])
def test_zero_entries_count_below_a_negative_threshold(p_thr):
    p = random_problem(1300, B=1, L=1, h_kv=2, G=2, d=64, b=40, N_max=4, w=4, extra_blocks=1, bf16=True, heavy=2)
    p.valid_len = np.array([[[150, 83]]], dtype=np.int32)
    p.keep = np.array([[[100, 60]]], dtype=np.int32)
    thr = pick_threshold(p, [p_thr - 1e-3 * i for i in range(1, 40)])
    run_extras_protocol(p, dict(use_F=False, lam=0.3, tau=0.05, p=thr), seed=3)
