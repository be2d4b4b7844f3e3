"""Lightning redundancy of large blocks with the rows in LDS: more column groups than the waves hold at once, last row tiles and column
groups of every fill, long rows, workgroups with fewer query blocks than waves, zero entries below a negative threshold."""
import numpy as np
import pytest

from tests.test_gpu_extras import pick_threshold, plant_similar_keys, run_extras_protocol
from tests.util import random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,d,Gq,w,b,N_max,p_thr", [
    (True, 128, 4, 8, 300, 3, 0.4), (True, 128, 4, 64, 129, 3, 0.4), (True, 128, 4, 60, 288, 2, 0.4), (True, 64, 4, 16, 97, 4, 0.4), (True, 64, 5, 30, 36, 5, 0.4),
    (True, 192, 3, 9, 100, 3, 0.4), (True, 512, 2, 6, 130, 2, 0.4), (True, 128, 5, 100, 160, 3, 0.4),
    (False, 64, 2, 9, 98, 3, 0.4), (False, 256, 2, 9, 40, 4, 0.4), (False, 128, 4, 32, 140, 3, 0.4), (True, 128, 4, 16, 100, 3, -0.2),
])
def test_redundancy_of_large_blocks(bf16, d, Gq, w, b, N_max, p_thr):
    p = random_problem(1500 + b + d, B=2, L=1, h_kv=2, G=Gq, d=d, b=b, N_max=N_max, w=w, extra_blocks=1, bf16=bf16, heavy=4)
    rng = np.random.default_rng(b)
    N, budget = N_max + 1, (N_max - 1) * b
    vl = rng.integers(max(w - b, 0), (N - 1) * b + 1, size=(2, 1, 2)).astype(np.int32)
    vl[0, 0, 0], vl[1, 0, 1] = (N - 1) * b, b + 1                 # whole blocks, one live row in the second block
    cap = np.minimum(budget, vl + b)
    p.valid_len, p.keep = vl, (w + (rng.random(vl.shape) * (cap - w + 1)).astype(np.int32)).clip(w, cap).astype(np.int32)
    plant_similar_keys(p, rng, 60 + 4 * b, noise=0.1)
    p.K[:, :, 5] = 0                                              # keys of norm 0
    thr = pick_threshold(p, [p_thr + 1e-3 * i for i in range(1, 40)])
    rep = run_extras_protocol(p, dict(alpha=0.8, pool_kernel=5, lam=0.3, tau=0.02, p=thr), seed=b)
    assert rep["worst"] < 1e-3
