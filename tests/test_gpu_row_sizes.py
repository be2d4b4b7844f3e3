"""Rows the matrix-core kernel pads (fp32, and bf16 of other sizes than 128 / 256 bytes): around every padded size, one and several
passes over the keys, windows at the edges of the wave counts, and sequences that leave no room for key tiles."""
import numpy as np
import pytest

from tests import gpu_util as G
from tests.util import random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,d,Gq,w,b,N_max", [
    (True, 8, 2, 5, 8, 9), (True, 56, 3, 9, 16, 5), (True, 72, 4, 8, 16, 7), (True, 96, 3, 20, 24, 6), (True, 104, 5, 7, 16, 6),
    (True, 136, 4, 17, 16, 6), (True, 192, 1, 33, 8, 12), (True, 200, 7, 10, 16, 5), (True, 256, 8, 40, 32, 4), (True, 264, 2, 16, 16, 4),
    (True, 512, 4, 12, 16, 4),
    (False, 4, 1, 3, 4, 5), (False, 60, 2, 16, 16, 5), (False, 64, 4, 33, 16, 8), (False, 68, 6, 6, 12, 7), (False, 128, 4, 32, 16, 9),
    (False, 132, 3, 12, 16, 5), (False, 256, 5, 31, 16, 4),
    (True, 96, 8, 130, 16, 12), (False, 32, 16, 20, 16, 6), (True, 128, 8, 600, 64, 11),   # 9 to 150 query blocks: several passes
])
def test_padded_rows(bf16, d, Gq, w, b, N_max):
    p = random_problem(700 + d + Gq, B=2, L=1, h_kv=2, G=Gq, d=d, b=b, N_max=N_max, w=w, extra_blocks=1, bf16=bf16, heavy=4)
    rng = np.random.default_rng(d)
    N, budget = N_max + 1, (N_max - 1) * b
    vl = rng.integers(max(w - b, 0), (N - 1) * b + 1, size=(2, 1, 2)).astype(np.int32)
    vl[0, 0, 0] = (N - 1) * b
    cap = np.minimum(budget, vl + b)
    p.valid_len, p.keep = vl, (w + (rng.random(vl.shape) * (cap - w + 1)).astype(np.int32)).clip(w, cap).astype(np.int32)
    pool, batch = G.to_device(p)
    rep = G.full_protocol(p, pool, batch)
    assert rep["worst_rel"] < 1e-3


@pytest.mark.parametrize("T", [31000, 32500])
def test_fp32_sequences_around_the_end_of_the_lds(T):
    """Two 64-key tiles of 256 padded bytes fit beside the scores of about 31500 positions; longer sequences take the vector-ALU kernel."""
    b = 250
    p = random_problem(800, B=1, L=1, h_kv=1, G=1, d=16, b=b, N_max=5, w=2, num_blocks=[T // b], heavy=2)
    pool, batch = G.to_device(p)
    rep = G.full_protocol(p, pool, batch)
    assert rep["worst_rel"] < 1e-3
