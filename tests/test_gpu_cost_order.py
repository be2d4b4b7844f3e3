"""Launches of more units than run at once, with heads of different lengths: the workgroups take the costliest units first, and every unit
is done once, with the bits that units in order of their number give (zp_compress_static never changes the order)."""
import numpy as np
import pytest
import torch

from paper_2603_08743_amd import binding
from tests import gpu_util as G
from tests.util import random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("units,d,Gq,w,ragged", [
    (257, 64, 4, 112, "live"), (511, 64, 5, 100, "live"), (1024, 64, 4, 112, "live"),     # several query blocks per wave: 256 workgroups at once
    (513, 64, 4, 64, "live"), (1023, 64, 4, 64, "live"), (700, 64, 4, 64, "same"),        # eight waves, one block each: 512 at once
])
def test_costliest_first_gives_the_bits_of_the_plain_order(units, d, Gq, w, ragged):
    p = random_problem(units + w, B=units, h_kv=1, G=Gq, d=d, b=16, N_max=64, w=w, bf16=True)
    rng = np.random.default_rng(units)
    if ragged == "live":
        p.valid_len = rng.integers(w, 63 * 16 + 1, size=(units, 1, 1)).astype(np.int32)
    else:                                                         # nearly one class of cost
        p.valid_len = np.full((units, 1, 1), 500, dtype=np.int32)
    p.keep = rng.integers(w, np.minimum(63 * 16, p.valid_len + 16) + 1).astype(np.int32)
    pool, batch = G.to_device(p)
    ref, ref_len = G.clone_pool(pool), torch.full((units, 1, 1), -7, dtype=torch.int32, device="cuda")
    binding.zp_compress_static(ref, batch, ref_len)
    for into in ("own", "valid_len"):              # the lengths may replace the array they come from
        out = G.clone_pool(pool)
        ln = torch.full_like(ref_len, -7) if into == "own" else getattr(batch, into)
        G.ctx().zp_compress(out, batch, ln)
        G.ctx().zp_sync_status()
        assert torch.equal(ln, ref_len)
        assert torch.equal(out.k.view(torch.int16), ref.k.view(torch.int16)) and torch.equal(out.v.view(torch.int16), ref.v.view(torch.int16))


def test_a_unit_with_a_bad_length_is_skipped_alone():
    p = random_problem(5, B=300, h_kv=1, G=4, d=64, b=16, N_max=64, w=112, bf16=True)
    p.valid_len = np.random.default_rng(5).integers(112, 63 * 16 + 1, size=(300, 1, 1)).astype(np.int32)
    p.keep = (p.valid_len // 2 + 64).clip(112, p.valid_len).astype(np.int32)
    pool, batch = G.to_device(p)
    for bad in (-5, 1 << 30):
        vl = p.valid_len.copy()
        vl[123] = bad
        batch.valid_len = G.dev_i32(vl)
        out, ref = G.clone_pool(pool), G.clone_pool(pool)
        ln, ref_len = (torch.full((300, 1, 1), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        binding.zp_compress_static(ref, batch, ref_len)
        G.ctx().zp_compress(out, batch, ln)
        with pytest.raises(binding.ZpError):
            G.ctx().zp_sync_status()
        assert ln[123].item() == -1 and torch.equal(ln, ref_len)
        assert torch.equal(out.k.view(torch.int16), ref.k.view(torch.int16)) and torch.equal(out.v.view(torch.int16), ref.v.view(torch.int16))
