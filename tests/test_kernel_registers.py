"""Register budget of the eight-wave kernels (compiled here, no GPU needed): sixteen waves per compute unit leave 128 vector registers
each, and what does not fit goes to scratch memory inside the tile loops."""
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2603_08743_amd.build import CSRC, FLAGS

GROUPS = (0, 4, 7)


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    d = tmp_path_factory.mktemp("regs")

    def compile_one(key):
        ref, g = key
        src = d / ("k%d_%d.hip" % key)
        src.write_text('#include "%s/zp_mfma.h"\nnamespace zp { hipError_t f(const Args &a, hipStream_t s) {\n'
                       "return launch_one<1, 256, false, 1, 8, %d, %d, false>(a, 1, s); } }\n" % (CSRC, g, ref))
        r = subprocess.run(["hipcc", *FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", str(src), "-o", "/dev/null"],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]

    keys = [(ref, g) for ref in (0, 1, 3) for g in GROUPS]
    with ThreadPoolExecutor(4) as ex:
        return dict(zip(keys, ex.map(compile_one, keys)))


@pytest.mark.parametrize("ref", [0, 1, 3])
def test_eight_wave_kernels_spill_no_vector_register(spills, ref):
    """Plain, with global score and pooling, and with the separate redundancy pass (bf16 rows of 256 bytes)."""
    for g in GROUPS:
        assert spills[ref, g] and not any(spills[ref, g]), (ref, g, spills[ref, g])
