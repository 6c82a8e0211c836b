"""GPU: decodes of a little more than one run per SIMD, whose kernel depends on the runs' length
where the shape is left open."""

import numpy as np
import pytest

from tests.test_gpu_decode import _say, _syms, gpu_decode

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_12141_amd as m
    return m


@pytest.mark.parametrize("W,dt,n", [(32, np.uint8, 11), (32, np.uint16, 12), (32, np.uint8, 16), (32, np.uint16, 14),
                                    (64, np.uint8, 12), (64, np.uint16, 12), (64, np.uint8, 16), (64, np.uint16, 16)])
def test_short_runs(rc, W, dt, n):
    """Short runs go to 8-wave workgroups of the throughput kernel, no more of them than they
    fill, and long ones to a shared workgroup on every CU; exact on both sides of every line."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    M = 6 * cus - 36                   # 1500 runs on 256 CUs
    A = 256 if dt == np.uint8 else 4000
    s = _syms(9500, M * 160 * W, A, dt, 1.1)
    for groups in (2, 12, 20, 40, 70, 100, 160):
        t = s[:M * groups * W - 5 * groups]
        blob = rc.encode(t, lanes=W, quant_bits=n, splits=M, alphabet=A)
        sh = rc.Plan(blob).shape()
        _say("case short runs", W, np.dtype(dt).name, n, "groups", groups, "runs", sh.runs, "blocks", sh.blocks)
        assert sh.runs == blob.splits and (sh.waves_per_block, sh.units_per_wave) == (8, 1)
        if groups <= 12 and sh.runs > 5 * cus:     # (very short streams give fewer split points)
            assert sh.blocks == -(-sh.runs // 8)
        if groups == 160:
            assert sh.blocks == cus
        assert np.array_equal(gpu_decode(rc, blob), t)
