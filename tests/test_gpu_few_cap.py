"""GPU: a cap on resident workgroups holds for decodes with few runs, whichever kernel takes them."""

import numpy as np
import pytest

from tests.test_gpu_decode import _say, _syms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_12141_amd as m
    return m


# Runs at and around one, two and four workgroups of one run per CU, and two runs per SIMD.
@pytest.mark.parametrize("W,dt,n,runs_per_cu", [(32, np.uint8, 11, 0.25), (64, np.uint8, 12, 1), (32, np.uint16, 12, 1.1),
                                                (64, np.uint8, 16, 2), (32, np.uint8, 12, 4), (64, np.uint16, 12, 6)])
@pytest.mark.parametrize("waves", [0, 1, 8])
def test_cap_on_resident_workgroups(rc, W, dt, n, runs_per_cu, waves):
    """blocks_per_cu bounds the grid also where the waves of a workgroup are chosen at launch."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    M = int(runs_per_cu * cus)
    A = 256 if dt == np.uint8 else 4096
    s = _syms(6800 + M, 600_011, A, dt, 1.1)
    blob = rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A)
    for cap in (1, 2, 4):
        plan = rc.Plan(blob)
        plan.set_tuning(waves, 4, cap, 1)
        sh = plan.shape()
        _say("case cap", W, np.dtype(dt).name, n, M, "waves", waves, "cap", cap, "blocks", sh.blocks)
        assert sh.runs == blob.splits and sh.blocks <= cap * cus
        ws = plan.allocate_workspace()
        plan.upload(ws)
        out = plan.allocate_output()
        out.fill_(0x5A)
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        plan.decode(ws, out, err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        assert np.array_equal(plan.symbols_of(out), s)
