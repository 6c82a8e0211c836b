"""GPU: W = 32 launches of unit pairs whose last pair has one unit."""

import numpy as np
import pytest

from tests.test_gpu_decode import _run_on_windows, _say, _syms, gpu_decode

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_12141_amd as m
    return m


def _odd():
    """The smallest odd number of W = 32 runs that a launch decodes in pairs."""
    return 16 * torch.cuda.get_device_properties(0).multi_processor_count + 1


def _pass_us(plan, passes=20):
    ws = plan.allocate_workspace()
    plan.upload(ws)
    out = plan.allocate_output()
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = float("inf")
    for _ in range(8):
        torch.cuda.synchronize()
        a.record()
        for _ in range(passes):
            plan.decode(ws, out, err)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / passes * 1e3)
    assert int(err.item()) == 0
    return best


@pytest.mark.parametrize("dt,n", [(np.uint8, 12), (np.uint16, 12), (np.uint8, 16)])
def test_a_unit_without_a_partner_keeps_the_pace(rc, dt, n):
    """One unit more than an even number costs no more than one unit: its predicated decode
    took 30 to 45 % longer than the whole launch of pairs. (The bound is halfway to that; one
    unit of 4099 is 0.02 %, and the times of the two launches differ by about 2 %.)"""
    A = 256 if dt == np.uint8 else 4096
    units = _odd() + 1
    plans = []
    for M in (units, units + 1):
        s = _syms(9100, M * 300 * 32, A, dt, 1.1)
        blob = rc.encode(s, lanes=32, quant_bits=n, splits=M, alphabet=A)
        assert blob.splits == M and rc.Plan(blob).shape().units_per_wave == 2
        plans.append(rc.Plan(blob))
    even, odd = (_pass_us(p) for p in plans)
    _say("case pace", np.dtype(dt).name, n, f"{units} units {even:.1f} us, {units + 1} units {odd:.1f} us")
    assert odd < 1.15 * even


@pytest.mark.parametrize("dt,n", [(np.uint8, 8), (np.uint8, 12), (np.uint16, 12), (np.uint8, 16), (np.uint16, 16)])
@pytest.mark.parametrize("groups", [1, 3, 29])
def test_odd_runs(rc, dt, n, groups):
    """Short and ordinary last units, full and ragged last groups, also in runs of several
    units, partitioned, and packed."""
    A = 200 if dt == np.uint8 else 4000
    M = _odd()
    for extra in (0, 1, 31):
        s = _syms(9200 + extra, M * groups * 32 + extra, A, dt, 1.1)
        _say("case odd runs", np.dtype(dt).name, n, groups, extra)
        blob = rc.encode(s, lanes=32, quant_bits=n, splits=M, alphabet=A)
        assert np.array_equal(gpu_decode(rc, blob), s)
        assert np.array_equal(gpu_decode(rc, rc.encode_partitioned(s, lanes=32, quant_bits=n, partitions=M, alphabet=A)), s)
    s = _syms(9300, (3 * M + 1) * groups * 32, A, dt, 1.1)
    blob = rc.encode(s, lanes=32, quant_bits=n, splits=3 * M + 1, alphabet=A)
    assert np.array_equal(gpu_decode(rc, blob, units_per_run=3), s)
    plan = rc.Plan(rc.encode(s, lanes=32, quant_bits=n, splits=M, alphabet=A), packed_target=0)
    ws = plan.allocate_workspace()
    plan.upload(ws)
    out = plan.allocate_output()
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    plan.decode(ws, out, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0 and np.array_equal(plan.symbols_of(out), s)


def test_odd_runs_write_counts(rc):
    """The unit without a partner stores each of its symbols once, and in its run-on window."""
    s = _syms(9400, _odd() * 40 * 32 + 5, 256, np.uint8, 1.1)
    blob = rc.encode(s, lanes=32, quant_bits=12, splits=_odd(), alphabet=256)
    plan = rc.Plan(blob)
    plan.set_tuning(chunk_groups=8, units_per_run=1)
    shape = plan.shape()
    assert shape.units_per_wave == 2 and shape.runs % 2
    ws = plan.allocate_workspace()
    plan.upload(ws)
    out = plan.allocate_output()
    counts = torch.zeros(len(s), dtype=torch.int32, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    plan.decode_count_writes(ws, out, counts, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0 and np.array_equal(plan.symbols_of(out), s)
    allowed = np.ones(-(-len(s) // 32), dtype=np.int64)
    for lo, hi in _run_on_windows(plan.units(), shape, 8):
        if hi >= lo:
            allowed[lo:hi + 1] += 1
    c = counts.cpu().numpy()
    assert c.min() >= 1 and np.all(c <= np.repeat(allowed, 32)[:len(s)])


@pytest.mark.parametrize("extra", [0, 7])
def test_odd_runs_adaptive(rc, extra):
    import synth
    N = _odd() * 29 * 32 + extra
    pmfs, tidx, s = synth.adaptive_stream(93, N)
    f = np.stack([rc.quantize(np.maximum(np.round(p * 65536), 1).astype(np.uint64), 9) for p in pmfs])
    blob = rc.encode_adaptive(s, f, tidx, lanes=32, quant_bits=9, splits=_odd(), alphabet=64)
    plan = rc.Plan(blob)
    assert plan.shape().units_per_wave == 2 and plan.shape().runs % 2
    ws = plan.allocate_workspace()
    plan.upload(ws)
    out = plan.allocate_output()
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    plan.decode_adaptive(ws, torch.from_numpy(tidx).cuda(), out, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0 and np.array_equal(plan.symbols_of(out), s)
