"""GPU parity of decodes with few runs (one run per workgroup, the bitstream ring holding
words already looked up). Integer path: exact, into buffers pre-filled with two patterns."""

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


def _simds():
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


# Lengths around the super-steps of a run (8 groups; 16 from 256 groups per run on; 4 where
# 8-group rings do not fit the LDS of a CU's runs), ragged last groups, one run, and as many
# runs as the chip has SIMDs.
@pytest.mark.parametrize("W,dt,n,N,M", [
    (32, np.uint8, 11, 31, 1), (32, np.uint8, 8, 32 * 255 + 5, 1), (32, np.uint8, 12, 32 * 256, 1),
    (64, np.uint8, 12, 64 * 4 * 256 - 1, 4), (64, np.uint8, 9, 64 * 4 * 256 + 1, 4),
    (32, np.uint8, 12, 600_011, 3), (64, np.uint16, 12, 600_011, 3), (32, np.uint16, 12, 1_000_003, 700),
    (64, np.uint16, 13, 400_009, 5), (32, np.uint8, 16, 700_001, 6), (64, np.uint8, 14, 700_001, 900),
    (64, np.uint8, 12, 2_000_003, 1000), (32, np.uint8, 12, 2_000_003, 1024), (64, np.uint16, 12, 2_000_003, 1024)])
def test_few_runs(rc, W, dt, n, N, M):
    _say("case few runs", W, np.dtype(dt).name, n, N, M)
    A = 256 if dt == np.uint8 else 4096
    s = _syms(6100 + M, N, A, dt, 1.1)
    blob = rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A)
    sh = rc.Plan(blob).shape()
    assert sh.runs == blob.splits <= _simds()
    assert (sh.blocks, sh.waves_per_block, sh.units_per_wave) == (sh.runs, 1, 1)
    assert np.array_equal(gpu_decode(rc, blob), s)
    for k in (2, 3):
        assert np.array_equal(gpu_decode(rc, blob, units_per_run=k), s)
    for P in (1, min(M, 7)):
        part = rc.encode_partitioned(s, lanes=W, quant_bits=n, partitions=P, alphabet=A)
        assert np.array_equal(gpu_decode(rc, part), s)


@pytest.mark.parametrize("W,dt,n,A", [(32, np.uint8, 12, 256), (64, np.uint8, 16, 256), (32, np.uint16, 12, 4095),
                                      (64, np.uint16, 16, 4096)])
@pytest.mark.parametrize("M", [1, 60])
def test_few_runs_word_rate(rc, W, dt, n, A, M):
    """Symbols of f = 1 take n bits each (at n = 16 every lane reads a word in every group, the
    most the ring has to supply) and alternate with stretches of one frequent symbol that
    hardly reads at all, in blocks of every length against the ring's chunks."""
    _say("case word rate", W, np.dtype(dt).name, n, A, M)
    f = np.ones(A, dtype=np.uint32)
    f[0] = (1 << n) - (A - 1)
    s = _syms(6300, 40_000 * M + 17, A, dt)
    at = 0
    for i, gap in enumerate(_syms(6301, 4 * M, 9_000, np.uint16)):
        at += 2_000 + 1_000 * i
        s[at:at + int(gap)] = 0
        at += int(gap)
    blob = rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A, freq=f)
    assert np.array_equal(gpu_decode(rc, blob), s)



@pytest.mark.parametrize("W,dt,n,A,M,groups", [
    (32, np.uint8, 11, 256, 300, 150), (64, np.uint8, 12, 256, 800, 130), (32, np.uint16, 12, 4095, 1000, 255),
    (64, np.uint16, 16, 4096, 900, 90), (64, np.uint8, 12, 256, 500, 300), (64, np.uint8, 12, 256, 1500, 70),
    (64, np.uint16, 11, 2047, 1027, 260)])
def test_few_runs_supply(rc, W, dt, n, A, M, groups):
    """The ring is filled by a second wave, told after each super-step of 4, 8 or 16 groups
    what is left: runs that read a word in almost every lane of every group, hardly any, and
    both in turn, next to one another in one launch."""
    _say("case supply", W, np.dtype(dt).name, n, A, M, groups)
    f = np.ones(A, dtype=np.uint32)
    f[0] = (1 << n) - (A - 1)
    s = _syms(6350, M * groups * W + 5, A, dt).reshape(-1)
    i = np.arange(s.size) // W
    s[(i // (3 * groups)) % 3 == 0] = 0                # whole runs without a word
    s[((i // (3 * groups)) % 3 == 1) & (i // 11 % 2 == 0)] = 0
    blob = rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A, freq=f)
    sh = rc.Plan(blob).shape()
    assert sh.waves_per_block == (1 if M <= _simds() else 8) and sh.runs <= 2 * _simds()
    assert np.array_equal(gpu_decode(rc, blob), s)


@pytest.mark.parametrize("W,dt,n,N,M", [
    (32, np.uint8, 12, 3_000_017, 1500), (32, np.uint8, 9, 64 * 2048 * 40, 1025), (64, np.uint16, 12, 3_000_003, 2048),
    (64, np.uint8, 16, 4_000_001, 1100), (32, np.uint8, 11, 1025 * 32 * 300, 1025)])
def test_two_runs_per_simd(rc, W, dt, n, N, M):
    """More runs than SIMDs and up to twice as many: one workgroup per CU, eight runs in
    each, some with waves that have none."""
    _say("case two runs per SIMD", W, np.dtype(dt).name, n, N, M)
    A = 256 if dt == np.uint8 else 4096
    s = _syms(6500 + M, N, A, dt, 1.1)
    blob = rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A)
    sh = rc.Plan(blob).shape()
    assert sh.runs == blob.splits and _simds() < sh.runs <= 2 * _simds()
    assert (sh.blocks, sh.waves_per_block, sh.units_per_wave) == (_simds() // 4, 8, 1)
    assert np.array_equal(gpu_decode(rc, blob), s)
    part = rc.encode_partitioned(s, lanes=W, quant_bits=n, partitions=M, alphabet=A)
    assert np.array_equal(gpu_decode(rc, part), s)


@pytest.mark.parametrize("dt,n", [(np.uint8, 12), (np.uint16, 12), (np.uint8, 16)])
def test_pairs_from_half_the_wave_slots(rc, dt, n):
    """W = 32: one unit per wave up to 16 waves per CU, pairs beyond, exact on both sides."""
    A = 256 if dt == np.uint8 else 4096
    s = _syms(6600, 3_000_017, A, dt, 1.1)
    slots = 4 * _simds()
    for M, per_wave in ((slots, 1), (slots + 1, 2), (slots + 2, 2)):
        _say("case pairs", np.dtype(dt).name, n, M)
        blob = rc.encode(s, lanes=32, quant_bits=n, splits=M, alphabet=A)
        assert blob.splits == M and rc.Plan(blob).shape().units_per_wave == per_wave
        assert np.array_equal(gpu_decode(rc, blob), s)
        assert np.array_equal(gpu_decode(rc, rc.encode_partitioned(s, lanes=32, quant_bits=n, partitions=M, alphabet=A)), s)


@pytest.mark.parametrize("W,N,M", [(32, 32 * 4 * 7 + 3, 1), (32, 400_003, 40), (64, 400_001, 40), (32, 3_000_019, 5000),
                                   (64, 3_000_001, 3000)])
def test_adaptive_index_blocks(rc, W, N, M):
    """Table indices are read four groups at a time: lengths around the blocks, one unit, one
    unit and a pair per wave, an index array that starts at an odd address."""
    import synth
    _say("case adaptive index blocks", W, N, M)
    pmfs, tidx, s = synth.adaptive_stream(66, N)
    f = np.stack([rc.quantize(np.maximum(np.round(p * 65536), 1).astype(np.uint64), 9) for p in pmfs])
    blob = rc.encode_adaptive(s, f, tidx, lanes=W, quant_bits=9, splits=M, alphabet=64)
    plan = rc.Plan(blob)
    ws = plan.allocate_workspace()
    plan.upload(ws)
    buf = torch.zeros(N + 64, dtype=torch.uint8, device="cuda")
    for off in (0, 1, 3):
        index = buf[off:off + N]
        index.copy_(torch.from_numpy(tidx))
        for poison in (0x5A, 0xA5):
            out = plan.allocate_output()
            out.fill_(poison)
            err = torch.zeros(1, dtype=torch.int32, device="cuda")
            plan.decode_adaptive(ws, index, out, err)
            torch.cuda.synchronize()
            assert int(err.item()) == 0 and np.array_equal(plan.symbols_of(out), s)


@pytest.mark.parametrize("W,dt,n,M", [(32, np.uint8, 11, 300), (64, np.uint16, 12, 1500), (64, np.uint8, 16, 1100)])
def test_tuned_waves(rc, W, dt, n, M):
    """One or eight waves asked for: the kernel for few runs where that is its shape, the
    throughput kernel otherwise and under a cap on resident workgroups; 16 keeps the latter."""
    _say("case tuned waves", W, np.dtype(dt).name, n, M)
    A = 256 if dt == np.uint8 else 4096
    s = _syms(6700 + M, 2_000_011, A, dt, 1.1)
    blob = rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A)
    cus = _simds() // 4
    for waves in (1, 8, 16):
        for cap in (0, 1):
            for k in (4, 8):
                plan = rc.Plan(blob)
                plan.set_tuning(waves, k, cap, 1)
                sh = plan.shape()
                assert sh.runs == blob.splits and sh.waves_per_block == waves
                if waves == 8 and cap == 0 and blob.splits > 4 * cus:
                    assert sh.blocks == cus
                ws = plan.allocate_workspace()
                plan.upload(ws)
                out = plan.allocate_output()
                out.fill_(0x5A)
                err = torch.zeros(1, dtype=torch.int32, device="cuda")
                plan.decode(ws, out, err)
                torch.cuda.synchronize()
                assert int(err.item()) == 0
                assert np.array_equal(plan.symbols_of(out), s)
