"""GPU: the work items that a batch is cut into when the tuning leaves the shape to its size,
for launches that hold two workgroups per CU and for those that hold one (large tables beside
large rings, or a cap), and of streams of several table classes."""

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


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def _streams(rc, count, units, n, A, dt, seed):
    out = []
    for i in range(count):
        s = _syms(seed + i, units * 160 + 37 * i, A, dt, 1.1)
        freq = rc.quantize(np.bincount(s, minlength=A).astype(np.uint64) + 1, n)   # every symbol has a table entry
        out.append((s, rc.encode(s, lanes=64 if i % 5 == 4 else 32, quant_bits=n, splits=units, alphabet=A, freq=freq)))
    return out


def _batch(rc, streams, waves, K, cap, pairs_per_wave=2, ru=0):
    from paper_2306_12141_amd import _lib
    from paper_2306_12141_amd.batch import Batch
    return Batch([b for _, b in streams], _lib.Tuning(waves, K, pairs_per_wave, cap, ru))


def _decodes(batch, streams):
    ws, out, err = batch.allocate()
    batch.upload(ws)
    for poison in (0x5A, 0xA5):
        out.fill_(poison)
        batch.decode(ws, out, err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        for i, (s, _) in enumerate(streams):
            assert np.array_equal(batch.symbols_of(out, i, s.dtype), s), i


# Workgroups per CU: two of 16 waves fill its wave slots; 64 KiB of rings and a 32 KiB table,
# a 48 KiB two-level table with 32 KiB of rings, or a cap leave one.
SHAPES = {
    "plain": (12, 256, np.uint8, 16, 4, 0, 2),
    "plain 8 waves": (12, 256, np.uint8, 8, 4, 0, 4),
    "capped": (12, 256, np.uint8, 16, 4, 1, 1),
    "capped 8 waves": (11, 256, np.uint8, 8, 4, 1, 1),
    "large tables and rings": (12, 3000, np.uint16, 16, 8, 0, 1),
    "full two-level tables": (16, 4096, np.uint16, 16, 4, 0, 1),
}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("load", [0.05, 0.4, 0.9, 1.7])
def test_items_fill_the_launch(rc, shape, load):
    """load: unit pairs for each pair of a launch of full items. Up to 1, every item has a
    workgroup of its own and most workgroups have one; above, items are full (the queue)."""
    n, A, dt, waves, K, cap, per_cu = SHAPES[shape]
    groups, per_item, count = per_cu * _cus(), 2 * waves, 12
    # (10 of 12 streams have W = 32, whose units go in pairs once half of the waves have one.)
    units = max(1, int(load * groups * per_item / count * (12 / 7 if load > 0.5 else 1)))
    streams = _streams(rc, count, units, n, A, dt, 8100)
    batch = _batch(rc, streams, waves, K, cap)
    _say("case items", shape, "load", load, "units", units, "items", batch.items, "workgroups", groups)
    if load < 1:
        assert groups / 2 < batch.items <= groups
    else:
        assert batch.items > 1.25 * groups
    _decodes(batch, streams)


def test_classes_of_one_batch(rc):
    """Streams of the three table classes: the launches come one after the other, so each is
    cut as if its streams were alone; classes that share a launch are cut together."""
    small = _streams(rc, 9, 60, 11, 256, np.uint8, 8300)     # two workgroups per CU also with 8-group rings
    large = _streams(rc, 7, 90, 12, 3000, np.uint16, 8400)
    wide = _streams(rc, 8, 70, 16, 4096, np.uint16, 8500)
    mixed = [x for t in zip(small, large, wide) for x in t] + small[7:] + wide[7:]
    for K in (4, 8):
        items = lambda streams: _batch(rc, streams, 16, K, 0).items
        both = _batch(rc, mixed, 16, K, 0)
        plain = items(small + large) if K == 4 else items(small) + items(large)
        _say("case classes", K, both.items, plain, items(wide))
        assert both.items == plain + items(wide)
        _decodes(both, mixed)


def test_every_tuning_fits_the_workspace(rc):
    """The workspace of one tuning holds the items of every other."""
    from paper_2306_12141_amd import _lib
    streams = _streams(rc, 5, 3, 12, 256, np.uint8, 8600) + _streams(rc, 3, 700, 11, 256, np.uint8, 8700) + \
        _streams(rc, 2, 9, 14, 256, np.uint8, 8800) + _streams(rc, 2, 130, 12, 3000, np.uint16, 8900)
    batch = _batch(rc, streams, 16, 8, 0, 64, 64)
    ws, out, err = batch.allocate()
    batch.upload(ws)
    for waves in (8, 16):
        for pairs in (1, 3, 64):
            for cap in (0, 1):
                for ru in (0, 1, 5):
                    _say("case tuning", waves, pairs, cap, ru)
                    batch.set_tuning(_lib.Tuning(waves, 4, pairs, cap, ru), ws)
                    out.fill_(0x5A)
                    batch.decode(ws, out, err)
                    torch.cuda.synchronize()
                    assert int(err.item()) == 0
                    for i, (s, _) in enumerate(streams):
                        assert np.array_equal(batch.symbols_of(out, i, s.dtype), s), i
