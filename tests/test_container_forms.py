"""Containers whose packed sections are not in their one canonical form.

A reader accepts set padding bits, a zero with its sign bit set and a series one bit
wider than it needs where the section's length stays the same, and holds all of them in
canonical form (least widths, no signed zero, zero padding); a form whose canonical
section is shorter is refused. The canonical section is kept as it arrived and the
others are packed again: both have to give the same container and the same records.
"""

import numpy as np
import pytest

import synth
from tests._fmt import BitReader, bits, parse, unit_records


@pytest.fixture(scope="module")
def rc():
    import paper_2306_12141_amd as m
    return m


CASES = [
    # lanes, n, dtype, alphabet, N, splits
    (32, 11, np.uint8, 256, 50_000, 40),
    (64, 12, np.uint16, 4096, 9_000, 7),
    (1, 8, np.uint8, 3, 4_000, 5),
    (3, 8, np.uint8, 5, 3_001, 9),
    (32, 12, np.uint8, 256, 1_392, 400),
    (32, 11, np.uint8, 256, 40_000, 1),
]


def _container(c, table, meta):
    """The container with other table and metadata bits (strings), zero-padded to bytes."""
    h = parse(c)
    raw = [int(s.ljust(-(-len(s) // 8) * 8, "0") or "0", 2).to_bytes(-(-len(s) // 8), "big") for s in (table, meta)]
    head = bytearray(c[:48])
    head[36:40] = len(raw[0]).to_bytes(4, "little")
    head[40:44] = len(raw[1]).to_bytes(4, "little")
    return bytes(head) + raw[0] + h["final"].tobytes() + raw[1] + h["words"].tobytes()


def _sections(c):
    """(table bits, metadata bits without their padding, [(bit, count, field, signed)] of its series)."""
    h = parse(c)
    t = BitReader(h["table"])
    t.series(h["alphabet"], 5, False)
    r, series = BitReader(h["meta"]), []
    for count, field, signed, states in ([(h["M"] - 1, 5, True, 0)] * 2 if h["M"] > 1 else []) + \
            [(h["lanes"], 4, False, h["lanes"])] * (h["M"] - 1):
        r.pos += 16 * states
        series.append((r.pos, count, field, signed))
        r.series(count, field, signed)
    return bits(h["table"], t.pos), bits(h["meta"], r.pos), series


def _wider(s, at, count, field, signed):
    """The series at bit `at` with every value one bit wider."""
    w = int(s[at:at + field], 2) + 1
    step = w + signed
    body = s[at + field:at + field + count * step]
    out = "".join(body[k:k + signed] + "0" + body[k + signed:k + step] for k in range(0, len(body), step))
    return s[:at] + format(w, f"0{field}b") + out + s[at + field + count * step:]


def _minus_zero(s, at, count, field):
    """The signed series at bit `at` with the sign of its first zero set, or None."""
    w = int(s[at:at + field], 2) + 1
    for k in range(count):
        p = at + field + k * (w + 1)
        if int(s[p + 1:p + 1 + w], 2) == 0:
            return s[:p] + "1" + s[p + 1:]
    return None


def _forms(c):
    """(name, container, bytes of its sections unchanged) for every other form of c."""
    table, meta, series = _sections(c)
    same = lambda a, b: -(-len(a) // 8) == -(-len(b) // 8)
    pad = lambda s: s + "1" * (-len(s) % 8)
    yield "canonical", _container(c, table, meta), True
    yield "table padding", _container(c, pad(table), meta), True
    yield "metadata padding", _container(c, table, pad(meta)), True
    wide = _wider(table, 0, parse(c)["alphabet"], 5, 0)
    yield "wider table", _container(c, wide, meta), same(wide, table)
    for i, (at, count, field, signed) in enumerate(series):
        if int(meta[at:at + field], 2) + 1 < (1 << field):
            wide = _wider(meta, at, count, field, int(signed))
            yield f"wider series {i}", _container(c, table, wide), same(wide, meta)
        signed_zero = _minus_zero(meta, at, count, field) if signed else None
        if signed_zero:
            yield f"minus zero {i}", _container(c, table, signed_zero), True


def _stream(rc, ci, seed=0):
    W, n, dt, A, N, M = CASES[ci]
    s = synth.draw_symbols(synth.zipf_pmf(A, 1.1), 900 + 10 * seed + ci, N, dt)
    return s, rc.encode(s, lanes=W, quant_bits=n, splits=M, alphabet=A)


@pytest.mark.parametrize("ci", range(len(CASES)))
def test_forms_read_as_canonical(rc, ci):
    """Every accepted form re-serialises to the canonical bytes, also after combining, and
    gives the records of the canonical stream; a longer section is refused."""
    seen = set()
    for seed in range(8):
        _, blob = _stream(rc, ci, seed)
        c = blob.to_bytes()
        for name, other, accepted in _forms(c):
            if not accepted:
                with pytest.raises(rc.RecoilError, match="corrupt"):
                    rc.Blob.from_bytes(other)
                seen.add("refused")
                continue
            b = rc.Blob.from_bytes(other)
            assert b.to_bytes() == c, name
            assert b.combine(3).to_bytes() == blob.combine(3).to_bytes(), name
            if CASES[ci][0] >= 32:
                assert np.array_equal(rc.Plan(b).units(), unit_records(c)[0]), name
            seen.add(name.rstrip(" 0123456789"))
    assert {"canonical", "table padding", "metadata padding", "refused"} <= seen


def test_forms_cover_signed_zero_and_same_length(rc):
    """The forms above hold a signed zero and a wider series of the same length."""
    names = {name.rstrip(" 0123456789") for ci in range(len(CASES)) for seed in range(8)
             for name, _, ok in _forms(_stream(rc, ci, seed)[1].to_bytes()) if ok}
    assert {"minus zero", "wider series"} <= names


@pytest.mark.gpu
@pytest.mark.parametrize("ci", [0, 1, 5])
def test_forms_packed_plan(rc, ci):
    """The device reads the section that a blob keeps: the packed plan of each form, kept
    as it arrived or packed again, decodes to the symbols."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests.test_gpu_unpack import _check
    s, blob = _stream(rc, ci)
    tried = {}
    for name, other, ok in _forms(blob.to_bytes()):
        if ok and tried.setdefault(name.rstrip(" 0123456789"), 0) < 2:
            tried[name.rstrip(" 0123456789")] += 1
            print(ci, name, flush=True)
            _check(rc, rc.Blob.from_bytes(other), s, [0, 5])
