"""The decoder's read step is inline assembly that reads the LDS ring, and the ring is filled
by plain C++ stores: the language orders the two only where an assembly statement with a
"memory" clobber stands between them. Checked on the source, since a compiler is free to
produce the right order without it."""

import os
import re

import pytest

DEVICE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_12141_amd", "csrc", "device")


def _source(name):
    with open(os.path.join(DEVICE, name)) as fh:
        return re.sub(r"//.*", "", fh.read())


def _body(text, head):
    """The braces' contents of the one function whose declaration matches head."""
    found = list(re.finditer(head + r"[^;{]*\{", text))
    assert len(found) == 1, head
    at, depth = found[0].end(), 1
    while depth:
        depth += {"{": 1, "}": -1}.get(text[at], 0)
        at += 1
    return text[found[0].end():at - 1]


def test_ring_stores_are_ordered_with_the_read_step():
    text = _source("decode_core.hpp")
    assert re.search(r'void order\(\)\s*\{\s*asm volatile\(""\s*:::\s*"memory"\);\s*\}', text)
    for head in (r"inline void fill\(", r"inline bool super_step\("):
        body = _body(text, head)
        steps = re.findall(r"\b(put_chunk|groups<MODE>|order)\(", body)
        assert "put_chunk" in steps
        last = None
        for s in steps + ["groups<MODE>"]:     # (what follows reads the ring)
            assert not (s == "groups<MODE>" and last == "put_chunk"), (head, steps)
            assert not (s == "put_chunk" and last == "groups<MODE>"), (head, steps)
            last = s
    # Nothing else fills the ring.
    assert len(re.findall(r"\bput_chunk\(", text)) == 3


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(DEVICE) if f.endswith((".hip", ".hpp"))))
def test_other_lds_assembly_has_the_clobber(name):
    text = _source(name)
    if name == "decode_core.hpp":
        text = text.replace(_body(text, r"inline void read_step\("), "")
        text = re.sub(r"#define RECOIL_READ_\w+\s*\\\n(?:.*\\\n)*.*", "", text)
    for m in re.finditer(r"\basm\b[^;]*;", text):
        if re.search(r"\bds_\w+|s_barrier|s_waitcnt", m.group()):
            assert '"memory"' in m.group(), m.group()
