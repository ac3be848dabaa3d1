"""The end of an update runs as one block of the next update's column or class pass.  Its
thread writes the solver state while the other blocks run, so no kernel with such a block may
read a field that vol_finish writes: each wave would read it at its own time, and the waves of
a block could part ways at its barriers.  Checked on the sources."""
import os
import re

from paper_2503_13802_amd import build

CSRC = os.path.join(build.PKG, "csrc")


def _sources():
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hpp", ".hip")):
            yield f, re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())


def _body(txt, start):
    """Text of the braces that open at or after start."""
    i = txt.index("{", start)
    depth, j = 0, i
    while True:
        depth += {"{": 1, "}": -1}.get(txt[j], 0)
        j += 1
        if not depth:
            return txt[i:j]


def test_passes_beside_a_finish_read_nothing_it_writes():
    txt = dict(_sources())
    head = re.search(r"__device__[^;{]*\bvol_finish\(", txt["kernels.hpp"])
    written = set(re.findall(r"st->(\w+)\s*=[^=]", _body(txt["kernels.hpp"], head.end())))
    assert {"done", "k", "last_k"} <= written and "skip" not in written
    seen = 0
    for name, t in txt.items():
        for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\(", t):
            body = _body(t, m.end())
            if "vol_finish<" not in body or "fin" not in re.findall(r"\w+", t[m.start():t.index("{", m.end())]):
                continue
            seen += 1
            read = set(re.findall(r"st->(\w+)", body))
            assert not read & written, (name, m.group(1), read & written)
            assert "solve_over(vd, fin)" in body, (name, m.group(1))
    assert seen == 3      # compile-time and run-time column pass, class pass
    over = _body(txt["kernels.hpp"], re.search(r"\bsolve_over\(", txt["kernels.hpp"]).end())
    assert "fin ? &st->skip : &st->done" in over
