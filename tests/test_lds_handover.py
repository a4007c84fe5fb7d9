"""Hand-overs between the lanes of one wave through LDS, checked on the CPU from the kernels' source.  Lanes store pieces of
a buffer that other lanes read; no address of a single lane depends on that, so the compiler may exchange the two unless a
`wave_lds_fence` stands between them.  Required, over two steps in a row: between a store into a buffer and a read of other
lanes' bytes of it, and between such a read and the next store, there is a fence.  Accesses are taken in the order in which
they are written down (a lambda's stand where it is defined, right before its use)."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_19760_amd", "csrc")
FENCE = (r"wave_lds_fence\(\)", [("fence", None)])


def _source(name):
    return [line.split("//")[0] for line in open(os.path.join(CSRC, name)).read().split("\n")]


def _between(lines, first, last):
    a = next(i for i, l in enumerate(lines) if re.search(first, l))
    return lines[a:next(i for i in range(a + 1, len(lines)) if re.search(last, lines[i]))]


def _events(lines, rules, names=None):
    """[(what, buffer)] of the lines; a rule is (pattern, events), `$1` in a buffer's name is the pattern's group."""
    out = []
    for line in lines:
        hits = sorted((m.start(), k, m) for k, (pattern, _) in enumerate(rules) for m in re.finditer(pattern, line))
        for _, k, m in hits:
            for what, buffer in rules[k][1]:
                buffer = m.group(1) if buffer == "$1" else buffer
                out.append((what, (names or {}).get(buffer, buffer)))
    return out


def _check(step):
    open_accesses = set()
    for what, buffer in step + step:
        if what == "fence":
            open_accesses.clear()
            continue
        other = ("read", buffer) if what == "store" else ("store", buffer)
        assert other not in open_accesses, f"no fence between a {other[0]} and the next {what} of {buffer}"
        open_accesses.add((what, buffer))


def test_sampling_by_whole_texels():
    body = _between(_source("lp_gather.h"), r"void wave_features\(", r"^}")
    step = _events(body, [FENCE, (r"\bpublish_gather<", [("store", "records")]),
                          (r"\bwave_gather<", [("read", "records"), ("store", "image")]), (r"= lds_chunk\(", [("read", "image")])])
    assert {b for w, b in step if w == "read"} == {"records", "image"}
    _check(step)


@pytest.mark.parametrize("hidden_layers", [1, 2])
def test_step_of_the_tile_backward(hidden_layers):
    body = _between(_source("lp_mfma_bwd_tile.h"), r"^    while \(live\) \{", r"^    // ---- sums|^    constexpr int kRegs")
    if hidden_layers == 1:   # without the part between the output layer and the first one
        a = next(i for i, l in enumerate(body) if l.rstrip() == "        if constexpr (NH == 2) {")
        b = next(i for i in range(a, len(body)) if body[i].rstrip() == "        }")
        body = body[:a] + body[b:]
    two = hidden_layers == 2
    names = {"kHere": "B" if two else "A", "kLast": "B" if two else "A", "kZ": "A" if two else "B", "kF": "B" if two else "A",
             "L::A": "A", "L::B": "B"}
    area = r"(L::A|L::B|kHere|kLast|kZ|kF)\b"
    step = _events(body, [
        FENCE,
        (r"activate_pair\([^()]*, " + area, [("store", "$1")]),
        (r"store_hidden\(" + area, [("store", "$1")]),
        (r"lds_put_chunk\(.*\+ " + area, [("store", "$1")]),
        (r"lds_put<u32x4>\(dz_at", [("store", "output gradients")]),
        (r"lds_tr\(zp ", [("read", "output gradients")]),
        (r"lds_tr\(hp [^;]*?\+ " + area, [("read", "$1")]),
        (r"I(?:H|W1)::read\((?:col_h|col16_h|col_f)\b[^;]*?" + area, [("read", "$1")]),
        (r"lds_get<\w+>\(geo ", [("read", "rays")]),
        (r"lds_put<\w+>\(geo ", [("store", "rays")]),
        (r"lds_get<double>\(depth_at", [("read", "depths")]),
        (r"lds_put<double>\(depth_at", [("store", "depths")]),
        (r"\bload_rays\(\)", [("fence", None), ("store", "rays"), ("store", "depths"), ("fence", None)]),
        (r"\bscatter_step<", [("fence", None), ("store", "A"), ("fence", None), ("read", "A")]),
    ], names)
    assert {b for w, b in step if w == "read"} == {"A", "B", "output gradients", "rays", "depths"} == {b for w, b in step if w == "store"}
    _check(step)


@pytest.mark.parametrize("function", ["scatter_window", "scatter_walk"])
def test_scatter_begins_with_a_fence(function):
    """(As the check of the whole step assumes.)"""
    body = _between(_source("lp_tile_scatter.h"), r"void %s\(" % function, r"^}")
    lds = next(i for i, l in enumerate(body) if re.search(r"lds_put|lds_get|wave_lds_fence|write_scatter_record", l))
    assert "wave_lds_fence()" in body[lds]
