"""Hand-overs between the lanes of one wave through LDS, checked on the CPU from the kernels' source.  Lanes store pieces of
a buffer that other lanes read; no address of a single lane depends on that, so the compiler may exchange the two unless a
`wave_lds_fence` stands between them.  Required, over two steps in a row: between a store into a buffer and a read of other
lanes' bytes of it, and between such a read and the next store, there is a fence.  Accesses are taken in the order in which
they are written down (a lambda's stand where it is defined, right before its use)."""
import os
import re

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
