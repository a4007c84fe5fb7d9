"""Hand-overs between the lanes of one wave through LDS, checked on the CPU from the kernels' source.  Lanes store pieces of
a buffer that other lanes read; no address of a single lane depends on that, so the compiler may exchange the two unless a
`wave_lds_fence` stands between them.  Required, over two steps in a row: between a store into a buffer and a read of other
lanes' bytes of it, and between such a read and the next store, there is a fence (also from what stands before the loop).  Accesses are taken in the order in which
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


def _check(step, before=()):
    open_accesses = set()
    for what, buffer in [*before, *step, *step]:
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
    """The first rays are loaded in front of the loop, the next ones inside of it, through the bytes of a step tensor."""
    source = _source("lp_mfma_bwd_tile.h")
    load = _between(source, r"^    auto load_rays = ", r"^    };")
    body = _between(source, r"^    while \(live\) \{", r"^    // ---- sums|^    constexpr int kRegs")
    if hidden_layers == 1:   # without the part between the output layer and the first one
        a = next(i for i, l in enumerate(body) if l.rstrip() == "        if constexpr (NH == 2) {")
        b = next(i for i in range(a, len(body)) if body[i].rstrip() == "        }")
        body = body[:a] + body[b:]
    two = hidden_layers == 2
    names = {"kHere": "B" if two else "A", "kLast": "B" if two else "A", "kZ": "A" if two else "B", "kF": "B" if two else "A",
             "L::A": "A", "L::B": "B"}
    area = r"(L::A|L::B|kHere|kLast|kZ|kF)\b"
    at_rays = re.search(r"const uint32_t p = acts \+ " + area, "\n".join(load)).group(1)
    rays = [FENCE,
            (r"lds_put<\w+>\(p\b", [("store", at_rays)]),
            (r"lds_get<\w+>\(acts \+ " + area, [("read", "$1")]),
            (r"lds_put<f64x2>\(dz_at \+ L::SUMS", [("store", "sums")])]
    loading = _events(load, rays, names)
    rules = [
        FENCE,
        (r"activate_pair\([^()]*, " + area, [("store", "$1")]),
        (r"store_hidden\(" + area, [("store", "$1")]),
        (r"lds_put_chunk\(.*\+ " + area, [("store", "$1")]),
        (r"lds_put<u32x4>\(dz_at", [("store", "output gradients")]),
        (r"lds_tr\(zp ", [("read", "output gradients")]),
        (r"lds_tr\(hp [^;]*?\+ " + area, [("read", "$1")]),
        (r"I(?:H|W1)::read\((?:col_h|col16_h|col_f)\b[^;]*?" + area, [("read", "$1")]),
        (r"lds_get<f64x2>\(sums_at", [("read", "sums")]),
        (r"lds_put<f64x2>\(sums_at", [("store", "sums")]),
        (r"\bload_rays\(\)", loading),
        (r"\bscatter_step<", [("fence", None), ("store", "A"), ("fence", None), ("read", "A")]),
    ]
    for pattern, lines in [(r, load) for r, _ in rays] + [(r, body) for r, _ in rules]:
        assert any(re.search(pattern, l) for l in lines), f"nothing is checked by {pattern}"
    step = _events(body, rules, names)
    assert {b for w, b in step if w == "read"} == {"A", "B", "output gradients", "sums"} == {b for w, b in step if w == "store"}
    _check(step, loading)


@pytest.mark.parametrize("function", ["scatter_window", "scatter_walk"])
def test_scatter_begins_with_a_fence(function):
    """(As the check of the whole step assumes.)"""
    body = _between(_source("lp_tile_scatter.h"), r"void %s\(" % function, r"^}")
    lds = next(i for i, l in enumerate(body) if re.search(r"lds_put|lds_get|wave_lds_fence|write_scatter_record", l))
    assert "wave_lds_fence()" in body[lds]


def test_weights_of_a_patch():
    """The lanes of a ray add to its column of weights in turn: what one has stored another reads at the next point, so a fence
    stands in every turn of the loop, behind the clearing stores and in front of what follows."""
    body = _between(_source("lp_splat_patch.h"), r"^    for \(int i = lane; i < n_slots \* \(L::kRow", r"^    return n_slots;")
    events = _events(body, [FENCE, (r"lds_put<u32x4>\(area \+ 16 \* i", [("clear", "weights")]), (r"lds_get<float>\(where", [("read", "weights")]),
                            (r"lds_put<float>\(where", [("add", "weights")])])
    assert [w for w, _ in events] == ["clear", "fence", "read", "add", "fence"]
    loop = _between(body, r"^    for \(int k = 0; k < kPatchPoints; \+\+k\) \{", r"^    \}")
    assert [w for w, _ in _events(loop, [FENCE])] == ["fence"] and loop[-1] == "        wave_lds_fence();"   # all lanes pass it


def test_slots_of_a_patch():
    """The window's map: cleared, marked by the lanes that reach a texel, read and numbered by the lane that holds its byte, and read
    by the lanes that marked it."""
    body = _between(_source("lp_splat_patch.h"), r"int patch_weights\(", r"^}")
    step = _events(body, [FENCE, (r"lds_put<u32x4>\(area \+ L::MAP", [("store", "map")]),
                          (r"lds_put<uint8_t>\(area \+ L::MAP \+ dense", [("store", "map")]),
                          (r"lds_get<uint8_t>\(area \+ L::MAP \+ n\)", [("read", "map")]),   # (the number goes into the byte that the lane has read)
                          (r"lds_get<uint8_t>\(area \+ L::MAP \+ dense", [("read", "map")])])
    assert [w for w, _ in step].count("read") == 2 and [w for w, _ in step].count("store") == 2
    _check(step)
    number = [w for w, _ in _events(body, [FENCE, (r"lds_put<uint8_t>\(area \+ L::MAP \+ n, ", [("store", "map")]),
                                           (r"lds_get<uint8_t>\(area \+ L::MAP \+ dense", [("read", "map")])])]
    assert "fence" in number[number.index("store"):number.index("read")]


def test_rays_of_a_forward_in_pairs():
    body = _between(_source("lp_mfma_fwd.hip"), r"^    for \(long long item = sched.first", r"^    }")
    step = _events(body, [FENCE, (r"lds_put<\w+>\(ray_at", [("store", "rays")]), (r"lds_get<\w+>\(at\b", [("read", "rays")])])
    assert {w for w, _ in step} == {"fence", "store", "read"}
    _check(step)


def test_inputs_of_the_mlp_splatter_push():
    body = _between(_source("lp_splat_mfma.hip"), r"^        for \(int sub = 0;", r"^        }")
    step = _events(body, [FENCE, (r"\) ray_x\[", [("store", "inputs")]), (r"= ray_x \+", [("read", "inputs")]),
                          (r"\bscatter_step<|\bpush_ray_step<", [("fence", None)])])   # (an area of its own)
    assert {b for w, b in step if w == "read"} == {"inputs"} == {b for w, b in step if w == "store"}
    _check(step)


def test_a_ray_pushed_by_the_mlp_splatter():
    """push_ray_step's records, in the area that the next step's table or records take."""
    body = _between(_source("lp_splat_mfma.hip"), r"void push_ray_step\(", r"^}")
    walk = body[next(i for i, l in enumerate(body) if "float* info" in l):]
    step = _events(walk, [FENCE, (r"write_scatter_record<", [("store", "records")]), (r"rec\[k\] = ", [("store", "records")]),
                          (r"scatter_(?:channels|weights)<", [("read", "records")])])
    assert [w for w, _ in step][0] == "fence"
    _check(step)


def test_rays_of_the_mlp_splatter_backward():
    """Geometry, inputs, biases and sums of an item's rays; the scatter of the step's gradient begins with a fence and has an area of its own."""
    body = _between(_source("lp_splat_mfma_bwd.h"), r"^    auto march = ", r"^    };")
    step = _events(body, [
        FENCE,
        (r"lds_put<\w+>\(geo_at", [("store", "geometry")]),
        (r"\bgeometry\(\)", [("read", "geometry")]),
        (r"\) ray_x\[", [("store", "inputs")]),
        (r"= ray_x \+|\? ray_x\[", [("read", "inputs")]),
        (r"; \+\+r\) ray_bias\[", [("store", "biases")]),
        (r"\(acc, ray_bias", [("read", "biases")]),
        (r"; \+\+i\) ray_sum\[", [("store", "sums")]),
        (r"= ray_sum\[", [("read", "sums")]),
        (r"write_scatter_record<", [("store", "records")]),
        (r"\bscatter_channels<", [("read", "records")]),
        (r"\bscatter_step<", [("fence", None)]),
    ])
    buffers = {"geometry", "inputs", "biases", "sums", "records"}
    assert {b for w, b in step if w == "read"} == buffers == {b for w, b in step if w == "store"}
    _check(step)
