"""What a wave waits for inside of its loops, checked on the CPU from the kernels' source.  Loads from in front of a loop whose values only some
lanes use are outstanding to the compiler on the others' way; what takes their registers in the loop then waits, in every turn,
for all memory operations issued since, atomic adds among them.  So all loads are waited for in front of the loop."""
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2404_19760_amd", "csrc")


def test_tile_backward_waits_for_its_loads_in_front_of_the_loop():
    with open(os.path.join(CSRC, "lp_mfma_bwd_tile.h")) as f:
        source = re.sub(r"//[^\n]*", "", f.read())
    before = [l.strip() for l in source[:source.index("while (live) {")].splitlines() if l.strip()]
    assert before[-1] == "loads_done();"
