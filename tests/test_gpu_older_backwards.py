"""The older backward kernels of voxel grids of 16 channels under an MLP 16-64-64-4, which a switch in the environment
selects when the library is loaded: every storage type, with and without contract coordinates, at the oracle's bounds, and
run by another kernel than the default.  The weight gradients show the kernel: they are summed in a fixed order, so that one
kernel gives the same bits every time and another kernel gives others.  A process per switch; it ends with all its cases done."""
import dataclasses
import os
import subprocess
import sys

import numpy as np
import pytest

import lp_inputs
from lp_inputs import VOXEL

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CASES = {"fp32": ("float32", 0.0), "fp32 contract": ("float32", 1.3), "bf16 contract": ("bfloat16", 1.3),
         "bf16": ("bfloat16", 0.0), "fp16": ("float16", 0.0)}
SWITCHES = ["LP_BWD_ONE_WAVE", "LP_BWD_TWO_WAVE"]


def _case(dtype, contract):
    """2 100 rays: two and three of them per wave."""
    import torch
    inp = lp_inputs.make_small(VOXEL, channels=16, res=(14, 12, 13), mlp_dims=(16, 64, 64, 4), n_rays=2100, samples=41, seed=241,
                               grid_std=0.3, origin_radius=1.4, near=(0.0, 0.3), far=(4.0, 9.0))
    stored = [torch.from_numpy(g).to(getattr(torch, dtype)).float().numpy() for g in inp.grid]
    return dataclasses.replace(inp, grid=stored, contract_a=contract)


def _child(out):
    import torch

    import oracle
    import paper_2404_19760_amd as lp
    from parity import check_case, run_gpu, summary
    bits = {}
    for name, (dtype, contract) in CASES.items():
        inp, tdt = _case(dtype, contract), getattr(torch, dtype)
        print(name, summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=name, grid_dtype=tdt)), flush=True)
        ones = np.ones((inp.n_rays, 3), dtype=np.float32)
        first, second = (run_gpu(lp, inp, ones, math_mode=lp.LP_MATH_BF16X3, grid_dtype=tdt)["dW"] for _ in range(2))
        assert all(np.array_equal(a, b) for a, b in zip(first, second)), name
        bits[name] = first[1]
    np.savez(out, **bits)


@pytest.fixture(scope="module")
def weight_gradients(tmp_path_factory):
    got = {}

    def run(switch):
        if switch not in got:
            out = str(tmp_path_factory.mktemp("older") / "dW.npz")
            env = {k: v for k, v in os.environ.items() if not k.startswith("LP_BWD_")}
            env["PYTHONPATH"] = os.pathsep.join([ROOT, os.path.join(ROOT, "tests"), env.get("PYTHONPATH", "")])
            if switch:
                env[switch] = "1"
            res = subprocess.run([sys.executable, os.path.abspath(__file__), out], env=env, capture_output=True, text=True,
                                 timeout=100)
            print(switch, res.stdout[-2000:], flush=True)
            assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
            got[switch] = np.load(out)
        return got[switch]
    return run


@pytest.mark.parametrize("switch", SWITCHES)
@pytest.mark.parametrize("name", list(CASES))
def test_older_backward(weight_gradients, switch, name):
    default, older = weight_gradients("")[name], weight_gradients(switch)[name]
    assert not np.array_equal(default, older), f"{switch} runs the default kernel"


if __name__ == "__main__":
    _child(sys.argv[1])
