"""What the benchmark says of a timed direction: the kernels inside its event
bracket and the way the sums were evaluated (CPU only)."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


class _Context:
    def __init__(self, side):
        self.side = side

    def info(self):
        return {"transform_side": self.side}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "fp16x3"])
def test_a_direction_is_named_by_every_kernel_it_launches(prec):
    """The fast evaluation's launchers enqueue the kernels named for their
    direction, all of them (the last row pass lies outside the bracket)."""
    with open(os.path.join(ROOT, "paper_1703_02920_amd/csrc/k_trans.hip")) as f:
        src = f.read()

    def launched(*functions):
        out = []
        for fn in functions:
            body = re.search(r"^[^\n]*\b" + fn + r"\(const uvmem_ctx.*?^}\n", src, re.S | re.M).group(0)
            for k in re.findall(r"hipLaunchKernelGGL\(\(?(k_tr_\w+)", body):
                out += [] if k in out else [k]
        return out

    names = bench.direction_work(_Context(2048), 1.0, 1, prec)[3]
    assert names[0].split(" + ") == launched("fwd_lg", "interp_mode")
    assert names[1].split(" + ") == launched("spread_w", "inv_lg")
    assert bench.direction_work(_Context(0), 1.0, 1, prec)[3] == bench.KERNELS[prec]


def test_evaluation_is_said():
    assert bench.evaluation(_Context(0), "bf16x3") == "direct sum, bf16x3 products"
    assert "FP32 windows" in bench.evaluation(_Context(512), "fp16x3")
    assert "FP64 windows" in bench.evaluation(_Context(512), "fp32")
    assert "not evaluated one by one" in bench.evaluation(_Context(512), "fp32")
