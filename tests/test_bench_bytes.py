"""The bench line's byte counts follow what the library says it reads."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench
from paper_2311_13581_amd import synth


class Reads:
    """A library that reads the copies of these matrices (and of none of the transposes but the LM head's)."""

    def __init__(self, matrices, n):
        self.matrices, self.n = matrices, n

    def coded_use(self, i, rows):
        return i in self.matrices if i < self.n else i == self.n


def test_coded_matrices_count_three_quarters():
    sh = synth.ModelShape(2, 4096, 32, 128, 11008, 32000, dtype=synth.BF16)
    d, F, V = 4096, 11008, 32000
    g = Reads({0, 3, 8}, 9)  # the LM head, gate/up of the first layer, down of the second
    assert bench.coded_saving(g, sh, 5) == (V * d + 2 * F * d + d * F) // 2
    assert bench.coded_saving(g, sh, 5, only=3) == F * d
    assert bench.coded_saving(g, sh, 5, transposes=True) == V * d // 2
    rows = 5 * 4 * (d + F)
    assert bench.gate_up_kernel_bytes(sh, 5) == 4 * F * d + rows
    assert bench.gate_up_kernel_bytes(sh, 5, F * d) == 3 * F * d + rows
    assert bench.coded_saving(g, synth.WORKLOADS["tiny_fp32_greedy"].shape, 5) == 0
