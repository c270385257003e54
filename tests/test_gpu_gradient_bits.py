"""Gradients of a step where attention runs in the `expf` arithmetic, bit by bit: tests/golden/step_gradient_bits.txt holds
checksums of all gradients, taken with kernels in which one wavefront formed the sums over a whole row of keys.  Those sums
cancel (a step's gradient, a score's), so parts added in another order, or a probability rounded another way in the
query-major kernel than in the key-major one, move second moments of step sizes by half a percent.

`python tests/test_gpu_gradient_bits.py` prints the table of the library that is built."""
import os
import sys

import pytest

import test_gpu_reproducible as R

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "step_gradient_bits.txt")
# one to sixteen tiles of keys over one to four wavefronts, shares uneven and partly filled, key padding, both head
# dimensions, quantizers on and off
NAMES = ["d64_s1", "d64_s23", "d64_s63", "d64_s385", "d64_s512_whole", "d32_s40", "d32_s128_whole", "d32_s131", "d32_s500", "ragged_wide", "ragged_64",
         "off_d64_s30", "off_d64_s400", "off_d32_s140"]


@pytest.mark.parametrize("name", NAMES)
def test_step_gradient_bits(name):
    with open(GOLDEN) as f:
        ref = dict(line.split() for line in f if line.strip() and not line.startswith("#"))
    assert R.checksums(name, step=True) == [ref[name]]


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    for n in NAMES:
        print(n, *R.checksums(n, step=True), flush=True)
