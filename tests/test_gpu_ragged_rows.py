"""Products of 512 tokens and more in partly filled tiles: one order of sums (the even and the odd substeps of the contraction
apart, then together) on every tile that serves them."""
import os
import sys

import pytest

import test_gpu_gradient_bits as G
import test_gpu_reproducible as R

pytestmark = pytest.mark.gpu

# layers, hidden, heads, ffn, batch, seq, sentences of the small batch (from 512 tokens on: below, sums have another order).
# Products over 768 and 1024 in one round of large tiles, and in a second one that is nearly empty (264 tiles); 15 tokens into
# the last tile's second half; a single layer and two.
SHAPES = {"rows_768": (1, 768, 12, 3072, 30, 77, 10), "rows_1024": (1, 1024, 16, 3072, 28, 100, 7), "rows_768_2l": (2, 768, 12, 3072, 25, 87, 6),
          "rows_1024_s130": (1, 1024, 16, 3072, 20, 130, 4)}


@pytest.mark.parametrize("name", SHAPES)
def test_outputs_do_not_depend_on_the_batch(name):
    import torch
    *shape, small = SHAPES[name]
    mod, x_fp, x_q, _ = R._module(shape, 4, 8, 1, 11)
    mod.calibrate(x_fp)
    f_fp, f_q = (f.clone() for f in mod.forward(x_fp, x_q))
    g_fp, g_q = mod.forward(x_fp[:small].contiguous(), x_q[:small].contiguous())
    assert torch.equal(f_fp[:, :small], g_fp) and torch.equal(f_q[:, :small], g_q)


def gradients(name):
    import torch
    import zlib
    *shape, _ = SHAPES[name]
    mod, x_fp, x_q, _ = R._module(shape, 4, 8, 1, 12)
    mod.calibrate(x_fp)
    grads = torch.zeros_like(mod.params)
    mod.step(x_fp, x_q, 0.0, grads_out=grads)
    torch.cuda.synchronize()
    return f"{zlib.crc32(grads.cpu().numpy().tobytes()):08x}"


@pytest.mark.parametrize("name", [n for n in SHAPES if SHAPES[n][0] == 1])
def test_step_gradient_bits(name):
    """Single layers, whose weight gradients are products of their own.  The checksums are those of 128 x 64 tiles."""
    with open(G.GOLDEN) as f:
        ref = dict(line.split() for line in f if line.strip() and not line.startswith("#"))
    assert gradients(name) == ref[name]


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    for n in SHAPES:
        print(n, gradients(n), flush=True)
