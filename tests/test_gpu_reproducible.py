"""Results that do not depend on the version of the kernels.

The quantizers amplify rounding: one sum taken in another order flips codes, and flips multiply from layer to layer
until, after six layers of 1024 over 100 tokens, step-size gradients (sums that cancel) are tens of percent away.  Two
correct implementations may differ by that, but a user who calibrates with one build and trains with the next may not be
handed other numbers.  So calibration and both forward passes are pinned bit by bit: tests/golden/forward_bits.txt holds
checksums of the clip ranges and of both modules' outputs, taken with the scalar kernels of products and attention that
first served these sizes, and the step-size gradients of a deep step over few tokens.  (Full-precision outputs of 512
tokens or more are pinned only where whole tiles and the hardware's exponential serve them: "-".)

`python tests/test_gpu_reproducible.py` prints the table of the library that is built.
"""
import os
import sys
import zlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "forward_bits.txt")

# name: layers, hidden, heads, ffn, batch, seq, w_bits, a_bits, smallest length (0: no padding), per_channel
CASES = {
    # attention with the hardware's exponential (head dimension 64, 64 to 384 tokens): one chunk of keys and several,
    # products in whole tiles and not
    "d64_s64": (2, 128, 2, 512, 3, 64, 4, 8, 20, 1),
    "d64_s100": (2, 128, 2, 512, 3, 100, 4, 8, 0, 1),
    "d64_s128_whole": (2, 128, 2, 512, 2, 128, 4, 8, 0, 1),
    "d64_s129": (1, 128, 2, 256, 2, 129, 4, 8, 60, 1),
    "d64_s384_whole": (2, 256, 4, 512, 1, 384, 4, 8, 0, 1),
    # with expf: short and long rows, head dimension 32
    "d64_s1": (1, 128, 2, 256, 5, 1, 4, 8, 0, 1),
    "d64_s23": (3, 256, 4, 1024, 1, 23, 4, 8, 0, 1),
    "d64_s63": (2, 320, 5, 1280, 2, 63, 8, 8, 7, 0),
    "d64_s385": (1, 128, 2, 256, 2, 385, 4, 8, 0, 1),
    "d64_s512_whole": (1, 128, 2, 256, 2, 512, 8, 8, 200, 0),
    "d32_s40": (2, 128, 4, 512, 3, 40, 4, 8, 0, 1),
    "d32_s128_whole": (2, 128, 4, 512, 2, 128, 4, 4, 30, 1),
    "d32_s131": (1, 256, 8, 512, 2, 131, 2, 8, 1, 1),
    "d32_s500": (1, 128, 4, 256, 1, 500, 4, 8, 0, 1),
    # ragged products on each tile of the ordered kernel, and on most tiles of the others
    "ragged_wide": (1, 512, 8, 2048, 10, 50, 4, 8, 0, 1),
    "ragged_long": (1, 1024, 16, 4096, 23, 91, 4, 8, 0, 1),
    "ragged_64": (2, 64, 2, 256, 1, 37, 4, 8, 0, 1),
    # quantizers off: no operand is an integer code
    "off_d64_s77": (1, 128, 2, 512, 2, 77, 0, 0, 0, 1),
    "off_d64_s30": (1, 128, 2, 512, 2, 30, 0, 0, 11, 1),
    "off_d64_s400": (1, 128, 2, 256, 1, 400, 0, 0, 300, 1),
    "off_d32_s140": (1, 128, 4, 256, 1, 140, 0, 0, 0, 1),
}
#: the deep step: layers, hidden, heads, ffn, batch, seq
DEEP = (6, 512, 8, 2048, 1, 100)


def _module(shape, w_bits, a_bits, per_channel, seed):
    import torch
    from paper_2109_15082_amd import binding as B
    L, H, nh, F, batch, seq = shape
    mod = B.MremModule(L, H, nh, F, batch, seq, w_bits=w_bits, a_bits=a_bits, per_channel=per_channel)
    rng = np.random.default_rng(seed)
    t = (rng.standard_normal(mod.teacher.numel()) * 0.03).astype(np.float32)
    for l in range(L):
        for f in ("ln1_g", "ln2_g"):
            o = B.mrem_param_offset(mod.ctx, l, f)
            t[o:o + H] += 1.0
    mod.teacher.copy_(torch.from_numpy(t))
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    if w_bits:
        mod.init_steps()
    x = rng.standard_normal((batch, seq, H)).astype(np.float32)
    x[..., 7::50] *= 3.0
    x_fp = torch.from_numpy(x).cuda().bfloat16()
    x_q = torch.from_numpy(x + 0.05 * rng.standard_normal(x.shape).astype(np.float32)).cuda().bfloat16()
    return mod, x_fp, x_q, rng


#: cases whose whole step repeats: whole tiles and the hardware's exponential
STEPS = ("d64_s128_whole", "d64_s384_whole")


def checksums(name, step=False):
    import torch
    from paper_2109_15082_amd import binding as B
    *shape, w_bits, a_bits, lo, per_channel = CASES[name]
    mod, x_fp, x_q, rng = _module(shape, w_bits, a_bits, per_channel, zlib.crc32(name.encode()))
    batch, seq = shape[4:]
    lens = torch.from_numpy(rng.integers(lo, seq + 1, batch).astype(np.int32)).cuda() if lo else None
    steps = b""
    if a_bits:
        mod.calibrate(x_fp, lens)
        for l in range(mod.n_layers):
            for f in ("s_a", "z_a"):
                o = B.mrem_param_offset(mod.ctx, l, f)
                steps += mod.params[o:o + 8].cpu().numpy().tobytes()
    if step:
        grads = torch.zeros_like(mod.params)
        mod.step(x_fp, x_q, 0.0, lens, grads_out=grads)
        torch.cuda.synchronize()
        return [f"{zlib.crc32(grads.cpu().numpy().tobytes()):08x}"]
    f_fp, f_q = mod.forward(x_fp, x_q, lens)
    torch.cuda.synchronize()
    return [f"{zlib.crc32(b):08x}" for b in (steps, *(f.cpu().view(torch.int16).numpy().tobytes() for f in (f_fp, f_q)))]


def deep_step_gradients():
    import torch
    from paper_2109_15082_amd import binding as B
    mod, x_fp, x_q, _ = _module(DEEP, 4, 8, 1, 5)
    mod.calibrate(x_fp)
    grads = torch.zeros_like(mod.params)
    mod.step(x_fp, x_q, 0.0, grads_out=grads)
    torch.cuda.synchronize()
    return np.stack([grads[o:o + 8].cpu().numpy() for o in (B.mrem_param_offset(mod.ctx, l, "s_a") for l in range(mod.n_layers))])


def _golden():
    rows = {}
    with open(GOLDEN) as f:
        for line in f:
            if line.strip() and not line.startswith("#"):
                key, *vals = line.split()
                rows[key] = vals
    return rows


@pytest.mark.parametrize("name", CASES)
def test_calibration_and_forward_bits(name):
    ref = _golden()[name]
    got = [g if r != "-" else r for g, r in zip(checksums(name), ref)]
    assert got == ref, "clip ranges, full-precision outputs, quantized outputs"


@pytest.mark.parametrize("name", STEPS)
def test_step_gradient_bits(name):
    assert checksums(name, step=True) == _golden()["step_" + name]


def test_step_gradients_of_a_deep_step_over_few_tokens():
    """The forward passes repeat bit by bit, so what is left is the rounding of the backward pass to bf16 (2^-9 an element,
    in other places than before: its fp32 sums are not pinned), averaged by sums over at least 100 x 512 elements; forward
    passes of other rounding moved these gradients by 10 to 60 percent a layer."""
    ref = np.array([[float.fromhex(v) for v in _golden()[f"deep_step_s_a_{l}"]] for l in range(DEEP[0])])
    got = deep_step_gradients().astype(np.float64)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert np.all(err <= 1e-2), err


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    for n in CASES:
        print(n, *checksums(n), flush=True)
    for n in STEPS:
        print("step_" + n, *checksums(n, step=True), flush=True)
    for l, row in enumerate(deep_step_gradients()):
        print(f"deep_step_s_a_{l}", *(float(v).hex() for v in row))
