"""Clip ranges that the kernels of a calibration take of what they write: products on each of their tiles (ordered ones, 128 and
256 rows, the last tile partly filled), sections of the query/key/value projection that are no whole tiles, short and long rows
of attention, LayerNorm; with and without padded keys.  The reference is the layer in fp32; the largest values lie in the last
sentence, so in the last tiles."""
import math

import pytest

pytestmark = pytest.mark.gpu

# hidden, heads, ffn, batch, seq
SHAPES = {"one_token": (64, 2, 256, 1, 1), "sections_320": (320, 5, 1280, 3, 50), "tiles_128": (768, 12, 3072, 9, 128), "tiles_256": (1024, 16, 4096, 33, 128),
          "long_rows": (256, 4, 1024, 2, 300), "d32_long_rows": (128, 4, 512, 3, 140)}


@pytest.mark.parametrize("padded", [False, True])
@pytest.mark.parametrize("name", SHAPES)
def test_ranges(name, padded):
    import torch
    import torch.nn.functional as F
    from paper_2109_15082_amd import binding as B
    H, nh, ffn, batch, seq = SHAPES[name]
    g = torch.Generator("cuda").manual_seed(3)
    mod = B.MremModule(1, H, nh, ffn, batch, seq)
    t = torch.randn(mod.teacher.numel(), generator=g, device="cuda", dtype=torch.float32) * 0.05
    field = lambda f: t[B.mrem_param_offset(mod.ctx, 0, f):][:B.mrem_param_size(mod.ctx, f)]
    for f in ("ln1_g", "ln2_g"):
        field(f).add_(1.0)
    mod.teacher.copy_(t)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    x = torch.randn(batch, seq, H, generator=g, device="cuda", dtype=torch.float32)
    x[-1] *= 2.0
    x = x.bfloat16()
    # down to one valid key; the last sentence keeps its largest values
    lengths = torch.tensor([1 + (37 * b + seq // 2) % seq for b in range(batch)], device="cuda", dtype=torch.int32) if padded else None
    mod.calibrate(x, lengths)

    w = lambda f, n: field(f).reshape(n, -1).bfloat16().float()
    xf = x.float().reshape(-1, H)
    qkv = F.linear(xf, w("w_qkv", 3 * H), field("b_qkv"))
    q, k, v = (a.reshape(batch, seq, nh, H // nh).transpose(1, 2) for a in qkv.split(H, 1))
    scores = q @ k.transpose(-1, -2) / math.sqrt(H // nh)
    if padded:
        scores = scores.masked_fill(torch.arange(seq, device="cuda")[None, None, None] >= lengths[:, None, None, None], -math.inf)
    p = torch.softmax(scores, -1)
    ctx = (p @ v).transpose(1, 2).reshape(-1, H)
    x1 = F.layer_norm(xf + F.linear(ctx, w("w_o", H), field("b_o")), (H,), field("ln1_g"), field("ln1_b"), 1e-12)
    gelu = F.gelu(F.linear(x1, w("w_1", ffn), field("b_1")))
    sym = [a.abs().max() / 127 for a in (xf, *qkv.split(H, 1), ctx, x1)]
    ref = torch.stack([sym[0], sym[1], sym[2], p.max() / 255, sym[3], sym[4], sym[5], (gelu.max() - gelu.min()) / 255])
    got = mod.params[B.mrem_param_offset(mod.ctx, 0, "s_a"):][:8]
    z = mod.params[B.mrem_param_offset(mod.ctx, 0, "z_a") + 7]
    # a stored value is off by 2^-9 of itself; up to four roundings in a row, and a probability by the score's, at most 10 here
    tol = torch.tensor([2.0 ** -7] * 8, device="cuda", dtype=torch.float32)
    tol[3] = 10 * 2.0 ** -8
    assert torch.all((got - ref).abs() <= tol * ref), (got / ref).tolist()
    assert (z - gelu.min()).abs() <= 2.0 ** -7 * 0.17 + 2.0 ** -9
