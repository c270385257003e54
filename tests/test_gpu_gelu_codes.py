"""Codes that the quantized projections' kernels form of their output, on each tile that does it: sentences in a batch large
enough for tiles whose codes are formed from LDS, by table for the GELU, and by themselves, where small tiles form each value's
code from its own erf.  Sums of codes are exact and every other operation is the same, so the outputs are the same bits."""
import pytest

pytestmark = pytest.mark.gpu


# 128 x 128, 128 x 256 and 256 x 256 tiles over 4096 tokens; whole 128 x 256 tiles with an odd number of them over 2176
@pytest.mark.parametrize("hidden,heads,ffn,batch", [(256, 4, 1024, 32), (512, 8, 2048, 32), (1024, 16, 4096, 32), (768, 12, 3072, 17)])
@pytest.mark.parametrize("a_bits", [8, 5])
def test_same_bits(hidden, heads, ffn, batch, a_bits):
    import torch
    from paper_2109_15082_amd import binding as B
    g = torch.Generator("cuda").manual_seed(hidden + a_bits)
    mod = B.MremModule(1, hidden, heads, ffn, batch, 128, w_bits=8, a_bits=a_bits)
    t = torch.randn(mod.teacher.numel(), generator=g, device="cuda", dtype=torch.float32) * 0.03
    field = lambda f: t[B.mrem_param_offset(mod.ctx, 0, f):][:B.mrem_param_size(mod.ctx, f)]
    for f in ("ln1_g", "ln2_g"):
        field(f).add_(1.0)
    # values on both sides of the table's bounds, zeros among them
    w1, b1 = field("w_1").reshape(ffn, hidden), field("b_1")
    w1[::7] *= 20.0
    w1[3::7] *= 1e-4
    b1[3::7] *= 1e-3
    w1[5::14] = 0.0
    b1[5::14] = 0.0
    mod.teacher.copy_(t)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.randn(batch, 128, hidden, generator=g, device="cuda", dtype=torch.float32).bfloat16()
    mod.calibrate(x[:1].contiguous())
    _, among = mod.forward(x, x)
    among = among.clone()
    for i in (0, batch - 1):
        _, alone = mod.forward(x[i:i + 1].contiguous(), x[i:i + 1].contiguous())
        assert torch.equal(alone[:, 0], among[:, i])
    mod.close()
