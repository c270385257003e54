"""The ordered product (every sum one fp32 fused multiply-add after the other with k ascending) bit for bit, at the edges of
its tiles and stages and on both of its tiles.

With the quantizers off the first projection of the quantized module is such a product of real-valued bf16 operands, and the
workspace holds its result.  The product of two bf16 values is exact in fp32, so a chain of fused multiply-adds is a chain of
fp32 additions of exact products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# batch, seq, hidden, heads: one row and one chunk of k; rows and columns around 32; k around a stage of 64 and with a partly
# filled last stage; several passes over the four stages; tiles of 64 x 64 (1270 x 1536)
SHAPES = [(1, 1, 8, 1), (1, 5, 64, 1), (1, 31, 72, 3), (3, 11, 56, 1), (1, 32, 136, 17), (5, 13, 320, 5), (1, 65, 328, 41), (1, 40, 1032, 129),
          (5, 254, 512, 8)]


@pytest.mark.parametrize("batch,seq,hidden,heads", SHAPES)
def test_ordered_product_bits(batch, seq, hidden, heads):
    import torch
    from paper_2109_15082_amd import binding as B
    mod = B.MremModule(1, hidden, heads, 16, batch, seq, w_bits=0, a_bits=0)
    rng = np.random.default_rng(hidden + seq)
    t = rng.standard_normal(mod.teacher.numel()).astype(np.float32) * 0.05
    mod.teacher.copy_(torch.from_numpy(t))
    mod.params.copy_(mod.teacher)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    x = torch.from_numpy(rng.standard_normal((batch, seq, hidden)).astype(np.float32)).cuda().bfloat16()
    mod.forward(x, x)
    torch.cuda.synchronize()
    T = batch * seq
    o = B.mrem_workspace_offset(mod.ctx, batch, seq, 0, B.MREM_WS_QKV)
    got = mod.workspace[o:o + T * 3 * hidden * 2].view(torch.bfloat16).float().cpu().numpy().reshape(T, 3 * hidden)

    def field(name):
        f, n = B.mrem_param_offset(mod.ctx, 0, name), B.mrem_param_size(mod.ctx, name)
        return mod.params[f:f + n]
    w = field("w_qkv").bfloat16().float().cpu().numpy().reshape(3 * hidden, hidden)
    a = x.float().cpu().numpy().reshape(T, hidden)
    acc = np.zeros((T, 3 * hidden), np.float32)
    term = np.empty_like(acc)
    for k in range(hidden):
        np.multiply(a[:, k:k + 1], w[:, k], out=term)
        acc += term
    ref = torch.from_numpy(acc + field("b_qkv").cpu().numpy()).bfloat16().float().numpy()
    assert np.array_equal(got, ref)
    mod.close()
