"""Gradients through the GELU's and the context's quantizers, formed by the input-gradient products on each tile that does it,
against the sums over calls of few tokens, where kernels of their own form them.  The loss's scale differs by a power of two, so
what flows back is the same up to bf16 roundings of other orders of sums."""
import pytest

pytestmark = pytest.mark.gpu


# tiles of the second feed-forward projection's input gradient [T, ffn] and the context's [T, hidden]: 128 x 128 and none;
# 128 x 256 and 128 x 128; 256 x 256 and 128 x 128; 256 x 256 and 128 x 256
@pytest.mark.parametrize("hidden,heads,ffn,batch,parts", [(256, 4, 1024, 32, 2), (512, 8, 2048, 32, 4), (1024, 16, 4096, 32, 8), (1024, 16, 4096, 64, 16)])
@pytest.mark.parametrize("a_bits", [8, 4])
def test_step(hidden, heads, ffn, batch, parts, a_bits):
    import torch
    from paper_2109_15082_amd import binding as B
    g = torch.Generator("cuda").manual_seed(hidden + a_bits)
    mod = B.MremModule(1, hidden, heads, ffn, batch, 128, w_bits=4, a_bits=a_bits)
    t = torch.randn(mod.teacher.numel(), generator=g, device="cuda", dtype=torch.float32) * 0.03
    offset = {f: B.mrem_param_offset(mod.ctx, 0, f) for f in B.FIELDS}
    field = lambda v, f: v[offset[f]:][:B.mrem_param_size(mod.ctx, f)]
    for f in ("ln1_g", "ln2_g"):
        field(t, f).add_(1.0)
    # values on both sides of the table's bounds, zeros among them
    w1, b1 = field(t, "w_1").reshape(ffn, hidden), field(t, "b_1")
    w1[::7] *= 15.0
    w1[3::7] *= 1e-4
    b1[3::7] *= 1e-3
    w1[5::14] = 0.0
    b1[5::14] = 0.0
    mod.teacher.copy_(t)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.randn(batch, 128, hidden, generator=g, device="cuda", dtype=torch.float32).bfloat16()
    mod.calibrate(x[:2].contiguous())  # the others reach beyond these ranges
    # the context's quantizer clips too
    field(mod.params, "s_a")[5] *= 0.3

    def gradients(part):
        grads = torch.zeros_like(mod.params)
        mod.step(part, part, 0.0, grads_out=grads)
        return grads.double()

    whole = gradients(x)
    some = sum(gradients(p.contiguous()) for p in x.chunk(parts)) / parts
    for f in ("b_1", "w_1", "b_2", "ln1_g", "w_o", "b_qkv", "w_qkv"):
        a, b = field(whole, f), field(some, f)
        # an output that rounds the other way moves its difference of two outputs, a tenth of their size, by 2^-8 / 0.1
        assert (a - b).norm() <= 4e-2 * b.norm(), f
    a, b = field(whole, "s_a"), field(some, "s_a")
    for i in (5, 7):
        assert (a[i] - b[i]).abs() <= 4e-2 * b[i].abs(), i
    mod.close()
