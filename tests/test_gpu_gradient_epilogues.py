"""Gradients through the GELU's and the context's quantizers, formed by the input-gradient products on each tile that does it: against
the sums over calls of few tokens, where kernels of their own form them (the loss's scale differs by a power of two, so what flows
back is the same up to bf16 roundings of other orders of sums), and column by column in fp64."""
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
    field(mod.params, "ln2_b").add_(torch.randn(hidden, generator=g, device="cuda", dtype=torch.float32))
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
        # up to four tensors in a row may round the other way, by 2^-9 of themselves; of three million elements' errors (about as
        # normal as sums of 4096 terms are) the largest is 5.5 of these
        assert (a - b).norm() <= 2.0 ** -7 * b.norm(), f
        assert (a - b).abs().max() <= 5.5 * 2.0 ** -7 * b.square().mean().sqrt(), f
    a, b = field(whole, "s_a"), field(some, "s_a")
    for i in (5, 7):
        assert (a[i] - b[i]).abs() <= 2.0 ** -7 * b[i].abs(), i
    mod.close()


# All tokens alike, so that every gradient below is a token's times their number (a power of two: fp32 sums of equal bf16 values are
# exact) and each column's can be followed in fp64 from what the device itself gives: the gradients that enter (b_2's and b_o's), the
# gradients that leave (b_1's, b_qkv's), the query/key/value projection.  w_1 is zero, so that u is b_1: both sides of the table's bounds
# and of the quantizer's.
@pytest.mark.parametrize("hidden,heads,ffn,batch", [(256, 4, 1024, 32), (512, 8, 2048, 32), (1024, 16, 4096, 32), (1024, 16, 4096, 64)])
@pytest.mark.parametrize("a_bits", [8, 4])
def test_columns(hidden, heads, ffn, batch, a_bits):
    import torch
    from paper_2109_15082_amd import binding as B
    g = torch.Generator("cuda").manual_seed(hidden + a_bits)
    seq, T, layers, qu, qs = 128, batch * 128, 2, 2 ** a_bits - 1, 2 ** (a_bits - 1) - 1
    mod = B.MremModule(layers, hidden, heads, ffn, batch, seq, w_bits=4, a_bits=a_bits)
    field = lambda v, l, f: v[B.mrem_param_offset(mod.ctx, l, f):][:B.mrem_param_size(mod.ctx, f)]
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float32)
    t = randn(mod.teacher.numel()) * 0.03
    sweep = torch.tensor([0.0] + [s * c * 2.0 ** e for e in (-30, -20, -12, -11, -10, -4, -1, 0, 1, 2, 3, 4) for c in (1.0, 1.0078125, 1.9921875)
                                  for s in (-1, 1)], device="cuda", dtype=torch.float32)
    for l in range(layers):
        for f in ("ln1_g", "ln2_g"):
            field(t, l, f).add_(1.0)
        field(t, l, "w_1").zero_()
        field(t, l, "b_1").copy_(torch.cat([sweep, 1.5 * randn(ffn - sweep.numel())])[torch.randperm(ffn, generator=g, device="cuda")])
    mod.params.copy_(t)
    for l in range(layers):  # outputs to differ from these by their own size
        field(t, l, "ln2_b").copy_(randn(hidden))
    mod.teacher.copy_(t)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.init_steps()
    x = randn(1, 1, hidden).bfloat16().expand(batch, seq, hidden).contiguous()
    mod.calibrate(x)
    for l in range(layers):
        s_a, z_a = field(mod.params, l, "s_a"), field(mod.params, l, "z_a")
        s_a[3] = 2.0 ** -7 / qu  # every probability is 2^-7
        s_a[5] *= 0.5            # contexts on both sides of the bound
        s_a[7], z_a[7] = 4.0 / qu, -0.1
    before = mod.params.clone()
    grads = torch.zeros_like(mod.params)
    mod.step(x, x, 0.0, grads_out=grads)
    at = B.mrem_workspace_offset(mod.ctx, batch, seq, layers - 1, B.MREM_WS_QKV)

    def weights(l, f, n):
        w, s = field(before, l, f).reshape(n, -1), field(before, l, "s" + f)[:, None]
        return (s * (w / s).clamp(-7, 7).round()).bfloat16().double()

    def terms(v, lo, hi):
        """code - v inside, whether inside, which are not within 1e-4 of a bound or a tie"""
        code, inside = v.clamp(lo, hi).round(), (v >= lo) & (v <= hi)
        sure = ((v - lo).abs() > 1e-4) & ((v - hi).abs() > 1e-4) & ((v - v.floor() - 0.5).abs() > 1e-4)
        return code - torch.where(inside, v, 0.0), inside, sure

    ulp = 2.0 ** -8  # of a bf16 value at most, half of it a rounding
    for l in range(layers):
        s_a, z_a = field(before, l, "s_a").double(), field(before, l, "z_a").double()
        grad = lambda f: field(grads, l, f).double() / T
        # GELU and its quantizer
        dr2, w2 = grad("b_2"), weights(l, "w_2", hidden)
        dgh, mag = dr2 @ w2, dr2.abs() @ w2.abs()
        u = field(before, l, "b_1").bfloat16().double()
        cdf = 0.5 * (1 + torch.erf(u / 2 ** 0.5))
        slope = cdf + u * torch.exp(-0.5 * u * u) / (2 * torch.pi) ** 0.5
        y, inside, sure = terms((u * cdf - z_a[7]) / s_a[7], 0, qu)
        du = grad("b_1")
        assert torch.equal(du, du.bfloat16().double())  # every token counted once
        want = torch.where(inside, dgh * slope, 0.0)
        # two roundings to bf16, fp32 sums, slopes to 5e-6 of 1
        tol = 2 * ulp * want.abs() + 5e-6 * dgh.abs() + 2.0 ** -18 * mag
        assert ((du - want).abs() <= tol)[sure].all(), (l, ((du - want).abs() / tol)[sure].max().item())
        assert inside[sure].any() and not inside[sure].all() and (u[sure & inside] < 0).any()
        got, each = grad("s_a")[7], dgh * y
        tol = 4 * ulp * each.norm() + (each.abs() + 1e-3 * dgh.abs())[~sure].sum()
        assert (got - each.sum()).abs() <= tol, (l, got.item(), each.sum().item())
        # the context's quantizer, and through it the values' bias
        if l < layers - 1:
            continue
        v = mod.workspace[at:at + 6 * hidden].view(torch.bfloat16)[2 * hidden:].float()
        s32 = field(before, l, "s_a")
        ratio_v = v / s32[4]
        ctx = (128 * qu * ratio_v.clamp(-qs, qs).round() * (s32[3] * s32[4])).bfloat16().double()
        dr1, wo = grad("b_o"), weights(l, "w_o", hidden)
        dch = dr1 @ wo
        y, inside, sure = terms((ctx.float() / s32[5]).double(), -qs, qs)
        got, each = grad("s_a")[5], dch * y
        tol = 4 * ulp * each.norm() + (each.abs() + dch.abs())[~sure].sum()
        assert (got - each.sum()).abs() <= tol, (l, got.item(), each.sum().item())
        assert inside.any() and not inside.all()
        want = torch.where(inside & (ratio_v.abs() <= qs), dch, 0.0)
        tol = 3 * ulp * want.abs() + 2.0 ** -18 * (dr1.abs() @ wo.abs())
        bad = ((grad("b_qkv")[2 * hidden:] - want).abs() > tol) & sure & ((ratio_v.abs() - qs).abs() > 1e-4)
        assert not bad.any(), (l, int(bad.sum()))
    mod.close()
