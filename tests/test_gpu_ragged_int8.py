"""int8 products with any number of tokens, on each tile that serves them."""
import pytest

pytestmark = pytest.mark.gpu


# one token; 64 x 64, 128 x 64, 128 x 128, 128 x 256 and 256 x 256 tiles; contractions that are no even number of stages on
# 128 x 64 and on the 256 x 256 tile that refills whole stages
@pytest.mark.parametrize("hidden,heads,batch,seq", [(128, 2, 1, 1), (128, 2, 1, 100), (384, 6, 9, 111), (1024, 16, 9, 111), (1024, 16, 20, 111),
                                                    (1024, 16, 33, 111), (384, 6, 40, 111), (384, 6, 66, 111)])
def test_int8_products(hidden, heads, batch, seq):
    """The query/key/value projection against the integer dot products of Eq. 1's codes: s_a s_w[n] (codes . codes) + bias, rounded
    to bf16 once (2^-8 covers that and the fp32 roundings of the epilogue).  The weights' codes are those left in the workspace."""
    import torch
    from paper_2109_15082_amd import binding as B
    mod = B.MremModule(1, hidden, heads, hidden, batch, seq, w_bits=8)
    g = torch.Generator("cuda").manual_seed(hidden)
    mod.teacher.copy_(torch.randn(mod.teacher.numel(), generator=g, device="cuda", dtype=torch.float32) * 0.05)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.randn(batch, seq, hidden, generator=g, device="cuda", dtype=torch.float32).bfloat16()
    mod.calibrate(x)
    mod.workspace.fill_(255)
    mod.forward(x, x)
    T, N = batch * seq, 3 * hidden

    def item(i, n):
        o = B.mrem_workspace_offset(mod.ctx, batch, seq, 0, i)
        return mod.workspace[o:o + 2 * n].view(torch.bfloat16)

    def field(f, n):
        o = B.mrem_param_offset(mod.ctx, 0, f)
        return mod.params[o:o + n]

    codes_x = (x.float() / field("s_a", 8)[0]).clamp(-127, 127).round().reshape(T, hidden).double()
    s_w = field("sw_qkv", N)
    codes_w = item(B.MREM_WS_WCODES, N * hidden).reshape(N, hidden)
    assert torch.equal(codes_w.float(), (field("w_qkv", N * hidden).reshape(N, hidden) / s_w[:, None]).clamp(-127, 127).round())
    got = item(B.MREM_WS_QKV, T * N).reshape(T, N).double()
    prod = (codes_x @ codes_w.double().T) * (field("s_a", 8)[0].double() * s_w.double())
    bias = field("b_qkv", N).double()
    tol = 2.0 ** -8 * (prod + bias).abs() + 2.0 ** -22 * (prod.abs() + bias.abs())
    bad = ~((got - (prod + bias)).abs() <= tol)
    assert not bad.any(), (int(bad.sum()), (got - prod - bias).abs().max().item())
    mod.close()


@pytest.mark.parametrize("a_bits", [8, 4, 3])
def test_recentred_codes(a_bits):
    """The second feed-forward projection's codes are stored less half their range, which ragged sizes add back to the sums and
    whole tiles to the results.  Three sentences by themselves (150 tokens) and among 64 (25 tiles of 128); the weights of that
    projection are of one sign, so that a shift that is not undone changes every output by more than its own size."""
    import torch
    from paper_2109_15082_amd import binding as B
    H, F, seq = 256, 1024, 50
    g = torch.Generator("cuda").manual_seed(a_bits)
    mod = B.MremModule(1, H, 4, F, 64, seq, w_bits=4, a_bits=a_bits)
    t = torch.randn(mod.teacher.numel(), generator=g, device="cuda", dtype=torch.float32) * 0.05
    field = lambda f: t[B.mrem_param_offset(mod.ctx, 0, f):][:B.mrem_param_size(mod.ctx, f)]
    for f in ("ln1_g", "ln2_g"):
        field(f).add_(1.0)
    field("w_2").abs_()
    mod.teacher.copy_(t)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.randn(64, seq, H, generator=g, device="cuda", dtype=torch.float32).bfloat16()
    mod.calibrate(x)
    _, among = mod.forward(x, x)
    among = among[:, :3].float().clone()
    _, alone = mod.forward(x[:3].contiguous(), x[:3].contiguous())
    # fp32 roundings in another order: a bf16 value may round the other way (2^-8), and behind it a code flip, one step of at
    # most 2 / (2^a_bits - 2) of the range in few of the 1024 terms of a sum
    assert (alone.float() - among).norm() <= 2e-2 * among.norm()
    mod.close()
