"""int8 products with any number of tokens, on each tile that serves them, with the integer check of test_gpu_parity."""
import pytest

import test_gpu_parity as P

pytestmark = pytest.mark.gpu


# one token; 64 x 64, 128 x 64, 128 x 128, 128 x 256 and 256 x 256 tiles; contractions that are no even number of stages on
# 128 x 64 and on the 256 x 256 tile that refills whole stages
@pytest.mark.parametrize("hidden,heads,batch,seq", [(128, 2, 1, 1), (128, 2, 1, 100), (384, 6, 9, 111), (1024, 16, 9, 111), (1024, 16, 20, 111),
                                                    (1024, 16, 33, 111), (384, 6, 40, 111), (384, 6, 66, 111)])
def test_int8_products(hidden, heads, batch, seq):
    from paper_2109_15082_amd import binding
    P.test_int8_products_on_each_tile(binding, hidden, heads, batch, seq)


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
    t = torch.randn(mod.teacher.numel(), generator=g, device="cuda") * 0.05
    field = lambda f: t[B.mrem_param_offset(mod.ctx, 0, f):][:B.mrem_param_size(mod.ctx, f)]
    for f in ("ln1_g", "ln2_g"):
        field(f).add_(1.0)
    field("w_2").abs_()
    mod.teacher.copy_(t)
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.randn(64, seq, H, generator=g, device="cuda").bfloat16()
    mod.calibrate(x)
    _, among = mod.forward(x, x)
    among = among[:, :3].float().clone()
    _, alone = mod.forward(x[:3].contiguous(), x[:3].contiguous())
    # fp32 roundings in another order: a bf16 value may round the other way (2^-8), and behind it a code flip, one step of at
    # most 2 / (2^a_bits - 2) of the range in few of the 1024 terms of a sum
    assert (alone.float() - among).norm() <= 2e-2 * among.norm()
    mod.close()
