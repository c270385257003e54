"""The weight gradients of a layer formed by one launch, against the same step with each product launched by itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# Tiles of 128 x 256, whole and partly filled (320 and 576 wide), and of 256 x 256, whole (1024) and partly filled (992 wide);
# contractions of an even number of stages, and of any length (6, 97 and 99 tokens into the last two stages, one less than them); three layers alternate between the two sets of
# output gradients, four wait for the first one again.  Above 2^19 activations a layer, from 1024 tokens on.
@pytest.mark.parametrize("layers,hidden,heads,ffn,batch,seq", [(2, 768, 12, 3072, 16, 128), (4, 320, 5, 1280, 32, 128), (3, 576, 9, 2304, 17, 128),
                                                               (3, 1024, 16, 4096, 17, 128), (2, 992, 31, 3968, 18, 128), (2, 256, 4, 1024, 64, 40),
                                                               (2, 768, 12, 3072, 30, 77), (3, 1024, 16, 4096, 25, 91), (3, 320, 5, 1280, 33, 65),
                                                               (2, 768, 12, 3072, 25, 87), (3, 768, 12, 3072, 15, 100)])
def test_one_launch_equals_single_products(layers, hidden, heads, ffn, batch, seq):
    import torch
    from paper_2109_15082_amd import binding as B
    rng = np.random.default_rng(hidden + layers)
    x = torch.from_numpy(rng.standard_normal((batch, seq, hidden)).astype(np.float32)).cuda().bfloat16()
    got = []
    for single in (False, True):
        mod = B.MremModule(layers, hidden, heads, ffn, batch, seq)
        w = np.random.default_rng(layers).standard_normal(mod.teacher.numel(), dtype=np.float32) * np.float32(0.02)
        mod.teacher.copy_(torch.from_numpy(w))
        B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
        mod.params.copy_(mod.teacher)
        mod.init_steps()
        mod.calibrate(x)
        grads = torch.zeros_like(mod.params)
        if single:
            B.mrem_profile_gemm_begin(mod.ctx)  # times each product, on one stream
        f_fp, f_q = mod.step(x, x, 1e-4, grads_out=grads)
        torch.cuda.synchronize()
        if single:
            B.mrem_profile_gemm_end(mod.ctx)
        got.append((grads, f_q, mod))
    (g, f, mod), (g1, f1, _) = got
    assert torch.equal(f, f1)
    # the same products of 16-bit operands, summed in fp32 in another order: a sum of T terms of either sign rounds to within
    # sqrt(T) 2^-24 of their size, 4e-6 for 4096 of them
    for l in range(layers):
        for name in ("w_qkv", "w_o", "w_1", "w_2"):
            o, n = B.mrem_param_offset(mod.ctx, l, name), B.mrem_param_size(mod.ctx, name)
            a, b = g[o:o + n].double(), g1[o:o + n].double()
            assert float(b.norm()) > 0 and float((a - b).norm() / b.norm()) < 1e-5, (l, name)
