"""One step for a whole tensor, around the sizes where one block holds all weights (32768), where a thread has a second and a third
chunk of its part (1048576, 2097152) and where one block forms the step in a launch of its own (4194304).  The codes carry the parts'
maxima in between.  The reference is Eq. 1 in fp32, whose operations are the kernels' own."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(1, 32764), (1, 32767), (2, 16384), (1, 32769), (4, 8193), (5, 6555), (31, 4001), (512, 4099), (2048, 4096), (3001, 2999),
                                 (1, 1048579), (1, 1048580), (1, 2097155), (1, 2097156), (1, 4194303), (1, 4194305)])
@pytest.mark.parametrize("at", [0, 70, -1])  # the largest weight among the first codes or the last one
def test_tensor(N, K, at):
    import torch
    from paper_2109_15082_amd import binding as B
    g = torch.Generator("cuda").manual_seed(N + K)
    w = torch.randn(N, K, generator=g, device="cuda", dtype=torch.float32) * 0.02
    w.view(-1)[at] = -0.5
    scale, s = (torch.full((1,), float("nan"), device="cuda", dtype=torch.float32) for _ in range(2))
    s[:] = torch.tensor(0.5, dtype=torch.float32) / torch.tensor(127.0, dtype=torch.float32)
    ref = (w / s).clamp(-127, 127).round().to(torch.int8)
    codes = torch.full((N, K), 99, device="cuda", dtype=torch.int8)
    for _ in range(3):  # the codes of the call before lie where the maxima go
        B.mrem_quantize(w, N, K, 8, 0, 1, scale, codes)
        assert torch.equal(scale, s) and torch.equal(codes, ref)
    B.mrem_quantize(w, N, K, 8, 0, 0, scale, codes.fill_(99))
    assert torch.equal(codes, ref)
