"""Which feed-forward widths the quantized products take as int8 codes: sums must stay below 2^31.  Whole tiles hold the GELU's codes
recentred, so the largest product of two 8-bit codes is 128 * 127 there and 2^31 lies between 132096 and 132224 inputs."""
import pytest


@pytest.mark.parametrize("ffn,a_bits,w_bits,int8", [(132096, 8, 8, True), (132224, 8, 8, False), (1 << 20, 8, 8, False), (132224, 7, 8, True),
                                                    (264192, 7, 8, True), (264320, 7, 8, False), (1 << 20, 8, 4, True), (2396672, 8, 4, True), (2396800, 8, 4, False)])
def test_whole_tiles(ffn, a_bits, w_bits, int8):
    from paper_2109_15082_amd import binding as B
    assert (2 ** (a_bits - 1) * (2 ** (w_bits - 1) - 1) * ffn < 2 ** 31) == int8
    ctx = B.mrem_create(n_layers=1, hidden=128, n_heads=2, ffn=ffn, max_batch=2, max_seq=64, w_bits=w_bits, a_bits=a_bits, act_dtype=B.MREM_BF16)
    at = [B.mrem_workspace_offset(ctx, 2, 64, 0, i) for i in (B.MREM_WS_WCODES8 + 3, B.MREM_WS_XCODES8, B.MREM_WS_WCODES + 3)]
    B.mrem_destroy(ctx)
    assert [a >= 0 for a in at] == [int8, int8, not int8]
