"""The large product tiles (128 x 256 and 256 x 256, operands refilled by halves) at their edges, with the element-wise checks
of test_gpu_parity: forward product, weight gradient, input gradient and int8 codes."""
import pytest

import test_gpu_parity as P

pytestmark = pytest.mark.gpu


# (T, N, K).  Forward product [T, N] over K, then d a^ [T, K] over N, then dW [N, K] over T, each on both tiles: whole tiles,
# and 8 rows or columns into a last tile, whose second halves lie beyond the matrix.  Contractions of two stages (no loop),
# four and six.
@pytest.mark.parametrize("T,N,K", [(2056, 3080, 128), (2048, 4096, 256), (2312, 4104, 128), (4096, 4096, 384),
                                   (2056, 128, 3080), (2048, 256, 4096), (2312, 128, 4104), (4096, 384, 4096),
                                   (128, 2056, 3080), (256, 2048, 4096), (128, 2312, 4104), (384, 4096, 4096)])
def test_products(T, N, K):
    from paper_2109_15082_amd import binding
    P.test_products_at_tile_edges(binding, T, N, K)


# 128 x 256 and 256 x 256 tiles, the latter with 128 rows in the last one
@pytest.mark.parametrize("hidden,heads,batch,seq", [(1024, 16, 16, 128), (1024, 16, 25, 128), (1024, 16, 32, 128)])
def test_int8_products(hidden, heads, batch, seq):
    from paper_2109_15082_amd import binding
    P.test_int8_products_on_each_tile(binding, hidden, heads, batch, seq)
