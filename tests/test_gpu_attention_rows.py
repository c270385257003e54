"""Rows of keys that are shared out among the wavefronts of a block, where the shares are uneven or partly filled."""
import pytest

import test_gpu_parity as P

pytestmark = pytest.mark.gpu


# Tiles of 32 keys over four wavefronts: 5 (shares 2 2 1 0), 6 with one key in the last, 9 (3 3 3 0), 12 and 13 (both
# arithmetics' fullest shares), 16 less one key; fewer tiles than wavefronts through key padding; up to three tiles and as
# many wavefronts.  4096 tokens as in test_step_at_attention_length_edges_bf16, whose tolerance this is.
@pytest.mark.parametrize("seq,heads,lo", [(160, 2, 0), (161, 4, 0), (288, 2, 3), (384, 2, 353), (385, 2, 20), (416, 4, 0), (511, 4, 33), (511, 2, 480),
                                          (32, 4, 0), (63, 2, 33), (96, 4, 1)])
def test_step(seq, heads, lo):
    from paper_2109_15082_amd import binding
    P.test_step_at_attention_length_edges_bf16(binding, seq, heads, lo)
