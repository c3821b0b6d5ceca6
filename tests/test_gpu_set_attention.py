"""Gradients of the stack's attention (csrc/bw_set_attn.h) where its dispatch draws its lines: 128 query rows and one more, 128 keys (a query's
probabilities stay in registers) and one more, 288 keys (all of a head's in LDS at once) and one more; rows missing in the last tile on both sides,
users without a token.  Oracle, tolerances and their derivation as in test_gpu_backward."""
import pytest

import longer_synth as synth
from test_gpu_backward import _compare_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,k,keys,extra", [(64, 4, 120, 128, {}), (64, 4, 120, 129, dict(gmask="causal")), (128, 4, 120, 288, {}),
                                                  (64, 4, 121, 288, {}), (64, 2, 119, 289, dict(gmask="causal")), (64, 4, 25, 288, dict(k_uniform=7)),
                                                  (32, 2, 40, 127, dict(q_learnable=True))])
def test_query_and_key_sides_at_the_lines(d, heads, k, keys, extra):
    m = 8
    L = 4 * (keys - m)
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=3, L=L, K=4, m=m, k_recent=k, n_self=1, ragged=True, len_lo=0, len_hi=L,
                                      index=149, **extra)
    case = synth.make_case(cfg)
    case["lens"][:3] = [L, 0, L - 90]
    _compare_model("width %d, %d query rows, %d keys" % (d, m + k, keys), case)
