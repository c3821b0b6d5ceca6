"""Gradients of the stack's attention (csrc/bw_set_attn.h) where its dispatch draws its lines: 128 query rows and one more (also over few keys: a launch a
side, the query side with its probabilities in registers), 128 keys (a query's probabilities stay in registers) and one more, 288 keys (all of a head's in LDS
at once) and one more; rows missing in the last tile on both sides,
users without a token.  Oracle, tolerances and their derivation as in test_gpu_backward."""
import numpy as np
import pytest

import longer_synth as synth
from gpu_util import add_to_scores
from oracle import longer_oracle_grad as org
from test_gpu_backward import _compare_model, _rel, _run_model_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,k,keys,extra", [(64, 4, 120, 128, {}), (64, 4, 120, 129, dict(gmask="causal")), (128, 4, 120, 288, {}),
                                                  (64, 4, 121, 288, {}), (64, 2, 119, 289, dict(gmask="causal")), (64, 4, 25, 288, dict(k_uniform=7)),
                                                  (32, 2, 40, 127, dict(q_learnable=True)), (64, 4, 121, 127, {}), (64, 2, 130, 96, dict(gmask="causal"))])
def test_query_and_key_sides_at_the_lines(d, heads, k, keys, extra):
    m = 8
    L = 4 * (keys - m)
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=3, L=L, K=4, m=m, k_recent=k, n_self=1, ragged=True, len_lo=0, len_hi=L,
                                      index=149, **extra)
    case = synth.make_case(cfg)
    case["lens"][:3] = [L, 0, L - 90]
    _compare_model("width %d, %d query rows, %d keys" % (d, m + k, keys), case)


# Scores of -170 (log2 units) alone: the key side forms exp2(0 + 170) for the rows of a tile that hold no token, whose results must be zeros and not what
# an infinity times zero is.  Users of one to three merged tokens (dead rows and live ones in the same tiles); both sides in one launch, and two launches.
# Left out are the gradients of what only adds the constant (b_K, and feature 0 of LayerNorm's shift: zero in exact arithmetic, here sums of roundings times a
# query of 470).
@pytest.mark.parametrize("d,heads,k", [(64, 4, 100), (128, 4, 100), (64, 4, 130)])
def test_rows_without_a_token_where_scores_are_far_below_zero(d, heads, k):
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=4, L=12, K=4, m=8, k_recent=k, n_self=1, ragged=True, len_lo=1, len_hi=12, index=150)
    case = synth.make_case(cfg)
    case["lens"][:] = [1, 4, 9, 12]
    w = case["weights"]
    w["cross"] = add_to_scores(w["cross"], heads, -170.0)
    w["self"] = [add_to_scores(w["self"][0], heads, -170.0)]
    labels = synth.draw_labels(cfg)
    loss, logits, dH, dG, grads = _run_model_gpu(case, labels)
    ref_loss, ref_logits, dH_ref, dG_ref, ref = org.model_backward(cfg, w, case["H"], case["G"], case["lens"], labels)
    assert np.isfinite(loss) and np.isfinite(dH).all() and np.isfinite(dG).all()
    print("dH %.2e dG %.2e" % (_rel(dH, dH_ref), _rel(dG, dG_ref)))
    for name, got, want in [("inner", grads["inner"][0], ref["inner"][0]), ("cross", grads["cross"], ref["cross"]), ("self", grads["self"][0], ref["self"][0])]:
        print(name, " ".join("%s %.1e" % (p, _rel(got[p], want[p])) for p in org.PARAMS))
        for p in org.PARAMS:
            assert np.isfinite(got[p]).all(), (name, p)
            if name != "inner" and p == "bk":
                continue
            first = 1 if name != "inner" and p == "ln1_b" else 0
            if p != "bk":
                assert _rel(got[p][first:], want[p][first:]) <= 4e-2, (name, p)
    assert _rel(dH, dH_ref) <= 4e-2 and _rel(dG, dG_ref) <= 4e-2
