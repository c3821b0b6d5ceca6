"""The last block's W2 gradient from operands kept group by group (csrc/bw_block.h: groups of 8 and 16 tokens, mean merge).  Where that can go wrong: fewer
slots than a tile of 32 groups, one tile and one group more, a tile half of which no workgroup wrote (all of its tokens are padding), groups with fewer tokens
than K (their mean's divisor), empty users, two blocks (the first one's operands stay token by token, in records of another size), concatenation (no group
operands).  Below width 128 users of different length keep theirs token by token, users of one length (the last group filled up) by groups.  The workspace starts as NaN: what nobody wrote must not count.  Oracle and bars as in test_gpu_backward."""
import numpy as np
import pytest

import longer_synth as synth
from test_gpu_backward import _compare, _run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,B,L,layers,merge", [
    (128, 8, 1, 3, 1, "mean"), (128, 8, 3, 83, 1, "mean"), (128, 16, 5, 203, 2, "mean"), (64, 8, 9, 257, 2, "mean"), (64, 16, 2, 511, 1, "mean"),
    (32, 8, 4, 131, 1, "mean"), (32, 16, 3, 40, 1, "mean"), (128, 8, 6, 700, 1, "mean"), (64, 8, 2, 60, 1, "concat")])
def test_w2_from_group_operands(d, K, B, L, layers, merge):
    if merge == "concat":
        cfg = synth.CONFIGS["P1"].replace(B=B, L=L, d=d * K // 2, K=K // 2, heads=8, inner_heads=d // 16, k_recent=5, n_self=1, inner_layers=layers, index=97)
    else:
        cfg = synth.CONFIGS["C2"].replace(d=d, heads=d // 16, inner_heads=d // 16, K=K, B=B, L=L, k_recent=5, n_self=1, inner_layers=layers, ragged=True,
                                          len_lo=0, len_hi=L, index=97)
    case = synth.make_case(cfg)
    if cfg.ragged:
        case["lens"][0] = L
        if B > 2:
            case["lens"][1] = 0
        if B > 5:
            case["lens"][2:5] = [3, 0, 0]        # (L = 700: whole workgroups of padding inside a tile of 32 groups)
    _compare("d = %d, K = %d, %d x %d, %d blocks, %s" % (d, K, B, L, layers, merge), case, synth.draw_merge_gradient(cfg), ws_fill=0xFF)


@pytest.mark.parametrize("d,B,L,layers", [(64, 9, 257, 2), (64, 1, 3, 1), (64, 3, 83, 1), (32, 4, 131, 1), (32, 5, 264, 2), (128, 3, 260, 1)])
def test_w2_from_group_operands_of_users_of_one_length(d, B, L, layers):
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=d // 16, inner_heads=d // 16, K=8, B=B, L=L, k_recent=5, n_self=1, inner_layers=layers, index=97)
    _compare("d = %d, %d x %d, %d blocks, one length" % (d, B, L, layers), synth.make_case(cfg), synth.draw_merge_gradient(cfg), ws_fill=0xFF)


@pytest.mark.parametrize("d,K", [(128, 8), (128, 16), (64, 8)])
def test_w2_gradient_of_an_infinite_hidden_value(d, K):
    """A hidden unit whose bias is +infinity, upstream gradients above zero, no padding: its row of W2's gradient is +infinity (the rounding rest of an infinite mean
    is not infinity less infinity), and every other row is finite."""
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=d // 16, inner_heads=d // 16, K=K, B=2, L=64, k_recent=5, n_self=1, inner_layers=1, act="relu", index=97)
    case = synth.make_case(cfg)
    case["weights"]["inner"][0]["b1"][5] = np.inf
    _, grads = _run_gpu(case, np.abs(synth.draw_merge_gradient(cfg)) + 0.5)
    w2 = grads[0]["w2"]
    assert (w2[5] == np.inf).all()
    assert np.isfinite(np.delete(w2, 5, axis=0)).all()
