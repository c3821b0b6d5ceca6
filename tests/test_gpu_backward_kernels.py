"""GPU parity of the backward pass at the sizes where its kernels can go wrong: fewer rows than a tile or a
contraction step, remainders of both, more key rows than query rows by a factor, every width.  Oracle, tolerances
and their derivation as in test_gpu_backward."""
import pytest

import longer_synth as synth
from test_gpu_backward import _compare, _compare_model, _say

pytestmark = pytest.mark.gpu


# (width, heads, users, raw length, ragged): 1 row; 31 / 33 rows (a 32-row step and its neighbours); 129 rows and
# 3 x 257 (a 128-row tile and one more); a step that is all padding
@pytest.mark.parametrize("d,heads,B,L,ragged", [(32, 2, 1, 1, False), (64, 4, 1, 31, False), (128, 8, 1, 33, False),
                                                (128, 4, 1, 129, False), (64, 2, 3, 257, True), (256, 8, 2, 65, True)])
def test_parameter_gradients_at_row_remainders(d, heads, B, L, ragged):
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=B, L=L, k_recent=5, n_self=1, ragged=ragged,
                                      len_lo=0, len_hi=L, index=61)
    case = synth.make_case(cfg)
    if ragged:
        case["lens"][:2] = [L, 3]
    _compare("width %d, %d rows" % (d, B * L), case, synth.draw_merge_gradient(cfg))
    _compare_model("width %d, %d rows" % (d, B * L), case)


@pytest.mark.parametrize("n_self", [1, 3])
def test_parameter_gradients_many_more_key_rows_than_query_rows(n_self):
    """The cross layer's key and value gradients contract over m + T rows a user, the others over m + k: here 20 times
    as many, so their slices are cut finer than the launch's.  (Not with n_self = 0: b_2 then gets its gradient from
    the global rows alone, sum over the users of (sigmoid(logit) - label) / B times a fixed vector, and these three
    users' terms, -0.0129 - 0.1356 + 0.1473, cancel to -0.0012; a logit error of 3e-3 moves a term by up to
    3e-3 / 4 / 3 = 2.5e-4, a fifth of what is left.)"""
    cfg = synth.CONFIGS["C2"].replace(B=3, L=1000, K=4, m=2, k_recent=10, n_self=n_self, ragged=True, len_lo=300, len_hi=1000, index=62)
    _compare_model("T = 250, k = 10, n_self = %d" % n_self, synth.make_case(cfg))


# Token merge alone, two blocks, at every register window of the block kernel (K <= 8, 16, 32) and both head widths:
# lengths that are no multiple of K, tiles that hold several users or end inside one, users without a token, the
# last workgroup's empty tiles; both merges; the widest hidden layer (2048)
@pytest.mark.parametrize("d,dh,K,B,L,merge,ffn", [(32, 16, 4, 7, 9, "mean", 4), (32, 16, 32, 5, 70, "mean", 4), (64, 32, 16, 9, 50, "mean", 4),
                                                  (64, 16, 8, 33, 1, "mean", 4), (128, 16, 16, 6, 45, "mean", 4), (128, 32, 32, 3, 130, "mean", 4),
                                                  (128, 16, 1, 2, 77, "mean", 4), (64, 32, 2, 3, 65, "concat", 4), (32, 16, 8, 4, 131, "concat", 7)])
def test_block_kernel_windows_and_tile_remainders(d, dh, K, B, L, merge, ffn):
    w = d * K if merge == "concat" else d
    cfg = synth.CONFIGS["C2"].replace(d=w, heads=w // 16, inner_heads=d // dh, inner_layers=2, K=K, B=B, L=L, ragged=True, len_lo=0,
                                      len_hi=L, merge=merge, ffn_mult=ffn, m=2, k_recent=4, n_self=1, index=63)
    case = synth.make_case(cfg)
    case["lens"][0] = L
    if B > 1:
        case["lens"][1] = 0
    _compare("width %d, head width %d, K = %d, %d x %d, %s" % (d, dh, K, B, L, merge), case, synth.draw_merge_gradient(cfg))


def test_block_kernel_widest_hidden_layer():
    """One block with 2048 hidden features: its vectors and the weight ring no longer let two workgroups share a compute unit."""
    cfg = synth.CONFIGS["C2"].replace(d=128, heads=8, inner_heads=8, inner_layers=1, K=8, B=2, L=70, ffn_mult=16, index=64)
    _compare("2048 hidden features", synth.make_case(cfg), synth.draw_merge_gradient(cfg))


# The reduced stack's tiles where the hidden chunks do not fill its four (eight) waves evenly: 2, 3, 6 and 10 chunks, 8 at width 256;
# 33 query rows, so the second tile holds one.  (Not the draw of index 66: at width 256 its last b_2 gradient is the sum over the
# users of (sigmoid(logit) - label) / B, 0.333 - 0.186 - 0.123 = 0.0239, times a fixed vector; the logits' error of 1.4e-2, inside
# its bar, moves a term by up to 1.4e-2 / 4 / 3 = 1.2e-3, a twentieth of that.  With labels of one value the terms add up.)
@pytest.mark.parametrize("d,heads,ffn", [(32, 2, 2), (32, 2, 3), (64, 4, 1), (64, 4, 3), (64, 2, 5), (256, 8, 1)])
def test_stack_with_any_number_of_hidden_chunks(d, heads, ffn):
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=3, L=90, m=2, k_recent=9, n_self=2, ffn_mult=ffn, ragged=True,
                                      len_lo=20, len_hi=90, index=67)
    _compare_model("width %d, %d hidden features" % (d, d * ffn), synth.make_case(cfg))


# The stack's attention where a self layer's keys stay in registers and where they do not (four key tiles and one key more), with one to
# four key tiles, rows of the last one missing; every mask: global rows alone in a tile, beside sequence rows, causal ones; users without
# a token; sampled and learnable slots
@pytest.mark.parametrize("d,heads,m,k,extra", [(64, 4, 8, 120, {}), (64, 4, 8, 121, dict(gmask="causal")), (128, 4, 32, 33, dict(gmask="causal")),
                                               (64, 2, 4, 28, dict(k_uniform=9)), (32, 2, 16, 70, dict(q_learnable=True, gmask="causal"))])
def test_set_attention_key_tiles_and_masks(d, heads, m, k, extra):
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=4, L=700, K=4, m=m, k_recent=k, n_self=2, ragged=True, len_lo=0, len_hi=700,
                                      index=109, **extra)
    case = synth.make_case(cfg)
    case["lens"][:3] = [700, 0, 50]
    _compare_model("width %d, %d + %d rows" % (d, m, k), case)


# More blocks than one launch of the LayerNorm gradients takes (16): their gradients are made of the stack's sums over its rows, which a whole
# step forms together with the merge's.  With a merge in tiles and one without (width 256)
@pytest.mark.parametrize("d,heads,n_self,inner", [(64, 4, 15, 1), (64, 4, 16, 2), (32, 2, 30, 1), (256, 8, 16, 1), (64, 4, 14, 17)])
def test_gradients_of_deep_models(d, heads, n_self, inner):
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=4, L=90, m=4, k_recent=9, n_self=n_self, inner_layers=inner,
                                      ragged=True, len_lo=20, len_hi=90, index=127)
    _compare_model("width %d, %d self layers, %d InnerTrans blocks" % (d, n_self, inner), synth.make_case(cfg))


# Rows whose features are all alike and far from zero: their normalised rows are exact zeros, and with them the gradient of the first
# LayerNorm's gain.  (A normalised row of x / s - mean / s, the quotients rounded on their own, came out as up to 0.016 here, and the gain's gradient
# as 2e-3 of the shift's.  The gradients of W_Q and W_K are zero as well, all keys being alike, so they are not compared.)
@pytest.mark.parametrize("d,heads,K", [(128, 8, 8), (64, 4, 16), (32, 2, 4)])
def test_rows_without_spread(d, heads, K):
    import numpy as np
    from oracle import longer_oracle_grad as org
    from test_gpu_backward import TOL, _rel, _run_gpu
    cfg = synth.CONFIGS["C2"].replace(d=d, heads=heads, inner_heads=heads, B=4, L=150, K=K, m=2, k_recent=4, n_self=1, inner_layers=1, index=139)
    case = synth.make_case(cfg)
    value = synth.round_bf16(np.random.default_rng(11).uniform(300.0, 1000.0, size=case["H"].shape[:2] + (1,)).astype(np.float32))
    case["H"] = np.broadcast_to(value, case["H"].shape).astype(np.float32)
    dM = synth.draw_merge_gradient(cfg)
    dH, grads = _run_gpu(case, dM)
    gain, shift = (float(np.linalg.norm(grads[0][k])) for k in ("ln1_g", "ln1_b"))
    _say("rows without spread, width %d: gradient of the first LayerNorm's gain %.3e, shift %.3e" % (d, gain, shift))
    assert shift > 0 and gain <= 1e-6 * shift
    dH_ref, g_ref = org.token_merge_backward(cfg, case["weights"]["inner"], case["H"], None, dM, keep="input_only")
    assert _rel(dH, dH_ref) <= TOL
    for name in ("ln1_b", "wv", "wo", "ln2_g", "w1", "w2"):
        assert _rel(grads[0][name], g_ref[0][name]) <= TOL, name
