"""Running softmax over stored keys (bf16, key_tile_step in csrc/block_kernel.h) where scores are spread far: W_Q times 40 spreads them over +-150 log2
units, so that maxima grow from tile to tile by more than the 8 units that are let pass, and lie below -64 for queries whose few keys (a user's first
tokens see one, two, ..) all do; weights that underflowed, overflowed or kept an old factor show as zeros, non-finite values or wrong rows.  Such a
softmax nearly picks one key; rounding a query to bf16 moves a score of 100 by 100 x 2^-9 = 0.2 units or so, which changes the weights of two keys that
come that close.  So rows are judged together: against the fp64 oracle at least nine in ten must be within 5e-2 and half of them within 3e-2 (a wrong
factor between tiles would leave no row with keys in several tiles right; what one row alone would show, one key far below zero, is in the tests with a
constant further down).  Where these lie: the best two of a hundred scores with a spread of 60 units are 20 apart on average and less than 3 in one head
of seven, so that seven in ten rows of eight heads hold such a head; 0.1 to 0.2 units move up to a twentieth of its weight between two
unrelated values, 5e-2 sqrt(2) / sqrt(8) = 2.5e-2 of the row."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


def _case(**kw):
    cfg = synth.CONFIGS["C2"].replace(K=4, n_self=0, ragged=True, len_lo=1, **kw)
    case = synth.make_case(cfg)
    case["weights"]["cross"]["wq"] = synth.round_bf16(case["weights"]["cross"]["wq"] * np.float32(40))
    return cfg, case


def _judge(got, ref):
    assert np.isfinite(got).all()
    there = np.abs(ref).max(-1) > 0
    assert (np.abs(got[there]).max(-1) > 0).all() and (got[~there] == 0).all()
    err = np.linalg.norm(got - ref, axis=-1)[there] / np.linalg.norm(ref, axis=-1)[there]
    print("rows %d, within 5e-2: %.3f, median %.2e" % (err.size, (err < 5e-2).mean(), np.median(err)))
    assert bool((err < 5e-2).mean() >= 0.9 and np.median(err) < 3e-2)


# the few-tiles kernels and, with many users, the ones that keep a user's tiles in a workgroup
@pytest.mark.parametrize("d,heads,B,m,k", [(64, 4, 5, 4, 30), (64, 2, 3, 4, 100), (128, 8, 3, 8, 100), (128, 4, 3, 8, 40), (128, 8, 150, 8, 100), (256, 8, 3, 8, 60),
                                           (256, 8, 100, 8, 100)])
def test_query_side(d, heads, B, m, k):
    from oracle import longer_oracle as orc
    from test_gpu_parity import _runner
    cfg, case = _case(B=B, L=700, len_hi=700, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, index=85)
    case["lens"][:2] = [700, 37]
    case["H"][:2] = synth.round_bf16(np.random.default_rng(5).standard_normal(case["H"][:2].shape).astype(np.float32))
    Y, _ = _runner(case).forward()
    some = np.arange(min(B, 4))
    ref, _ = orc.forward(cfg, case["weights"], case["H"][some], case["G"][some], case["lens"][some])
    _judge(Y[some], ref)
    assert np.isfinite(Y).all()


@pytest.mark.parametrize("d,heads,C", [(64, 4, 20), (128, 8, 20), (128, 8, 1100), (256, 8, 20), (256, 8, 700)])
def test_scoring(d, heads, C):
    from oracle import longer_oracle as orc
    from test_gpu_parity import _runner
    cfg, case = _case(B=3, L=700, len_hi=700, d=d, heads=heads, inner_heads=heads, m=8, k_recent=9, C=C, index=87)
    case["lens"][:3] = [700, 9, 333]
    case["H"][:3] = synth.round_bf16(np.random.default_rng(5).standard_normal(case["H"].shape).astype(np.float32))
    Yg, _ = _runner(case).serve()
    cache = orc.kv_cache_build(cfg, case["weights"], case["H"], case["lens"])
    some = [0, 1, 2, 3, C - 2, C - 1]
    ref, _ = orc.score_candidates(cfg, case["weights"], cache, case["G_cand"][:, some])
    _judge(Yg[:, some], ref)
    assert np.isfinite(Yg).all()


# A constant added to all scores of a query changes no weight beyond the rounding of the scores, wherever they lie and however few keys there are: every
# query's first keys take away what the constant brought.  fp32 scores of 200 units are rounded by 2^-17, weights by 1e-5 of their size: one rounding to
# bf16 (2^-8 apart) in 400 falls the other way for a weight, an attention output, a row: 2^-8 sqrt(3 / 400) = 3.4e-4 of a row at 200 units, and next to
# nothing at 0.3.  Weights rounded wherever the scores happen to lie would be new roundings, all of them: 2^-9 / sqrt(3) x sqrt(2) = 1.6e-3.  (The rows are
# little more than the attention's output here: the projection is the identity, no FFN, small tokens.)
SAME = 8e-4


def _attention_alone(cfg, units):
    case = synth.make_case(cfg)
    w = case["weights"]
    from gpu_util import add_to_scores
    for b in w["inner"]:
        for k in ("wo", "bo", "w2", "b2"):
            b[k][:] = 0
    w["cross"] = add_to_scores(w["cross"], cfg.heads, units)
    w["cross"]["wo"] = np.eye(cfg.d, dtype=np.float32)
    for k in ("bo", "w2", "b2"):
        w["cross"][k][:] = 0
    for k in ("H", "G", "G_cand"):
        if k in case and case[k] is not None:
            case[k] = synth.round_bf16(case[k] * np.float32(0.03125))
    return case


def _same(a, b):
    assert np.isfinite(a).all() and np.isfinite(b).all()
    there = np.abs(a).max(-1) > 0
    assert (there == (np.abs(b).max(-1) > 0)).all()
    err = np.linalg.norm(a[there] - b[there]) / np.linalg.norm(a[there])
    row = (np.linalg.norm(a - b, axis=-1)[there] / np.linalg.norm(a, axis=-1)[there]).max()
    print("difference %.2e, worst row %.2e, %.4f of the values" % (err, row, (a[there] != b[there]).mean()))
    return err


@pytest.mark.parametrize("units", [0.3, 200.0, -200.0])
@pytest.mark.parametrize("d,heads,B,m,k", [(64, 4, 5, 4, 30), (64, 2, 3, 4, 100), (128, 8, 3, 8, 100), (128, 4, 3, 8, 40), (128, 8, 150, 8, 100), (256, 8, 3, 8, 60),
                                           (256, 8, 100, 8, 100)])
def test_query_side_does_not_see_a_constant(d, heads, B, m, k, units):
    from test_gpu_parity import _runner
    cfg = synth.CONFIGS["C2"].replace(K=4, n_self=0, ragged=True, len_lo=1, B=B, L=200, len_hi=200, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, index=91)
    rows = []
    for c in (0.0, units):
        case = _attention_alone(cfg, c)
        case["lens"][:3] = [1, 37, 120]
        rows.append(_runner(case).forward()[0])
    assert _same(*rows) < SAME


@pytest.mark.parametrize("units", [0.3, 200.0, -200.0])
@pytest.mark.parametrize("d,heads,m,C", [(64, 4, 8, 20), (64, 4, 1, 40), (64, 2, 8, 20), (128, 8, 16, 20), (128, 8, 8, 1100), (128, 8, 8, 2100), (256, 8, 32, 20), (256, 8, 8, 700)])
def test_scoring_does_not_see_a_constant(d, heads, m, C, units):
    from test_gpu_parity import _runner
    cfg = synth.CONFIGS["C2"].replace(K=4, n_self=0, ragged=True, len_lo=0, B=3, L=200, len_hi=200, d=d, heads=heads, inner_heads=heads, m=m, k_recent=9, C=C, index=92)
    rows = []
    for c in (0.0, units):
        case = _attention_alone(cfg, c)
        case["lens"][:3] = [0, 9, 150]
        rows.append(_runner(case).serve()[0])
    assert _same(*rows) < SAME
