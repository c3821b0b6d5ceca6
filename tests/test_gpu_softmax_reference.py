"""Running softmax over stored keys (bf16, key_tile_step in csrc/block_kernel.h) where scores leave the span in which nothing is subtracted from
them: W_Q times 40 spreads them over +-150 log2 units, so that references move up from tile to tile, and down for queries
whose few keys (a user's first tokens see one, two, ..) all lie below -64; weights that underflowed, overflowed or kept an old factor
show as zeros, non-finite values or wrong rows.  Such a softmax nearly picks one key; rounding a query to bf16 moves a score of 100 by
100 x 2^-9 = 0.2 units or so, which changes the weights of two keys that come that close.  So rows are judged together: against the
fp64 oracle at least nine in ten must be within 5e-2 and half of them within 3e-2 (a wrong factor between tiles would leave no row with keys in
several tiles right).  Where these lie: the best two of a hundred scores with a spread of 60 units are 20 apart on average and less than 3 in one head
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
