"""Short users of width 64: the stack's launch makes the cross layer's K and V itself (csrc/chain_kernel.h; m + T at most 96 rows, a launch of their own beyond).
Where that can go wrong: one, two and three key tiles, the last row of the last one and one row more (the other way), a user with fewer tokens than the others or none (its
key tiles end early, the barriers do not), one merged token, learnable query tokens (keys are the merged tokens, not the query rows), sampled queries, causal globals, sixteen
globals, as many users as one round takes and one more, no self layer.  Against the fp64 oracle at the bf16 bar, outputs between guard bands."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("B,T,m,k,n_self,kw", [
    (1, 1, 4, 3, 1, {}), (3, 28, 4, 32, 2, {}), (5, 60, 4, 20, 1, {"k_uniform": 7}), (4, 92, 4, 60, 1, {}), (4, 93, 4, 32, 1, {}),
    (6, 64, 8, 40, 2, {"q_learnable": True}), (3, 80, 16, 48, 1, {"gmask": "causal"}), (2, 40, 2, 5, 0, {}), (256, 13, 4, 8, 1, {}), (257, 13, 4, 8, 1, {})])
def test_keys_in_the_stack_launch(B, T, m, k, n_self, kw):
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    L = 8 * T - 3
    cfg = synth.CONFIGS["C2"].replace(B=B, L=L, K=8, m=m, k_recent=k, n_self=n_self, ragged=True, len_lo=0, len_hi=L, index=93, **kw)
    case = synth.make_case(cfg)
    case["lens"][0] = L
    if B > 2:
        case["lens"][1:3] = [0, min(5, L)]
    r = _runner(case)
    Y, logits = r.forward()
    Yr, lr = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    _check("longer_forward", Y, Yr, TOL["bf16"])
    # a logit is <head_w, global rows>: rows within the bar move it by at most the bar times both norms
    hw = np.asarray(case["weights"]["head_w"], np.float64)
    for u in range(B):
        assert abs(logits[u] - lr[u]) <= TOL["bf16"] * np.linalg.norm(hw) * np.linalg.norm(Yr[u, :m]) + 1e-3, u
