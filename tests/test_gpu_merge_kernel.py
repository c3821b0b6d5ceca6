"""The merge kernel of width 128 (bf16, csrc/merge_kernel.h) at the sizes where its weight stream and its tiles can go wrong:
one to four blocks back to back in the stream, four (no chunk between the first and the last pair but one round), eight, sixteen
and 28 hidden chunks (the vectors fill their segment), every softmax window, one slot, exactly a workgroup's 128 slots and one
more group, workgroups that hold nothing but padding.  Against the fp64 oracle at the bf16 bar (per user 1e-2, a row twice that:
about ten bf16 roundings of 2^-9 per block on the way of a value)."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("heads,K,ffn_mult,layers,B,L,act", [
    (8, 1, 4, 1, 1, 1, "gelu_erf"), (8, 8, 1, 2, 3, 43, "gelu_erf"), (4, 16, 2, 3, 2, 64, "relu"), (8, 32, 7, 1, 5, 97, "gelu_erf"),
    (4, 4, 1, 4, 1, 132, "gelu_erf"), (8, 16, 4, 2, 4, 700, "gelu_erf"), (8, 8, 1, 1, 2, 130, "relu")])
def test_merge_and_inner_transformer(heads, K, ffn_mult, layers, B, L, act):
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=B, L=L, K=K, d=128, heads=8, inner_heads=heads, ffn_mult=ffn_mult, inner_layers=layers, act=act,
                                      k_recent=3, n_self=1, ragged=True, len_lo=0, len_hi=L, index=83)
    case = synth.make_case(cfg)
    case["lens"][0] = L
    if B > 3:
        case["lens"][1:3] = [0, min(L, 5)]     # whole workgroups of padding behind a few tokens
    case["H"][0] = synth.round_bf16(np.random.default_rng(12).standard_normal(case["H"][0].shape).astype(np.float32))
    r = _runner(case)
    _check("longer_token_merge", r.token_merge(), orc.token_merge(cfg, case["weights"]["inner"], case["H"], case["lens"]), TOL["bf16"])
    _check("longer_inner_transformer", r.inner_transformer(), orc.inner_transformer(cfg, case["weights"]["inner"], case["H"], case["lens"]), TOL["bf16"])


@pytest.mark.parametrize("d,K,L", [(128, 8, 250), (128, 16, 203), (64, 4, 250), (64, 32, 130)])
def test_padding_in_many_workgroups(d, K, L):
    """More workgroups than start at once ask whether they are all padding before they ask for rows, and all threads write such a workgroup's zeros: the same users again
    and again, empty ones in between and at the end (the last workgroup is partly empty as well), each copy against the oracle's one result.  Outputs sit between guard
    bands and hold no zeros beforehand."""
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=7, L=L, K=K, d=d, heads=d // 16, inner_heads=d // 16, ffn_mult=2, inner_layers=1, k_recent=3, n_self=1, ragged=True,
                                      len_lo=0, len_hi=L, index=92)
    case = synth.make_case(cfg)
    case["lens"][:] = [L, 0, 3, L // 2, 0, 1, 0]
    case["H"][0] = synth.round_bf16(np.random.default_rng(17).standard_normal(case["H"][0].shape).astype(np.float32))
    inner, n = case["weights"]["inner"], 7
    refs = orc.token_merge(cfg, inner, case["H"], case["lens"]), orc.inner_transformer(cfg, inner, case["H"], case["lens"])
    copies = 900 * 128 // (n * cfg.T * K) + 1
    case.update(cfg=cfg.replace(B=n * copies), H=np.tile(case["H"], (copies, 1, 1)), lens=np.tile(case["lens"], copies), G=np.tile(case["G"], (copies, 1, 1)))
    assert n * copies * cfg.T * K > 768 * 128
    r = _runner(case)
    for name, got, ref in (("M", r.token_merge(), refs[0]), ("Z", r.inner_transformer(), refs[1])):
        for i in range(copies):
            _check("%s, copy %d" % (name, i), got[n * i:n * (i + 1)], ref, TOL["bf16"])
