"""The merge's last FFN product on the groups' sums (csrc/user_kernel.h: width 256, bf16, K = 8, 16 and 32, mean merge).  Where that can go wrong: every
K against every register window, K = 4 (stays token by token), groups with fewer tokens than K (masked start values, the divisor), users without a token, a
workgroup with nothing but padding beside one that has some, one slot, a last workgroup that is partly empty, one hidden chunk a wave and several, both
activations, one block and several in front of it, fp32 and bf16 merged tokens (stand-alone and inside longer_forward).  The same at width 128, where every token goes through
that product (csrc/merge_kernel.h).  Against the fp64 oracle at the bf16 bar."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("d,inner_heads,K,ffn_mult,layers,B,L,act", [
    (128, 8, 8, 4, 1, 1, 1, "gelu_erf"), (128, 4, 16, 1, 1, 3, 203, "relu"), (128, 8, 32, 2, 1, 5, 97, "gelu_erf"), (128, 8, 8, 3, 1, 6, 643, "gelu_erf"),
    (128, 8, 4, 4, 1, 3, 61, "gelu_erf"), (256, 8, 8, 1, 2, 3, 83, "gelu_erf"), (256, 16, 16, 4, 1, 6, 401, "gelu_erf"), (256, 8, 32, 2, 1, 3, 100, "relu"),
    (256, 16, 8, 2, 1, 1, 3, "relu")])
def test_group_sums(d, inner_heads, K, ffn_mult, layers, B, L, act):
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=B, L=L, K=K, d=d, heads=8, inner_heads=inner_heads, ffn_mult=ffn_mult, inner_layers=layers, act=act,
                                      k_recent=3, n_self=1, ragged=True, len_lo=0, len_hi=L, index=91)
    case = synth.make_case(cfg)
    case["lens"][0] = L
    if B > 3:
        case["lens"][1:4] = [0, min(L, 5), 0]
    case["H"][0] = synth.round_bf16(np.random.default_rng(14).standard_normal(case["H"][0].shape).astype(np.float32))
    r = _runner(case)
    _check("longer_token_merge", r.token_merge(), orc.token_merge(cfg, case["weights"]["inner"], case["H"], case["lens"]), TOL["bf16"])
    _check("longer_inner_transformer", r.inner_transformer(), orc.inner_transformer(cfg, case["weights"]["inner"], case["H"], case["lens"]), TOL["bf16"])
    Y, logits = r.forward()[:2]
    Yr, lr = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    _check("longer_forward", Y, Yr, TOL["bf16"])


@pytest.mark.parametrize("inner_heads,K,L,act", [(8, 8, 643, "gelu_erf"), (4, 16, 401, "relu"), (8, 32, 97, "gelu_erf")])
def test_group_sums_of_many_users(inner_heads, K, L, act):
    """Many rounds of workgroups, several of them with nothing but padding between others: the case's users again and again, the last workgroup partly empty, and
    each copy against the oracle's one result (a user's groups lie anywhere in a workgroup)."""
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=6, L=L, K=K, d=128, heads=8, inner_heads=inner_heads, ffn_mult=2, inner_layers=1, act=act, k_recent=3, n_self=1,
                                      ragged=True, len_lo=0, len_hi=L, index=91)
    case = synth.make_case(cfg)
    case["lens"][0] = L
    case["lens"][1:4] = [0, min(L, 5), 0]
    ref = orc.token_merge(cfg, case["weights"]["inner"], case["H"], case["lens"])
    copies = 3584 * 128 // (6 * -(-L // K) * K) + 1
    case["cfg"] = cfg.replace(B=6 * copies)
    case["H"] = np.tile(case["H"], (copies, 1, 1))
    case["lens"] = np.tile(case["lens"], copies)
    case["G"] = np.tile(case["G"], (copies, 1, 1))
    M = _runner(case).token_merge()
    for i in (0, 1, copies // 2, copies - 1):
        _check("copy %d" % i, M[6 * i:6 * i + 6], ref, TOL["bf16"])


@pytest.mark.parametrize("K,L,act", [(8, 83, "gelu_erf"), (16, 83, "relu"), (32, 100, "gelu_erf")])
def test_a_hidden_value_of_infinity(K, L, act):
    """A hidden unit whose bias is +infinity (each of its activations is infinite, W2 gives the sign): every feature of every group with a token is an infinity of
    that sign, not the NaN of infinity less infinity in the sum's rounding rest.  A group without a token stays zero."""
    from test_gpu_parity import _runner
    cfg = synth.CONFIGS["C2"].replace(B=3, L=L, K=K, d=256, heads=8, inner_heads=8, inner_layers=1, act=act, k_recent=3, n_self=1, ragged=True, len_lo=0, len_hi=L,
                                      index=91)
    case = synth.make_case(cfg)
    case["lens"][:] = [L, 0, K + 3]
    block = case["weights"]["inner"][0]
    sign = np.where(np.random.default_rng(15).random(256) < 0.5, -1.0, 1.0).astype(np.float32)
    block["b1"][5] = np.inf
    block["w2"][5] = 0.5 * sign
    M = _runner(case).token_merge()
    for u, n in enumerate(case["lens"]):
        groups = -(-int(n) // K)
        assert np.array_equal(M[u, :groups], np.broadcast_to(np.inf * sign, (groups, 256))), u
        assert not M[u, groups:].any(), u
