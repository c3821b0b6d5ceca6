"""The merge kernel at width 64 (bf16, csrc/merge_kernel.h): a segment is four products long, so that every fragment of the next is requested under
it.  Two hidden chunks (no full round between the first and the last pair), four and fourteen (the vectors fill their segment), both activations (a chunk's
bias replaces values that the activation has to have taken), every softmax window, one slot, a workgroup's 128 slots and one more group, padding alone; from
the raw inputs as well.  Oracle and bar as in test_gpu_merge_kernel."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("heads,K,ffn_mult,layers,B,L,act", [
    (4, 1, 4, 1, 1, 1, "gelu_erf"), (4, 8, 1, 2, 3, 43, "relu"), (2, 16, 2, 3, 2, 64, "relu"), (4, 32, 7, 1, 5, 97, "gelu_erf"),
    (2, 4, 1, 4, 1, 132, "gelu_erf"), (4, 16, 4, 2, 4, 700, "relu"), (4, 8, 4, 1, 2, 130, "gelu_erf")])
def test_merge_and_inner_transformer(heads, K, ffn_mult, layers, B, L, act):
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=B, L=L, K=K, d=64, heads=4, inner_heads=heads, ffn_mult=ffn_mult, inner_layers=layers, act=act,
                                      k_recent=3, n_self=1, ragged=True, len_lo=0, len_hi=L, index=84)
    case = synth.make_case(cfg)
    case["lens"][0] = L
    if B > 3:
        case["lens"][1:3] = [0, min(L, 5)]     # whole workgroups of padding behind a few tokens
    case["H"][0] = synth.round_bf16(np.random.default_rng(13).standard_normal(case["H"][0].shape).astype(np.float32))
    r = _runner(case)
    _check("longer_token_merge", r.token_merge(), orc.token_merge(cfg, case["weights"]["inner"], case["H"], case["lens"]), TOL["bf16"])
    _check("longer_inner_transformer", r.inner_transformer(), orc.inner_transformer(cfg, case["weights"]["inner"], case["H"], case["lens"]), TOL["bf16"])


@pytest.mark.parametrize("d_e,B,L", [(32, 3, 77), (32, 2, 200)])
def test_input_generation_and_forward_from_inputs(d_e, B, L):
    from test_gpu_parity import test_forward_from_inputs, test_input_generation
    test_input_generation("C2", d_e, B, L)
    test_forward_from_inputs("C2", d_e, B, L)
