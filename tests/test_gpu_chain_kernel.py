"""The wave-per-head kernels (csrc/chain_kernel.h; bf16, heads of 16 features) on both sides of the line to the kernels that take
two heads a wave (csrc/quad_kernel.h): 256 tiles at width 128.  Both add in the same order, so the same rows come out bit for bit,
whichever kernel had them: candidates in a list of 1024 (256 tiles) and of 1028, for users with no, one, five and ten key tiles, every window of
the candidate's own softmax and hidden chunks that do not fill the waves' rounds."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("m,ffn_mult,L,gmask", [(8, 4, 1270, "full"), (8, 3, 600, "causal"), (16, 1, 25, "full"), (32, 2, 1270, "full"), (2, 4, 5, "full")])
def test_candidates_on_both_sides_of_the_line(m, ffn_mult, L, gmask):
    import paper_2505_04421_amd as lg
    cfg = synth.CONFIGS["C2"].replace(B=1, L=L, K=4, d=128, heads=8, inner_heads=8, m=m, k_recent=70, n_self=2, ffn_mult=ffn_mult, gmask=gmask, index=89)
    case = synth.make_case(cfg)
    model = lg.DeviceModel(cfg, case["weights"])
    ws, cache = model.workspace(1, L), model.kv_cache(1, L)
    H = model.upload(case["H"])
    few = 256 * 32 // m
    G = model.upload(np.random.default_rng(7).standard_normal((1, few + 4, m, 128)).astype(np.float32))
    for n in (L, 0):
        lens = torch.tensor([n], dtype=torch.int32, device=model.device)
        lg.longer_kv_cache_build(model.ccfg, model.weights, H, lens, 1, L, cache, ws)
        out = []
        for C in (few, few + 4):
            Y, lo = model.empty(1, C, m, 128), model.empty(1, C, dtype=torch.float32)
            lg.longer_score_candidates(model.ccfg, model.weights, cache, lens, 1, L, G[:, :C].contiguous(), C, Y, lo, ws)
            out.append((Y[:, :few].float().cpu().numpy(), lo[:, :few].cpu().numpy()))
        assert np.isfinite(out[0][0]).all() and np.abs(out[0][0]).max() > 0
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


# the stack of at most two tiles at width 64 (a wave per head there): against the oracle, one row, one tile, one more, two tiles
@pytest.mark.parametrize("m,k,n_self,ffn_mult", [(1, 1, 1, 1), (4, 28, 3, 3), (4, 29, 2, 4), (8, 56, 1, 6)])
def test_stack_of_width_64(m, k, n_self, ffn_mult):
    from test_gpu_parity import _entry_points, TOL
    cfg = synth.CONFIGS["C2"].replace(B=4, L=300, K=4, m=m, k_recent=k, n_self=n_self, ffn_mult=ffn_mult, ragged=True, len_lo=0, len_hi=300, index=90)
    case = synth.make_case(cfg)
    case["lens"][:] = [300, 0, 7, 131]
    _entry_points(case, TOL["bf16"], with_inner=False, logits_by_terms=True)
