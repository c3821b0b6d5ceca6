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


# Users in multiples of eight are dealt to the accelerator dies, others in a row: every user's candidates score as the user's alone do, bit for bit
@pytest.mark.parametrize("d,heads,U,C,m", [(64, 4, 8, 11, 4), (64, 4, 16, 40, 8), (128, 8, 8, 11, 4), (128, 8, 16, 40, 8), (128, 8, 7, 11, 4)])
def test_users_dealt_to_the_dies(d, heads, U, C, m):
    import paper_2505_04421_amd as lg
    cfg = synth.CONFIGS["C2"].replace(B=U, L=300, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=20, n_self=1, index=93)
    case = synth.make_case(cfg)
    model = lg.DeviceModel(cfg, case["weights"])
    n = np.random.default_rng(8).integers(0, 301, size=U).astype(np.int32)
    n[:2] = [0, 300]
    H, lens = model.upload(case["H"]), torch.from_numpy(n).to(model.device)
    G = model.upload(np.random.default_rng(9).standard_normal((U, C, m, d)).astype(np.float32))
    ws = model.workspace(U, 300)

    def score(H, lens, G):
        u = H.shape[0]
        cache, Y, lo = model.kv_cache(u, 300), model.empty(u, C, m, d), model.empty(u, C, dtype=torch.float32)
        lg.longer_kv_cache_build(model.ccfg, model.weights, H, lens, u, 300, cache, ws)
        lg.longer_score_candidates(model.ccfg, model.weights, cache, lens, u, 300, G, C, Y, lo, ws)
        return Y.float().cpu().numpy(), lo.cpu().numpy()

    Y, lo = score(H, lens, G)
    assert np.isfinite(Y).all() and (np.abs(Y).max((1, 2, 3)) > 0).all()
    for u in range(U):
        Y1, lo1 = score(H[u:u + 1].contiguous(), lens[u:u + 1].contiguous(), G[u:u + 1].contiguous())
        assert np.array_equal(Y[u], Y1[0]) and np.array_equal(lo[u], lo1[0]), u
