"""The FFN loops whose activation goes behind other chunks' or other row tiles' products, with either activation and hidden widths of one to three times the
rows' (the loops' entry and exit meet, an odd number of turns).  Two waves a tile (csrc/pair_kernel.h): scoring beyond 768 tiles at width 128 and 512 at 256; at 256 the
weight panels come in another order than they lie, but for the smallest hidden width and for GELU with heads of 16.  The stack's row tiles in halves (csrc/user_kernel.h):
three and four tiles of rows a user at width 256 (four with ReLU and heads of 16 together), more users than the launch-a-layer
plan takes; together at width 128.  Against the fp64 oracle at the bf16 bar; every row of a long list also against the same rows in short lists (other kernels)."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("d,heads,m,U,C,ffn_mult,act", [(128, 8, 8, 1, 3073, 1, "relu"), (128, 4, 32, 8, 97, 3, "gelu_erf"), (256, 8, 8, 3, 683, 3, "relu"),
                                                        (256, 16, 16, 8, 129, 2, "relu"), (256, 8, 32, 1, 513, 2, "gelu_erf"), (256, 8, 8, 8, 257, 1, "relu"),
                                                        (256, 16, 16, 3, 345, 3, "gelu_erf")])
def test_scoring_in_two_waves(d, heads, m, U, C, ffn_mult, act):
    import paper_2505_04421_amd as lg
    from test_gpu_parity import _check, TOL
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=U, L=150, d=d, heads=heads, inner_heads=heads, m=m, k_recent=9, n_self=2, C=C, ffn_mult=ffn_mult, act=act, ragged=True,
                                      len_lo=1, len_hi=150, index=93)
    assert U * -(-C * m // 32) > (768 if d == 128 else 512)
    case = synth.make_case(cfg)
    model = lg.DeviceModel(cfg, case["weights"])
    lens = torch.from_numpy(case["lens"].astype(np.int32)).to(model.device)
    G = model.upload(np.random.default_rng(16).standard_normal((U, C, m, d)).astype(np.float32))
    ws, cache = model.workspace(U, cfg.L), model.kv_cache(U, cfg.L)
    lg.longer_kv_cache_build(model.ccfg, model.weights, model.upload(case["H"]), lens, U, cfg.L, cache, ws)

    def score(Gc):
        n = Gc.shape[1]
        Y, lo = model.empty(U, n, m, d), model.empty(U, n, dtype=torch.float32)
        lg.longer_score_candidates(model.ccfg, model.weights, cache, lens, U, cfg.L, Gc.contiguous(), n, Y, lo, ws)
        return Y.float().cpu().numpy().astype(np.float64), lo.cpu().numpy().astype(np.float64)
    Y, lo = score(G)
    step = max(1, 32 * 256 // (m * U))
    Y2, lo2 = (np.concatenate(a, 1) for a in zip(*(score(G[:, i:i + step]) for i in range(0, C, step))))
    # two bf16 evaluations, each within the parity tests' bar of the exact result
    for c in range(C):
        assert np.linalg.norm(Y[:, c] - Y2[:, c]) < 2 * TOL["bf16"] * np.linalg.norm(Y2[:, c]), c
    assert np.abs(lo - lo2).max() < 6e-2 * np.sqrt(np.mean(lo2 ** 2))
    some = sorted({0, 1, C // 2, C - 2, C - 1})
    ref, lref = orc.score_candidates(cfg, case["weights"], orc.kv_cache_build(cfg, case["weights"], case["H"], case["lens"]), G[:, some].float().cpu().numpy())
    _check("rows", Y[:, some].reshape(-1, m, d), ref.reshape(-1, m, d), TOL["bf16"])
    assert np.abs(lo[:, some] - lref).max() < 3e-2 * np.sqrt(np.mean(lo ** 2))


@pytest.mark.parametrize("d,heads,m,k,B,ffn_mult,act", [(128, 8, 8, 57, 173, 1, "relu"), (128, 4, 4, 124, 131, 3, "gelu_erf"), (128, 8, 16, 93, 133, 3, "relu"),
                                                        (256, 8, 8, 64, 87, 3, "relu"), (256, 16, 8, 88, 86, 1, "gelu_erf"), (256, 8, 2, 99, 66, 1, "relu"),
                                                        (256, 16, 2, 103, 66, 3, "relu"), (256, 16, 32, 96, 65, 3, "gelu_erf")])
def test_stack_of_row_tiles_in_halves(d, heads, m, k, B, ffn_mult, act):
    from test_gpu_parity import _check, _runner, TOL
    from oracle import longer_oracle as orc
    tiles = -(-(m + k) // 32)
    assert 64 < m + k <= 128 and B * tiles > (512 if d == 128 else 256)      # one launch for the stack
    cfg = synth.CONFIGS["C2"].replace(B=B, L=300, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, n_self=2, inner_layers=1, ffn_mult=ffn_mult, act=act,
                                      ragged=True, len_lo=0, len_hi=300, index=94)
    case = synth.make_case(cfg)
    case["lens"][:4] = [300, 0, 1, 131]
    Y, logits = _runner(case).forward()
    assert np.isfinite(Y).all() and np.isfinite(logits).all()
    some = np.array([0, 1, 2, 3, B // 2, B - 1])
    ref, lref = orc.forward(cfg, case["weights"], case["H"][some], case["G"][some], case["lens"][some])
    _check("rows", Y[some], ref, TOL["bf16"])
    assert np.abs(logits[some] - lref).max() < 3e-2 * np.sqrt(np.mean(logits ** 2))
