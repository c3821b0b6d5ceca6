"""The one-wave-per-tile STACK / SCORE kernels at d = 128 and d = 256 stay in the library as the fallback
of the two-waves-per-tile kernels (wider query sets, LDS limits) and as their comparison.  With
LONGER_DISABLE_PAIR_KERNELS=1 every launch uses them; the switch is read once per process, so the parity
cases that exercise those shapes run once more in ONE child process with it set."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASES = ("test_c3_bf16_all_entry_points or test_c5_bf16_serving or test_bf16_other_head_widths "
         "or test_bf16_d256_forward_entry_points or test_parameters_packed_once_equal_packing_per_call")


@pytest.mark.gpu
def test_parity_with_the_pair_kernels_switched_off():
    env = dict(os.environ, LONGER_DISABLE_PAIR_KERNELS="1")
    r = subprocess.run([sys.executable, "-u", "-m", "pytest", os.path.join(ROOT, "tests", "test_gpu_parity.py"),
                        "-x", "-q", "-m", "gpu", "-k", CASES, "--timeout", "300", "--timeout-method", "thread",
                        "-p", "no:cacheprovider"],
                       cwd=ROOT, env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=900)
    tail = "\n".join(r.stdout.splitlines()[-25:])
    assert r.returncode == 0, tail
    assert " passed" in tail and "failed" not in tail, tail


# Scoring more candidates than the few-tiles kernels take (512 tiles, 768 at d = 128) runs the same rows through the
# two-wave (d = 128 / 256) or one-wave (d = 64) kernels: both against the oracle for the candidates at the ends of the
# list, and against each other, a call of 40 candidates at a time, for all of them.  Users dealt to the dies (8) and not (3);
# one row more than whole tiles, rows that end inside a tile, m = 32 (one candidate fills a tile).
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,U,C", [(64, 4, 4, 3, 1367), (64, 2, 2, 8, 1025), (128, 8, 8, 1, 2049), (128, 4, 32, 8, 65),
                                           (256, 8, 8, 3, 343), (256, 16, 16, 8, 65), (128, 8, 8, 1, 3073), (128, 4, 32, 8, 97),
                                           (256, 8, 8, 3, 683), (256, 16, 16, 8, 129)])
def test_many_candidates_equal_the_same_candidates_in_short_lists(d, heads, m, U, C):
    import numpy as np
    import torch
    import longer_synth as synth
    import paper_2505_04421_amd as lg
    from oracle import longer_oracle as orc
    cfg = synth.CONFIGS["C2"].replace(B=U, L=150, d=d, heads=heads, inner_heads=heads, m=m, k_recent=9, n_self=2, C=C, ragged=True,
                                      len_lo=1, len_hi=150, index=71)
    case = synth.make_case(cfg)
    model = lg.DeviceModel(cfg, case["weights"])
    H, lens = model.upload(case["H"]), torch.from_numpy(case["lens"].astype(np.int32)).to(model.device)
    g = np.random.default_rng(5).standard_normal((U, C, m, d)).astype(np.float32)
    G = model.upload(g)
    ws, cache = model.workspace(U, cfg.L), model.kv_cache(U, cfg.L)
    lg.longer_kv_cache_build(model.ccfg, model.weights, H, lens, U, cfg.L, cache, ws)

    def score(Gc):
        n = Gc.shape[1]
        Y, lo = model.empty(U, n, m, d), model.empty(U, n, dtype=torch.float32)
        lg.longer_score_candidates(model.ccfg, model.weights, cache, lens, U, cfg.L, Gc.contiguous(), n, Y, lo, ws)
        return Y.float().cpu().numpy().astype(np.float64), lo.cpu().numpy().astype(np.float64)
    Y, lo = score(G)
    step = 40 if m * U * 40 < 32 * 256 else 4
    parts = [score(G[:, i:i + step]) for i in range(0, C, step)]
    Y2, lo2 = np.concatenate([a for a, _ in parts], 1), np.concatenate([b for _, b in parts], 1)
    rel = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)
    # two bf16 evaluations, each within 1e-2 of the exact result (the parity tests' bar)
    assert rel(Y, Y2) < 1e-2 and rel(lo, lo2) < 2e-2, (rel(Y, Y2), rel(lo, lo2))
    ends = [0, 1, C - 2, C - 1]
    Gr = G[:, ends].float().cpu().numpy()
    for i, c in enumerate(ends):
        Yr, lr = orc.forward(cfg, case["weights"], case["H"], Gr[:, i], case["lens"])
        for got in (Y, Y2):
            assert rel(got[:, c], Yr[:, :m]) < 1e-2, (c, rel(got[:, c], Yr[:, :m]))
        # (a logit is a sum of m d products of either sign: its error goes with the logits' spread over the list, not with how
        # near to zero one of them happens to come; 3e-2 of it is the parity tests' bar for a batch of logits)
        for got in (lo, lo2):
            assert np.abs(got[:, c] - lr).max() < 3e-2 * np.sqrt(np.mean(lo ** 2)), (c, got[:, c], lr)


# The reduced stack of users with at most two tiles (m + k <= 64), bf16, d = 64 / 128: one and two tiles, rows that end inside
# them, users without a token, every mask and query strategy; and the same model with one query more than two tiles hold
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,k,extra", [(64, 4, 4, 32, {}), (64, 2, 1, 5, dict(gmask="causal")), (64, 4, 8, 56, {}), (64, 4, 8, 57, {}),
                                               (128, 8, 8, 24, dict(k_uniform=10)), (128, 4, 32, 32, dict(gmask="causal")), (128, 8, 2, 31, {}),
                                               (128, 8, 8, 57, {})])
def test_stack_of_at_most_two_tiles(d, heads, m, k, extra):
    import numpy as np
    import longer_synth as synth
    from test_gpu_parity import _entry_points, TOL
    cfg = synth.CONFIGS["C2"].replace(B=5, L=200, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, n_self=3, ragged=True,
                                      len_lo=0, len_hi=200, index=73, **extra)
    case = synth.make_case(cfg)
    case["lens"][:3] = [200, 0, 9]
    _entry_points(case, TOL["bf16"], with_inner=False, logits_by_terms=True)


# The few-tiles kernels where the hidden chunks do not fill the waves evenly (1 to 10 chunks for four or eight waves), and more
# key tiles than are on their way at once (ten, and users with none, one and five): every entry point and serving
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,ffn_mult", [(64, 4, 1), (64, 4, 3), (64, 2, 5), (128, 8, 1), (256, 8, 1), (256, 16, 2)])
def test_few_tiles_with_any_number_of_hidden_chunks_and_key_tiles(d, heads, ffn_mult):
    import longer_synth as synth
    from test_gpu_parity import _entry_points, _serving, TOL
    cfg = synth.CONFIGS["C2"].replace(B=4, L=1200, K=4, d=d, heads=heads, inner_heads=heads, m=4, k_recent=40, n_self=1, ffn_mult=ffn_mult,
                                      C=11, ragged=True, len_lo=0, len_hi=1200, index=79)
    case = synth.make_case(cfg)
    case["lens"][:] = [1200, 0, 20, 633]
    _entry_points(case, TOL["bf16"], with_inner=False, logits_by_terms=True)
    _serving(case, TOL["bf16"], logits_by_terms=True)


# The reduced stack of users with up to four tiles (m + k <= 128), bf16, d = 128 / 256: two tiles (256), three, four, rows that end
# inside a tile, users without a token and with fewer tokens than query slots, every mask and query strategy, one hidden chunk a wave
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,k,extra", [(128, 8, 8, 57, {}), (128, 4, 8, 88, dict(gmask="causal")), (128, 8, 32, 96, {}), (128, 8, 4, 93, dict(k_uniform=40)),
                                               (128, 4, 2, 101, dict(q_learnable=True)), (256, 8, 1, 5, {}), (256, 16, 8, 56, dict(gmask="causal")),
                                               (256, 8, 8, 64, dict(k_uniform=20)), (256, 16, 8, 100, {}), (256, 8, 32, 96, dict(ffn_mult=1)),
                                               (256, 8, 8, 100, dict(q_learnable=True, gmask="causal"))])
def test_stack_of_up_to_four_tiles(d, heads, m, k, extra):
    import longer_synth as synth
    from test_gpu_parity import _entry_points, TOL
    cfg = synth.CONFIGS["C2"].replace(B=5, L=700, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, n_self=2, ragged=True,
                                      len_lo=0, len_hi=700, index=83, **extra)
    case = synth.make_case(cfg)
    case["lens"][:4] = [700, 0, 9, 260]
    _entry_points(case, TOL["bf16"], with_inner=False, logits_by_terms=True)


# Workgroups without a row to work on: key tiles past a user's last merged token are not projected (workspace and cache start as
# NaN, 40 key tiles a user, of which users here need 40, 1, none and 2), padded raw tokens of the input generation come out as zeros
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,heads,k", [("f32", 32, 2, 9), ("bf16", 64, 4, 40), ("bf16", 64, 4, 90), ("bf16", 128, 8, 100), ("bf16", 256, 8, 40)])
def test_workgroups_of_missing_rows_only(dtype, d, heads, k):
    import numpy as np
    import torch
    import longer_synth as synth
    import paper_2505_04421_amd as lg
    from oracle import longer_oracle as orc
    from test_gpu_parity import TOL, _check
    cfg = synth.CONFIGS["C2"].replace(dtype=dtype, B=4, L=5000, K=4, d=d, heads=heads, inner_heads=heads, m=4, k_recent=k, n_self=1, C=6, ragged=True,
                                      len_lo=0, len_hi=5000, index=89)
    case = synth.make_case(cfg)
    case["lens"][:] = [5000, 3, 0, 130]
    model = lg.DeviceModel(cfg, case["weights"])
    H, G, lens = model.upload(case["H"]), model.upload(case["G"]), torch.from_numpy(case["lens"].astype(np.int32)).to(model.device)
    Gc = model.upload(case["G_cand"])
    ws, cache = model.workspace(4, cfg.L).fill_(255), model.kv_cache(4, cfg.L).fill_(255)
    Y, lo = model.empty(4, cfg.n, d), model.empty(4, dtype=torch.float32)
    lg.longer_forward(model.ccfg, model.weights, H, G, lens, 4, cfg.L, Y, lo, ws)
    ref, _ = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    _check("longer_forward Y", Y.float().cpu().numpy().astype(np.float64), ref, TOL[dtype])
    ws.fill_(255)
    lg.longer_kv_cache_build(model.ccfg, model.weights, H, lens, 4, cfg.L, cache, ws)
    Yg, ls = model.empty(4, cfg.C, 4, d), model.empty(4, cfg.C, dtype=torch.float32)
    lg.longer_score_candidates(model.ccfg, model.weights, cache, lens, 4, cfg.L, Gc, cfg.C, Yg, ls, ws)
    ref, _ = orc.score_candidates(cfg, case["weights"], orc.kv_cache_build(cfg, case["weights"], case["H"], case["lens"]), case["G_cand"])
    _check("scores", Yg.float().cpu().numpy().astype(np.float64).reshape(-1, 4, d), ref.reshape(-1, 4, d), TOL[dtype])
    if d == 64:
        inp = synth.make_input_case(cfg, 32)
        inp["lens"][:] = case["lens"]
        pos = np.arange(cfg.L)[None, :, None]
        g = np.random.default_rng(3)
        E, td = (np.where(pos < inp["lens"][:, None, None], synth.round_bf16(g.standard_normal((4, cfg.L, 32)).astype(np.float32)), np.float32("nan"))
                 for _ in range(2))
        mlp = {n: model.upload(v) for n, v in inp["mlp"].items()}
        iw = lg.CInputWeights(**{n: v.data_ptr() for n, v in mlp.items()})
        X = model.empty(4, cfg.L, d).fill_(float("nan"))
        lg.longer_input_generation(model.ccfg, iw, model.upload(E), model.upload(td), lens, 4, cfg.L, 32, X, ws)
        got, ref = X.float().cpu().numpy().astype(np.float64), orc.input_generation(cfg, inp["mlp"], E, td, inp["lens"])
        for u, n in enumerate(inp["lens"]):
            assert not got[u, n:].any()
            if n:
                assert np.linalg.norm(got[u, :n] - ref[u, :n]) <= TOL[dtype] * np.linalg.norm(ref[u, :n])


# Full precision at width 32 in small launches: one and two tiles of query rows, the cross layer's keys made in the stack's launch
# (at most 64 global and merged tokens) and not, groups of every register window, hidden chunks below, at and past four, users without a
# token; and one merge with more tiles than the small kernel takes
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,K,L,ffn_mult,extra", [(2, 8, 4, 64, 4, {}), (8, 24, 1, 56, 1, dict(gmask="causal")), (8, 25, 8, 457, 3, {}), (2, 62, 4, 249, 5, {}),
                                                    (4, 9, 16, 970, 7, dict(act="relu")), (32, 32, 32, 1500, 4, dict(k_uniform=20)), (2, 20, 2, 131, 4, dict(q_learnable=True)),
                                                    (2, 8, 4, 5000, 4, {})])
def test_full_precision_small_launches(m, k, K, L, ffn_mult, extra):
    import longer_synth as synth
    from test_gpu_parity import _entry_points, TOL
    cfg = synth.CONFIGS["C1"].replace(B=5, L=L, K=K, m=m, k_recent=k, n_self=2, inner_layers=2, ffn_mult=ffn_mult, ragged=True, len_lo=0, len_hi=L,
                                      index=97, **extra)
    case = synth.make_case(cfg)
    case["lens"][:4] = [L, 0, 1, min(L, 40)]
    _entry_points(case, TOL["f32"], with_inner=False, logits_by_terms=True)


# The InnerTrans blocks and both merges at width 256 (a feature tile per wave, four tiles a workgroup): groups of every register window, lengths
# that are no multiple of K, workgroups that end inside a user, hold several or nothing but padding, one and two blocks, both head widths
@pytest.mark.gpu
@pytest.mark.parametrize("heads,K,B,L,layers,extra", [(8, 8, 5, 333, 1, {}), (16, 16, 3, 700, 2, {}), (8, 32, 2, 129, 1, dict(ffn_mult=1)), (16, 1, 3, 50, 1, {}),
                                                      (8, 4, 7, 31, 2, dict(act="relu")), (16, 2, 1, 1, 1, {})])
def test_merge_of_width_256(heads, K, B, L, layers, extra):
    import numpy as np
    import longer_synth as synth
    from test_gpu_parity import _entry_points, TOL
    cfg = synth.CONFIGS["C2"].replace(B=B, L=L, K=K, d=256, heads=8, inner_heads=heads, m=2, k_recent=5, n_self=1, inner_layers=layers, ragged=True, len_lo=0,
                                      len_hi=L, index=101, **extra)
    case = synth.make_case(cfg, pad_value=float("nan"))
    case["lens"][0] = L
    case["H"][0] = synth.round_bf16(np.random.default_rng(3).standard_normal(case["H"][0].shape).astype(np.float32))
    if B > 2:
        case["lens"][1] = 0
        case["H"][1] = np.float32("nan")
    _entry_points(case, TOL["bf16"], with_inner=True, logits_by_terms=True)


# The reduced stack layer by layer (few tiles: the next layer's K and V alternate between two places, so both parities of n_self, and
# none) and the same users repeated until the one-launch plan takes the call; also a workspace one byte short of the layered plan's
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,k,n_self,extra", [(64, 4, 8, 57, 3, {}), (64, 2, 4, 120, 0, dict(gmask="causal")), (128, 8, 8, 100, 3, {}), (128, 4, 32, 33, 1, {}),
                                                      (128, 8, 8, 88, 2, dict(k_uniform=40)), (128, 8, 8, 150, 3, {}), (256, 8, 8, 57, 3, dict(q_learnable=True)),
                                                      (256, 16, 32, 96, 1, dict(gmask="causal"))])
def test_stack_layer_by_layer_and_in_one_launch(d, heads, m, k, n_self, extra):
    import numpy as np
    import torch
    import longer_synth as synth
    import paper_2505_04421_amd as lg
    from oracle import longer_oracle as orc
    from gpu_util import GuardedModel, check_all_guards
    from test_gpu_parity import TOL, _check
    cfg = synth.CONFIGS["C2"].replace(B=5, L=500, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, n_self=n_self, ragged=True, len_lo=0,
                                      len_hi=500, index=103, **extra)
    case = synth.make_case(cfg)
    case["lens"][:4] = [500, 0, 9, 260]
    ref, ref_lo = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    lo_bar = 3e-2 * np.sqrt(np.mean(ref_lo ** 2))            # (the parity tests' bar for a batch of logits)
    model = GuardedModel(cfg, case["weights"])
    for copies in (1, 512 // (5 * ((m + k + 31) // 32)) + 1):
        B = 5 * copies
        H, G = (model.upload(np.concatenate([case[n]] * copies)) for n in ("H", "G"))
        lens = torch.from_numpy(np.concatenate([case["lens"]] * copies).astype(np.int32)).to(model.device)
        ws = model.workspace(B, cfg.L).fill_(255)
        for room in (ws, ws[:-1]) if (m + k) % 32 else (ws,):       # (whole tiles of rows: the smaller workspace is refused)
            Y, lo = model.empty(B, cfg.n, d), model.empty(B, dtype=torch.float32)
            lg.longer_forward(model.ccfg, model.weights, H, G, lens, B, cfg.L, Y, lo, room)
            check_all_guards()
            got, got_lo = Y.float().cpu().numpy().astype(np.float64), lo.cpu().numpy()
            for c in range(copies):
                _check("copy %d Y" % c, got[5 * c:5 * c + 5], ref, TOL["bf16"])
                assert np.abs(got_lo[5 * c:5 * c + 5] - ref_lo).max() < lo_bar


# K and V of one attention layer where a workgroup goes through several tiles (more than 512 of them at width 128, 256 at width 256): users whose
# key tiles are all needed, one, and none, the last tile with rows missing, tiles with and without global rows; rows in bf16 as this entry
# point takes them, and (the forward pass) in fp32
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,B,T", [(128, 8, 8, 75, 250), (128, 4, 32, 130, 97), (256, 8, 8, 40, 250), (256, 16, 1, 90, 95)])
def test_key_value_projection_of_many_tiles(d, heads, m, B, T):
    import numpy as np
    import longer_synth as synth
    from oracle import longer_oracle as orc
    from gpu_util import Runner
    from test_gpu_parity import TOL, _check
    cfg = synth.CONFIGS["C2"].replace(B=5, L=4 * T - 3, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=3, n_self=0, ragged=True, len_lo=0,
                                      len_hi=4 * T - 3, index=113)
    case = synth.make_case(cfg)
    case["lens"][:4] = [4 * T - 3, 0, 9, 2 * T]
    ref, _ = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    big = cfg.replace(B=B)
    many = dict(case, cfg=big, **{n: np.concatenate([case[n]] * (B // 5)) for n in ("H", "G", "lens")})
    Y, _ = Runner(many).forward()
    for c in range(B // 5):
        _check("copy %d" % c, Y[5 * c:5 * c + 5], ref, TOL["bf16"])
    M = synth.round_bf16(np.random.default_rng(7).standard_normal((5, T, d)).astype(np.float32))
    ref = orc.hybrid_cross_attn(cfg, case["weights"]["cross"], case["G"], M, case["lens"], L=cfg.L)
    X = Runner(many).cross(np.concatenate([case["G"]] * (B // 5)), np.concatenate([M] * (B // 5)))
    for c in range(B // 5):
        _check("copy %d, bf16 rows" % c, X[5 * c:5 * c + 5], ref, TOL["bf16"])


# Users of different length, many tiles: which tiles are needed is dealt out evenly, whatever key tiles a user has (4, 7 and 16; dividing the
# workgroups or not), with users of no token at the front, between others and at the end; more users than a workgroup has threads
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,B,T", [(128, 8, 8, 600, 120), (128, 8, 1, 85, 223), (256, 8, 8, 40, 504), (256, 16, 32, 550, 40)])
def test_key_value_projection_of_ragged_users(d, heads, m, B, T):
    import numpy as np
    import longer_synth as synth
    from oracle import longer_oracle as orc
    from gpu_util import Runner
    from test_gpu_parity import TOL, _check
    n = 10
    cfg = synth.CONFIGS["C2"].replace(B=n, L=T, K=1, d=d, heads=heads, inner_heads=heads, m=m, k_recent=3, n_self=0, ragged=True, len_lo=0, len_hi=T, index=131)
    case = synth.make_case(cfg)
    case["lens"][:] = [0, 0, T, 1, T // 2, 32 - m % 32, 0, 33, T - 1, 0]
    ref, _ = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    pick = np.concatenate([np.arange(n), np.random.default_rng(3).integers(0, n, size=B - 2 * n), np.arange(n)])
    many = dict(case, cfg=cfg.replace(B=B), **{k: case[k][pick] for k in ("H", "G", "lens")})
    Y, _ = Runner(many).forward()
    _check("all users", Y, ref[pick], TOL["bf16"])


# Users of one length, more tiles than workgroups: dealt out by a stride, of 7, 16 and 5 key tiles (dividing the workgroups or not, a last round
# that is nearly empty or full)
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,B,T", [(128, 8, 8, 80, 216), (128, 8, 4, 33, 500), (256, 8, 8, 40, 210), (256, 16, 2, 103, 158)])
def test_key_value_projection_of_many_users_of_one_length(d, heads, m, B, T):
    import numpy as np
    import longer_synth as synth
    from oracle import longer_oracle as orc
    from gpu_util import Runner
    from test_gpu_parity import TOL, _check
    n = 3
    cfg = synth.CONFIGS["C2"].replace(B=n, L=T, K=1, d=d, heads=heads, inner_heads=heads, m=m, k_recent=3, n_self=0, ragged=False, index=151)
    case = synth.make_case(cfg)
    ref, _ = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    pick = np.random.default_rng(9).integers(0, n, size=B)
    many = dict(case, cfg=cfg.replace(B=B), lens=None, **{k: case[k][pick] for k in ("H", "G")})
    Y, _ = Runner(many).forward()
    _check("all users", Y, ref[pick], TOL["bf16"])


# ... and evenly enough: with half of the tiles needed the launch takes clearly less than with all of them (0.52 and 0.58 times as long at widths
# 128 and 256; 0.71 and 0.92 where a workgroup met the same key tile of every user)
@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 256])
def test_key_value_projection_of_ragged_users_is_balanced(d):
    import numpy as np
    import torch
    import longer_synth as synth
    import paper_2505_04421_amd as lg
    B, T = 512, 504
    cfg = synth.CONFIGS["C2"].replace(B=B, L=T, K=1, d=d, heads=8, inner_heads=8, m=8, k_recent=8, n_self=0, index=137)
    model = lg.DeviceModel(cfg, synth.make_case(cfg.replace(B=1, L=4))["weights"])
    weights = model.pack()
    H, G = (torch.randn(*shape, device=model.device).to(model.tdtype) for shape in ((B, T, d), (B, 8, d)))
    lens = np.random.default_rng(5).permutation(np.linspace(T // 50, T, B)).astype(np.int32)
    ws, Y, logits = model.workspace(B, T), model.empty(B, 16, d), model.empty(B, dtype=torch.float32)
    ms = {}
    for name, n in (("all", np.full(B, T, np.int32)), ("half", lens)):
        n = torch.from_numpy(n).to(model.device)
        times = []
        for _ in range(15):
            lg.longer_stage_timing(True, stages=["kvproj"])
            lg.longer_forward(model.ccfg, weights, H, G, n, B, T, Y, logits, ws)
            times.append(lg.longer_stage_timing_read()["kvproj"][0])
            lg.longer_stage_timing(False)
        ms[name] = sorted(times)[7]
    print("K / V of %d users, width %d: %.1f us, half of the tiles %.1f us" % (B, d, 1e3 * ms["all"], 1e3 * ms["half"]), flush=True)
    assert ms["half"] < 0.66 * ms["all"]


# Query sets of more than four tiles in more tiles than the few-tiles plan takes: every layer's K and V in a launch of their own, the self layers' from
# fp32 rows, several tiles a workgroup, all of them needed whatever the lengths
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,m,k,B,extra", [(256, 8, 8, 150, 110, {}), (256, 16, 32, 101, 105, dict(gmask="causal")), (128, 8, 8, 150, 160, {}),
                                                 (256, 8, 8, 150, 105, dict(q_learnable=True)), (128, 4, 8, 129, 155, dict(k_uniform=60))])
def test_wide_query_sets_in_many_tiles(d, heads, m, k, B, extra):
    import numpy as np
    import longer_synth as synth
    from oracle import longer_oracle as orc
    from gpu_util import Runner
    from test_gpu_parity import TOL, _check
    n = 5
    cfg = synth.CONFIGS["C2"].replace(B=n, L=800, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, n_self=2, ragged=True, len_lo=0, len_hi=800,
                                      index=149, **extra)
    case = synth.make_case(cfg)
    case["lens"][:4] = [800, 0, 9, 500]
    ref, _ = orc.forward(cfg, case["weights"], case["H"], case["G"], case["lens"])
    pick = np.concatenate([np.arange(n), np.random.default_rng(7).integers(0, n, size=B - n)])
    many = dict(case, cfg=cfg.replace(B=B), **{name: case[name][pick] for name in ("H", "G", "lens")})
    Y, _ = Runner(many).forward()
    _check("all users", Y, ref[pick], TOL["bf16"])
