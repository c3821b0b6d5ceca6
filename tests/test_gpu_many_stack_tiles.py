"""The training stack's row kernels beyond 512 tiles (their operands in LDS, csrc/bw_stack.h) against the same users in two batches of half the
size, which take the other variant: both multiply and add in the same order, and a batch twice as large halves every upstream gradient, a power of
two, so the raw tokens' and global tokens' gradients are the same bits times two; parameter gradients are sums over the batch in fp32, in another
order (1e-5, the bar of fp32 sums).  Users of full and of no length and rows that end inside a tile."""
import numpy as np
import pytest
import torch

import longer_synth as synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("d,heads,B,m,k,act", [(128, 8, 170, 8, 99, "gelu_erf"), (64, 4, 180, 4, 101, "relu"), (64, 2, 200, 4, 90, "gelu_erf")])
def test_a_batch_equals_its_halves(d, heads, B, m, k, act):
    import paper_2505_04421_amd as lg
    cfg = synth.CONFIGS["C2"].replace(B=B, L=40, K=4, d=d, heads=heads, inner_heads=heads, m=m, k_recent=k, n_self=2, act=act, ragged=True, len_lo=0,
                                      len_hi=40, index=91)
    assert B // 2 * (m + k) <= 512 * 32 < B * (m + k)
    case = synth.make_case(cfg)
    case["lens"][:2] = [40, 0]
    labels = synth.draw_labels(cfg)

    def step(lo, hi):
        n = hi - lo
        model = lg.DeviceModel(cfg, case["weights"])
        dev, f32 = model.device, torch.float32
        lens = torch.from_numpy(case["lens"][lo:hi].astype(np.int32)).to(dev)
        H = model.upload(np.nan_to_num(case["H"][lo:hi]))
        bws = torch.empty(lg.longer_forward_backward_workspace_bytes(model.ccfg, n, cfg.L), dtype=torch.uint8, device=dev)
        dH, dG = torch.empty(n, cfg.L, d, dtype=f32, device=dev), torch.empty(n, m, d, dtype=f32, device=dev)
        grads = torch.empty(lg.longer_model_grad_floats(model.ccfg), dtype=f32, device=dev)
        loss, logits = torch.empty(4, dtype=f32, device=dev), torch.empty(n, dtype=f32, device=dev)
        lg.longer_forward_backward(model.ccfg, model.weights, H, model.upload(case["G"][lo:hi]), lens, n, cfg.L,
                                   torch.from_numpy(labels[lo:hi]).to(dev), loss, logits, dH, dG, grads, bws)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (logits, dH, dG, grads)]
    whole, a, b = step(0, B), step(0, B // 2), step(B // 2, B)
    for i in range(3):
        assert np.isfinite(whole[i]).all()
        assert np.array_equal(whole[i] * (1 if i == 0 else 2), np.concatenate([a[i], b[i]])), i
    both = (a[3].astype(np.float64) + b[3]) / 2
    assert np.linalg.norm(whole[3] - both) <= 1e-5 * np.linalg.norm(both)
