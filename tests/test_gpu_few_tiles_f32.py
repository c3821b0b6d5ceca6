"""The full-precision small launches (csrc/few_f32_kernel.h) at the lines between one and two tiles of a user: query rows that fill one and one more,
keys that fill one, two, and one more each (the second tile's waves have rows, keys only, or nothing), rows and keys ending in every quarter of a tile;
users shorter than that and one without a token.  Oracle and tolerance as in test_gpu_parity."""
import numpy as np
import pytest

import longer_synth as synth
from test_gpu_parity import TOL, _entry_points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k,T", [(2, 30, 30), (2, 30, 31), (2, 31, 30), (2, 8, 62), (2, 8, 63), (8, 1, 9), (1, 15, 16), (4, 20, 21), (2, 40, 40)])
def test_one_and_two_tiles_of_rows_and_keys(m, k, T):
    cfg = synth.CONFIGS["C1"].replace(B=4, L=4 * T, K=4, m=m, k_recent=k, n_self=2, ragged=True, len_lo=0, len_hi=4 * T, index=151)
    case = synth.make_case(cfg)
    case["lens"][:3] = [4 * T, 0, 4 * (T - 1)]
    case["H"][2] = np.random.default_rng(17).standard_normal(case["H"][2].shape).astype(np.float32)
    case["H"][0] = np.random.default_rng(18).standard_normal(case["H"][0].shape).astype(np.float32)
    _entry_points(case, TOL["f32"], with_inner=False)
