"""The last layer of the stack in a training step: only the global rows go through its tail and back (csrc/bw_stack.h, StackRows), side by side in
tiles of their own.  Where that can go wrong: fewer global rows than a tile, a last tile that is partly empty, as many as queries
nearly, the last layer being the cross layer (no self layer), width 256, users without a token, more than one round of tiles before and fewer after.  The
workspace and every output start as NaN (bytes 0xFF), so that a row which nobody writes is not read either.  Oracle and bars as in test_gpu_backward."""
import pytest

import gpu_util
from test_gpu_backward import _bf16_case, _compare_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,users,m,k,n_self,L", [
    ("C2", 1, 1, 3, 1, 40), ("C2", 5, 8, 5, 2, 130), ("C2", 9, 8, 1, 0, 70), ("C3", 3, 16, 30, 1, 203), ("C3", 2, 8, 4, 0, 90),
    ("P1", 2, 4, 9, 1, 64), ("C3", 40, 4, 100, 1, 150)])
def test_global_rows_of_the_last_layer(monkeypatch, base, users, m, k, n_self, L):
    monkeypatch.setattr(gpu_util, "SENTINEL", 0xFF)
    case = _bf16_case(base, users=users, L=L, m=m, k_recent=k, n_self=n_self, ragged=True, len_lo=0, len_hi=L)
    case["lens"][0] = L
    if users > 4:
        case["lens"][1] = 0
    _compare_model("%s, %d users, m = %d, k = %d, %d self layers" % (base, users, m, k, n_self), case)
