"""GPU test of the order in which the waves' partial sums are added: in pairs.  Each wave
contributes one row: 2^24 from one of them and 1 from every other.  Added in turn, every 1
after the 2^24 is rounded away (an error of up to one per wave); in pairs at most one is."""

import numpy as np
import pytest
import torch

from gpu_harness import D, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [8, 40])                   # 4 waves; 8 for 128x128 and M = 40
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 64), (64, 128), (128, 64)])
@pytest.mark.parametrize("path", ["readout", "step", "eager"])
def test_partial_sums_of_waves_are_added_in_pairs(path, dk, dv, M):
    dl = D()
    waves = 8 if dk == dv == 128 and M > 17 and path != "eager" else 4
    rows = [w * 64 // (dv // 4) for w in range(waves)]    # the first row of each wave
    B = waves                                             # slot b: the 2^24 in wave b
    S = np.zeros((B, 1, dk, dv), np.float32)
    S[:, 0, rows] = 1.0
    for b in range(B):
        S[b, 0, rows[b]] = 2.0 ** 24
    desc = dl.make_desc("linattn", B, 1, dk, dv, M, "f32")
    q = torch.ones((B, 1, dk), device="cuda")
    zero_k, zero_v = torch.zeros((B, 1, dk), device="cuda"), torch.zeros((B, 1, dv), device="cuda")
    o = torch.empty((B, 1, dv), device="cuda")
    st = dl.DeltaLogState(desc, to_dev(S, torch.float32))
    if path == "readout":
        dl.dl_readout(desc, st, q, o)
    elif path == "step":
        dl.dl_append_step(desc, st, dl.Token(desc, B, q, zero_k, zero_v, None), o)
    else:
        dl.dl_eager_step(desc, st.S, dl.Token(desc, B, q, zero_k, zero_v, None), o)
    err = np.abs(o.cpu().numpy().astype(np.float64) - (2.0 ** 24 + waves - 1)).max()
    assert err <= 2                                       # one unit in the last place of 2^24
