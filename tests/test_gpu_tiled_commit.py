"""GPU test of the value-tiled step's length commit: through whole cycles at the edges of
the log capacity (no log, one entry, one past a merge chunk, the largest), with slot lists
that leave slots out, the live lengths and the shared log entries equal the untiled
kernel's bit for bit after every step, and outputs and bases agree with it."""

import numpy as np
import pytest
import torch

from oracle import eager as OE
from paper_2608_15533_amd import workloads as W

from gpu_harness import D, to_dev, token

pytestmark = pytest.mark.gpu

# Two orders of the same fp32 sums (at most 128 rows and 63 entries): a few 1e-7 apart.
TOL = 4e-6


@pytest.mark.parametrize("split", [True, False], ids=["split", "fused"])
@pytest.mark.parametrize("op,dk,dv,M,nv", [
    ("gdn", 128, 128, 2, 4), ("gdn", 64, 64, 17, 4), ("kda", 128, 64, 18, 4),
    ("rwkv6", 64, 128, 64, 2), ("linattn", 128, 128, 1, 2), ("gla", 128, 128, 34, 2),
    ("retnet", 64, 64, 1, 4)])
def test_lengths_and_entries_follow_the_untiled_step(op, dk, dv, M, nv, split):
    dl = D()
    w = W.Workload(f"commit_{op}_{M}", 70 + M, op, 4, 3, dk, dv, M, M + 3)
    desc = dl.make_desc(op, w.B, w.H, dk, dv, M, w.in_dtype)
    S0 = to_dev(W.initial_state(w), torch.float32)
    a, b = dl.DeltaLogState(desc, S0), dl.DeltaLogState(desc, S0)
    ws = dl.tiled_workspace(desc, w.B)
    u = W.bonus(w)
    for t in range(w.steps):
        rows = np.arange(w.B) if t % 4 != 1 else np.array([3, 1])
        tok = token(desc, W.step_inputs(w, t), u, rows=rows)
        sl = torch.from_numpy(rows.astype(np.int32)).cuda()
        o1, o2 = (torch.empty((len(rows), w.H, dv), device="cuda") for _ in range(2))
        dl.dl_append_step(desc, a, tok, o1, slots=sl)
        dl.dl_append_step_tiled(desc, b, tok, o2, slots=sl, value_tiles=nv, split_replay=split,
                                workspace=ws)
        torch.cuda.synchronize()
        for k in ("len", "k_log", "lam_log", "err"):
            x, y = a.buffers()[k], b.buffers()[k]
            if x is not None:
                assert torch.equal(x, y), f"{k} after step {t}"
        assert OE.rel_fro(o2.cpu().numpy(), o1.cpu().numpy()) <= TOL
        assert OE.rel_fro(b.S.cpu().numpy(), a.S.cpu().numpy()) <= TOL
