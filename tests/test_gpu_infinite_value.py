"""GPU test of an infinite value in the newest log entry: the column it belongs to comes out
as the recurrence has it (an infinity, or NaN where infinities of both signs meet), whatever
the live length leaves idle in the replay, and every other column is untouched.

Keys, queries, the bonus and the initial state are positive, so the recurrence's column is
an infinity of known sign until the delta rule subtracts one from it."""

import numpy as np
import pytest
import torch

from oracle import eager as OE
from paper_2608_15533_amd import workloads as W

from gpu_harness import TOL_F32_STATE, D, oracle_step, rel, to_dev, token

pytestmark = pytest.mark.gpu

COL = 5                                    # the value column of the infinity
LIVE = {8: (1, 2, 3, 5, 7), 24: (17, 18, 23), 40: (33, 35, 39)}   # interval: live lengths
CASES = [("gdn", 128, 128, "f32"), ("kda", 64, 64, "bf16"), ("rwkv6", 128, 64, "bf16"),
         ("linattn", 64, 128, "f32"), ("retnet", 128, 128, "bf16"), ("gla", 128, 128, "f32"),
         ("gla", 64, 64, "bf16")]


def _same_class(got, ref):
    """Infinities by sign and NaN in the same places."""
    for f in (np.isposinf, np.isneginf, np.isnan):
        np.testing.assert_array_equal(f(got), f(ref))


def _check(got, ref):
    rest = np.arange(ref.shape[-1]) != COL
    _same_class(got[..., COL], ref[..., COL])
    assert rel(got[..., rest], ref[..., rest]) <= TOL_F32_STATE


@pytest.mark.parametrize("path", ["step", "split2", "split4", "fused2", "fused4"])
@pytest.mark.parametrize("op,dk,dv,inp", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_infinite_newest_value(op, dk, dv, inp, path):
    dl, B, H = D(), 1, 2
    rng = np.random.default_rng(dk + dv + OE.OPS.index(op))
    for M, lengths in LIVE.items():
        desc = dl.make_desc(op, B, H, dk, dv, M, inp)
        ws = dl.tiled_workspace(desc, B)
        w = W.Workload("inf", 1, op, B, H, dk, dv, M, M + 1, in_dtype=inp)
        xs = [W.step_inputs(w, t) for t in range(M + 1)]
        for x in xs:
            for n in "qk":                 # positive and of length 1 (a stable delta rule)
                x[n] = np.abs(x[n]) + 0.01
                x[n] /= np.linalg.norm(x[n], axis=-1, keepdims=True)
                x[n] = W.round_bf16(x[n])
            x["v"] = np.abs(x["v"])
        u = None if op != "rwkv6" else np.full((H, dk), 0.5, np.float32)
        S0 = rng.uniform(0.01, 0.05, (B, H, dk, dv)).astype(np.float32)
        for L in lengths:
            x_inf = dict(xs[L - 1], v=xs[L - 1]["v"].copy())
            x_inf["v"][..., COL] = np.inf
            st, S = dl.DeltaLogState(desc, to_dev(S0, torch.float32)), S0.astype(np.float64)
            o = torch.empty((B, H, dv), dtype=torch.float32, device="cuda")

            def step(x):
                if path == "step":
                    dl.dl_append_step(desc, st, token(desc, x, u), o)
                else:
                    dl.dl_append_step_tiled(desc, st, token(desc, x, u), o,
                                            value_tiles=int(path[5:]),
                                            split_replay=path.startswith("split"), workspace=ws)
                return o.cpu().numpy()

            with np.errstate(invalid="ignore", over="ignore"):
                for t, x in enumerate(xs[: L - 1] + [x_inf]):
                    got = step(x)
                    S, ref = oracle_step(op, S, {k: None if a is None else a.astype(np.float64)
                                                 for k, a in x.items()}, u)
                _check(got, ref)
                q = to_dev(xs[L]["q"], torch.bfloat16 if inp == "bf16" else torch.float32)
                dl.dl_readout(desc, st, q, o)
                _check(o.cpu().numpy(),
                       np.einsum("bhi,bhij->bhj", xs[L]["q"].astype(np.float64), S))
                # one token more: an append, or the merge where the log is full
                x = {k: None if a is None else a.astype(np.float64) for k, a in xs[L].items()}
                S_next, ref = oracle_step(op, S, x, u)
                _check(step(xs[L]), ref)
                if L < M - 1 and op in OE.DELTA_OPS:      # the corrected value it appends
                    Sd = OE.row_decay(x["lam"], dk, op in OE.PER_KEY_OPS) * S
                    b = x["beta"][..., None] * (x["v"] - np.einsum("bhi,bhij->bhj", x["k"], Sd))
                    _check(st.u_log[:, :, L].cpu().numpy(), b)
                dl.dl_merge(desc, st)
                _check(st.S.cpu().numpy(), S_next)
            assert int(st.err.item()) == 0
