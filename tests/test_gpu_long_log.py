"""GPU tests of the step, merge and readout kernels' builds for logs of more than 16 entries
(32 and 64, which the host picks from the merge interval; the whole log of a build is
replayed from registers, and a merge stages it in chunks of 32 entries).  Every operator
against the fp64 oracle at capacities of 17 (one entry past the build below), 31 and 47, a
forced merge through dl_merge on both sides of a chunk's end, readouts at the edges of the
builds, a bf16 state, and bitwise equality where every intermediate is exact."""

import numpy as np
import pytest
import torch

from oracle import eager as OE
from paper_2608_15533_amd import workloads as W

from gpu_harness import TOL_BF16_STATE, TOL_F32_STATE, D, Rollout, log, to_dev, token
from test_gpu_properties import dyadic_inputs, oracle_run, rel, run_deltalog

pytestmark = pytest.mark.gpu

WL = {"gdn": W.GDN_B64, "kda": W.KDA_B128, "rwkv6": W.RWKV6_B128,
      "linattn": W.LINATTN_B64, "retnet": W.RETNET_B64, "gla": W.GLA_B128}


def _check(r, what, tol=TOL_F32_STATE):
    e_flush = r.flush_and_check()
    log(f"{what}: max out err {r.err_out:.2e}, max state err {r.err_state:.2e} "
        f"({r.n_state_checks} merge checks), flush {e_flush:.2e}")
    assert r.device_error_word() == 0
    assert r.err_out <= tol, what
    assert r.err_state <= tol, what


@pytest.mark.parametrize("M", [18, 32, 48])
@pytest.mark.parametrize("op", list(WL))
def test_long_log_mid_size(op, M):
    """Full head shape, 3 slots, 2M+5 steps: two merges of a long log and a ragged cycle,
    every slot and every step against the oracle."""
    r = Rollout(WL[op], M=M, B=3, steps=2 * M + 5).run()
    assert r.n_state_checks == 2
    _check(r, f"{op} long M={M}")


@pytest.mark.parametrize("op", list(WL))
def test_long_log_bf16_state(op):
    """The 32-entry build with a bf16 dense state, M = 32."""
    M = 32
    r = Rollout(WL[op], M=M, B=3, steps=2 * M + 5, state_dtype="bf16").run()
    _check(r, f"{op} long M={M} bf16 state", tol=TOL_BF16_STATE)


@pytest.mark.parametrize("op", list(WL))
def test_long_log_forced_merge_mid_chunk(op):
    """M = 40: 25 appends (within the first chunk of the 64-entry build), then dl_merge with
    the next token (Eq. 6 at L = 25 < C = 39), then 20 more steps and a flush, against the
    eager oracle.  (Live lengths in the second chunk: test_forced_merge_and_readout.)"""
    dl = D()
    w = WL[op].with_(B=3)
    M = 40
    S0 = W.initial_state(w)
    xs = [W.step_inputs(w, t) for t in range(46)]
    u = W.bonus(w)
    desc = dl.make_desc(op, w.B, w.H, w.dk, w.dv, M, w.in_dtype)
    ref_o, ref_S = oracle_run(op, S0, xs, u)
    outs, st = run_deltalog(desc, S0, xs[:25], u)
    assert np.all(st.len.cpu().numpy() == 25)
    o = torch.empty((w.B, w.H, w.dv), dtype=torch.float32, device="cuda")
    dl.dl_merge(desc, st, token(desc, xs[25], u), o)
    torch.cuda.synchronize()
    e_o, e_S = rel(o.cpu().numpy(), ref_o[25]), rel(st.S.cpu().numpy(), ref_S[25])
    log(f"{op} forced merge at L = 25 of C = 39: out {e_o:.2e}, state {e_S:.2e}")
    assert e_o <= TOL_F32_STATE and e_S <= TOL_F32_STATE
    assert np.all(st.len.cpu().numpy() == 0)
    for t in range(26, 46):
        dl.dl_append_step(desc, st, token(desc, xs[t], u), o)
        torch.cuda.synchronize()
        assert rel(o.cpu().numpy(), ref_o[t]) <= TOL_F32_STATE, t
    dl.dl_merge(desc, st)
    torch.cuda.synchronize()
    assert rel(st.S.cpu().numpy(), ref_S[45]) <= TOL_F32_STATE
    assert int(st.err.item()) == 0


@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 64)])
@pytest.mark.parametrize("op", OE.OPS)
def test_long_log_exact_dyadic_bitwise(op, dk, dv):
    """M = 40 on inputs where every intermediate is exact in fp32 (one-hot keys, integer
    state and values, beta = 1, lambda = 0): 45 steps through the 64-entry build, outputs of
    every step and the base after the merge and after a flush equal the oracle bit for
    bit -- any indexing slip in either chunk shows."""
    B, H, M, steps = 2, 2, 40, 45
    S0, xs, u = dyadic_inputs(op, B, H, dk, dv, steps, seed=400 + dk + OE.OPS.index(op))
    for x in xs:
        if x["beta"] is not None:
            x["beta"][:] = 1.0          # integers stay integers over many writes
    desc = D().make_desc(op, B, H, dk, dv, M, "bf16")
    outs, st = run_deltalog(desc, S0, xs, u)
    ref_o, ref_S = oracle_run(op, S0, xs, u)
    for t in range(steps):
        np.testing.assert_array_equal(outs[t].astype(np.float64), ref_o[t], err_msg=f"step {t}")
    D().dl_merge(desc, st)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(st.S.cpu().numpy().astype(np.float64), ref_S[-1])


# Live length and interval: either side of the 32-entry chunk in the 64-entry build, and the
# largest and smallest lengths of each build.
EDGES = [(1, 64), (16, 18), (17, 18), (31, 32), (31, 64), (32, 33), (32, 64), (33, 34),
         (33, 64), (40, 64), (62, 64), (63, 64)]


@pytest.mark.parametrize("op,dk,dv,inp", [("gdn", 128, 128, "bf16"), ("kda", 128, 64, "f32"),
                                          ("kda", 64, 128, "f32"), ("linattn", 64, 64, "bf16"),
                                          ("rwkv6", 128, 128, "bf16"), ("gla", 128, 64, "bf16"),
                                          ("retnet", 64, 128, "bf16")])
def test_forced_merge_and_readout(op, dk, dv, inp):
    """L appends, a readout (which leaves every buffer as it is), then dl_merge with the next
    token, at every pair of EDGES: both outputs and the merged base against the oracle."""
    dl, B, H = D(), 2, 3
    w = W.Workload("edges", 9, op, B, H, dk, dv, 64, 65, in_dtype=inp)
    S0, u = W.initial_state(w), W.bonus(w)
    xs = [W.step_inputs(w, t) for t in range(w.steps)]
    ref_o, ref_S = oracle_run(op, S0, xs, u)
    it = torch.bfloat16 if inp == "bf16" else torch.float32
    o = torch.empty((B, H, dv), dtype=torch.float32, device="cuda")
    for L, M in EDGES:
        desc = dl.make_desc(op, B, H, dk, dv, M, inp)
        _, st = run_deltalog(desc, S0, xs[:L], u)
        assert np.all(st.len.cpu().numpy() == L)
        before = {k: v.clone() for k, v in st.buffers().items() if v is not None}
        dl.dl_readout(desc, st, to_dev(xs[L]["q"], it), o)
        ref = np.einsum("bhi,bhij->bhj", xs[L]["q"].astype(np.float64), ref_S[L - 1])
        assert rel(o.cpu().numpy(), ref) <= TOL_F32_STATE, (L, M)
        for k, v in before.items():
            assert torch.equal(st.buffers()[k], v), (k, L, M)
        dl.dl_merge(desc, st, token(desc, xs[L], u), o)
        assert rel(o.cpu().numpy(), ref_o[L]) <= TOL_F32_STATE, (L, M)
        assert rel(st.S.cpu().numpy(), ref_S[L]) <= TOL_F32_STATE, (L, M)
        assert np.all(st.len.cpu().numpy() == 0) and int(st.err.item()) == 0
