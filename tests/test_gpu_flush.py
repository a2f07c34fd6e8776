"""GPU test of the flush (dl_merge without a token) at every edge of its chunks of 16 log
entries and of the four entries a contraction step takes: one call over slots at live
lengths 0 to 63, against Eq. 7 in float64 on the same buffers.  The slot list leaves one slot
out, names one outside the state and one whose length is corrupt: those stay as they are and
the error word says so."""

import numpy as np
import pytest
import torch

from gpu_harness import D

pytestmark = pytest.mark.gpu

# One rounding per product and sum of at most 64 terms of like size, and decay factors from
# the hardware exponential (below 2e-6): a few 1e-7 observed.  A bf16 state is rounded to 8
# bits, so within 2^-8 of its norm.
TOL = {"f32": 3e-6, "bf16": 4e-3}
LIVE = (0, 1, 2, 3, 4, 5, 7, 8, 12, 15, 16, 17, 20, 31, 32, 33, 47, 48, 49, 60, 63)


@pytest.mark.parametrize("M", [16, 17, 64])
@pytest.mark.parametrize("inp,state", [("bf16", "f32"), ("f32", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 64), (64, 128), (128, 64)])
@pytest.mark.parametrize("op", ["gdn", "kda", "linattn", "rwkv6"])
def test_flush_at_chunk_edges(op, dk, dv, inp, state, M):
    dl = D()
    live = [n for n in LIVE if n < M]
    B, H, C = len(live) + 2, 3, M - 1
    desc = dl.make_desc(op, B, H, dk, dv, M, inp, state)
    width = dl.decay_width(desc)
    g = torch.Generator(device="cuda").manual_seed(M + dk + 2 * dv)
    z = lambda *s: torch.randn(s, generator=g, device="cuda")   # noqa: E731
    st = dl.DeltaLogState(desc, z(B, H, dk, dv))
    st.k_log.copy_(z(B, H, C, dk))
    st.u_log.copy_(z(B, H, C, dv))
    lam = torch.zeros((B, H, C, 1), device="cuda")
    if width:
        lam = torch.cumsum(-0.2 * z(B, H, C, width).abs(), 2)
        st.lam_log.copy_(lam[..., 0].transpose(1, 2) if width == 1 else lam)
    L = torch.tensor(live + [1, M + 3], dtype=torch.int32, device="cuda")   # left out, corrupt
    st.len.copy_(L[:, None].expand(B, H))
    before = {k: v.clone() for k, v in st.buffers().items() if v is not None}
    order = np.random.default_rng(M).permutation(len(live)).tolist()
    slots = torch.tensor(order[:2] + [B - 1] + order[2:] + [B], dtype=torch.int32, device="cuda")
    dl.dl_merge(desc, st, slots=slots)
    assert int(st.err.item()) == 3
    st.err.zero_()
    S, lam = before["S"].double(), lam.double()
    for b, n in enumerate(live):
        ell = lam[b, :, n - 1] if n else torch.zeros_like(lam[b, :, 0])
        ref = torch.exp(ell)[..., None] * S[b]
        if n:
            kd = torch.exp(ell[:, None] - lam[b, :, :n]) * before["k_log"][b, :, :n].double()
            ref = ref + kd.transpose(1, 2).contiguous() @ before["u_log"][b, :, :n].double()
        err = (st.S[b].double() - ref).norm() / ref.norm()
        assert err <= TOL[state], (n, float(err))
        assert int(st.len[b].abs().max()) == 0
    rest = slice(len(live), B)
    for k, v in before.items():
        x = st.buffers()[k]
        assert torch.equal(x[rest], v[rest]) if k in ("S", "len") else torch.equal(x, v), k
