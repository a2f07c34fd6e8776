"""Performance cases: the decode work a user of this library has it do.

Each case drives the public entry points (``deltalog`` binding, ``decode.DecodeEngine``)
on seeded synthetic inputs with the distributions of ``workloads.py``.  Kinds:

``decode``     one merge cycle of one recurrent layer: M calls of ``dl_append_step``, each
               slot starting from its own live length (``fill``).  ``graph`` submits the
               cycle as one captured HIP graph, the way a serving loop submits small
               launches.  ``active`` < ``B`` steps a part of the slots through a slot
               list; with staggered logs the list orders all of them by live length.
``engine``     one token of a stack of layers through ``DecodeEngine`` (graphs on, slots
               admitted over several steps, so each step merges some of them).
``eager``      a few tokens of the dense recurrence, ``dl_eager_step``.
``lifecycle``  what surrounds decoding: appends, a read-only readout, a forced merge with
               the token, more appends, and the flush of every other slot (eviction).
``tiled``      one merge cycle through the value-tiled step with split replay, its
               scratch the caller's workspace or the library's own (``noalloc``).
"""

import math

import torch

from paper_2608_15533_amd import decode as E
from paper_2608_15533_amd import deltalog as D

OPS = ("gdn", "kda", "rwkv6", "linattn", "retnet", "gla")
DELTA = ("gdn", "kda")
PER_KEY = ("kda", "rwkv6", "gla")
EAGER_STEPS = 4


def _case(name, kind, op, B, H, dk, dv, M, inp="bf16", state="f32", fill="fresh", active=0,
          graph=False, layers=1, tiles=0, noalloc=False):
    c = {"kind": kind, "op": op, "B": B, "H": H, "dk": dk, "dv": dv, "M": M, "in": inp,
         "state": state, "fill": fill, "active": active or B, "graph": graph,
         "layers": layers, "tiles": tiles, "noalloc": noalloc}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest workload of the repository (one sequence, two heads, fp32
        # activations): the latency of a launch and of the kernel's dependent chain.
        _case("gdn_b1_h2_d64_graph", "decode", "gdn", 1, 2, 64, 64, 8, inp="f32", graph=True),
        # A short stack serving 8 sequences that were admitted at different times: the
        # interactive end of the decode loop (the loop's small batch).
        _case("engine_gdn_b8_l8", "engine", "gdn", 8, 32, 128, 128, 16, layers=8),
        # Odd everything: part of the slots, few heads, rectangular heads, fp32
        # activations, an interval that is no power of two.
        _case("linattn_7of11_h5_graph", "decode", "linattn", 11, 5, 64, 128, 13, inp="f32",
              fill="staggered", active=7, graph=True),
        # The single-layer workloads: scalar decay at a middling batch ...
        _case("gdn_b64", "decode", "gdn", 64, 32, 128, 128, 16),
        # ... 64 x 64 heads with per-key decay (16 KiB of state per head) ...
        _case("rwkv6_b128_d64", "decode", "rwkv6", 128, 40, 64, 64, 16),
        # ... and per-key decay with a log longer than one pass of the replay.
        _case("kda_b128_m32", "decode", "kda", 128, 32, 128, 128, 32),
        # The longest merge interval the library takes, on a ragged batch.
        _case("retnet_b33_m64", "decode", "retnet", 33, 16, 128, 128, 64),
        # The bf16 dense state, odd batch, slots at different points of their cycles.
        _case("gla_b100_bf16state", "decode", "gla", 100, 32, 128, 128, 16, state="bf16",
              fill="staggered"),
        # One layer of the serving stack: 256 staggered sequences (the largest launch).
        _case("gdn_b256_staggered", "decode", "gdn", 256, 32, 128, 128, 16, fill="staggered"),
        # The dense recurrence (prompt tails, or a model without the log).
        _case("eager_kda_b48", "eager", "kda", 48, 32, 128, 128, 1),
        # Eviction, checkpoint and speculative readouts around decoding.
        _case("lifecycle_kda_b40", "lifecycle", "kda", 40, 32, 128, 128, 16),
        # The value-tiled step with split replay and the library's own scratch.
        _case("tiled_gdn_b32_m8", "tiled", "gdn", 32, 32, 128, 128, 8, tiles=4, noalloc=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["engine", "eager", "lifecycle", "tiled", "tiled"])
    op = rng.choice(OPS)
    dk, dv = rng.choice([(128, 128)] * 3 + [(64, 64)] * 2 + [(64, 128), (128, 64)])
    H = rng.choice([2, 3, 5, 8, 16, 24, 32, 40])
    M = {"eager": 1, "tiled": _log_int(rng, 4, 16), "lifecycle": _log_int(rng, 4, 32)}.get(
        kind, _log_int(rng, 2, 64))
    B = _log_int(rng, 1, 64 if kind in ("engine", "tiled", "lifecycle") else 256)
    inp = rng.choice(["bf16"] * 3 + ["f32"])
    state = "f32" if kind == "tiled" else rng.choice(["f32"] * 3 + ["bf16"])
    fill = rng.choice(["fresh", "staggered"]) if kind in ("decode", "tiled") else "fresh"
    active = max(1, B - rng.randrange(0, B // 2 + 1)) if kind == "decode" and rng.random() < 0.3 else B
    layers = rng.randrange(2, 9) if kind == "engine" else 1
    graph = kind == "decode" and B * H <= 512 and rng.random() < 0.7
    c = _case("", kind, op, B, H, dk, dv, M, inp, state, fill, active, graph, layers,
              rng.choice([2, 4]) if kind == "tiled" else 0, kind == "tiled" and rng.random() < 0.5)
    limit = 0.7 * max(work(x)["bytes"] for x in listed())
    while work(c)["bytes"] > limit:
        c["B"] = max(1, c["B"] * 2 // 3)
        c["active"] = min(c["active"], c["B"])
    if c["noalloc"] and c["B"] * H * (M - 1) * 8 > D.DL_NOALLOC_SCRATCH_BYTES:
        c["noalloc"] = False
    return c


# ------------------------------------------------------------------ inputs
def _dl(c):
    return 0 if c["op"] == "linattn" else c["dk"] if c["op"] in PER_KEY else 1


def _norm(x):
    return x / x.norm(dim=-1, keepdim=True)


class _Draw:
    """Seeded device tensors with the distributions of ``workloads.py``."""

    def __init__(self, c, seed):
        self.c = c
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.it = torch.bfloat16 if c["in"] == "bf16" else torch.float32

    def z(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")

    def keys(self, *shape):
        op, x = self.c["op"], self.z(*shape)
        if op == "linattn":
            x = torch.nn.functional.elu(x) + 1
        return (x if op == "rwkv6" else _norm(x)).to(self.it)

    def decay(self, *lead):
        """Per-step log-decay [*lead] or [*lead, dk] (the last of ``lead`` is H)."""
        c, op = self.c, self.c["op"]
        if op == "linattn":
            return None
        if op == "retnet":
            h = torch.arange(c["H"], device="cuda")
            return torch.log1p(-(2.0 ** (-5.0 - 5.0 * h / c["H"]))).expand(*lead).contiguous()
        z = self.z(*lead) if op == "gdn" else self.z(*lead, c["dk"])
        if op == "gdn":
            return torch.nn.functional.logsigmoid(3.0 + 0.5 * z)
        if op == "kda":
            return -torch.nn.functional.softplus(z) / 16.0
        if op == "rwkv6":
            return -torch.exp(-0.5 + 0.5 * z)
        return torch.nn.functional.logsigmoid(z) / 16.0

    def tokens(self, T, n):
        """T steps of n rows: q, k [T,n,H,dk], v [T,n,H,dv], lam, beta (None if unused)."""
        c = self.c
        H = c["H"]
        return {"q": self.keys(T, n, H, c["dk"]), "k": self.keys(T, n, H, c["dk"]),
                "v": self.z(T, n, H, c["dv"]).to(self.it), "lam": self.decay(T, n, H),
                "beta": torch.sigmoid(self.z(T, n, H)) if c["op"] in DELTA else None}

    def bonus(self):
        c = self.c
        return 0.1 * self.z(c["H"], c["dk"]) if c["op"] == "rwkv6" else None

    def base(self, *lead):
        """The state a prefill leaves: [*lead, dk, dv] in the state dtype."""
        s = 0.02 * self.z(*lead, self.c["dk"], self.c["dv"])
        return s.to(torch.bfloat16) if self.c["state"] == "bf16" else s

    def log(self, live):
        """A log with ``live[b]`` entries per slot: k_log, u_log, lam_log (binding layout)."""
        c = self.c
        B, H, C, dl = c["B"], c["H"], c["M"] - 1, _dl(c)
        on = torch.arange(C, device="cuda")[None, :] < live[:, None]            # [B, C]
        k = self.keys(B, H, C, c["dk"]) * on[:, None, :, None]
        u = 0.5 * self.z(B, H, C, c["dv"]) * on[:, None, :, None]
        u = u if c["op"] in DELTA else u.to(self.it)
        lam = None
        if dl == 1:
            lam = torch.cumsum(self.decay(B, C, H), 1) * on[:, :, None]
        elif dl:
            lam = torch.cumsum(self.decay(B, C, H), 1).transpose(1, 2) * on[:, None, :, None]
        return k, u, None if lam is None else lam.contiguous()


def _steps(c):
    return {"decode": c["M"], "tiled": c["M"], "eager": EAGER_STEPS, "engine": 1,
            "lifecycle": c["M"] // 2 + 1 + c["M"] // 3}[c["kind"]]


def _live0(c, d):
    if c["fill"] == "staggered":
        return torch.randint(0, c["M"], (c["B"],), generator=d.g, device="cuda")
    return torch.zeros(c["B"], dtype=torch.long, device="cuda")


def _rows(c, d, live):
    """The slot list of the launches (None: all slots in order)."""
    if c["active"] < c["B"]:
        return torch.randperm(c["B"], generator=d.g, device="cuda")[: c["active"]].to(torch.int32)
    if c["fill"] == "staggered":                       # rows by live length, longest first
        return torch.argsort(live, descending=True, stable=True).to(torch.int32)
    return None


def _inputs(c, seed):
    """Everything a pass of a single-layer case reads, drawn in a fixed order."""
    d = _Draw(c, seed)
    x = {"S0": d.base(c["B"], c["H"])}
    live = _live0(c, d)
    x["live"], x["slots"] = live, _rows(c, d, live)
    if c["M"] > 1 and c["fill"] == "staggered":
        x["log"] = d.log(live)
    x["u"] = d.bonus()
    x["tok"] = d.tokens(_steps(c), c["active"])
    x["q"] = d.keys(c["active"], c["H"], c["dk"]) if c["kind"] == "lifecycle" else None
    return x


def _engine_steps(c):
    """(slots admitted before each step, steps) of an engine's start: an equal share of
    the slots per step over one merge cycle."""
    n = min(c["M"], c["B"])
    return [c["B"] * (t + 1) // n - c["B"] * t // n for t in range(n)]


# ------------------------------------------------------------------ the measured interface
def prepare(case, seed):
    c = case
    if c["kind"] == "engine":
        return _prepare_engine(c, seed)
    desc = D.make_desc(c["op"], c["B"], c["H"], c["dk"], c["dv"], c["M"], c["in"], c["state"])
    x = _inputs(c, seed)
    n, T, H = c["active"], _steps(c), c["H"]
    tk = x["tok"]
    at = lambda a, t: None if a is None else a[t]  # noqa: E731
    toks = [D.Token(desc, n, tk["q"][t], tk["k"][t], tk["v"][t], at(tk["lam"], t), at(tk["beta"], t),
                    x["u"]) for t in range(T)]
    s = {"case": c, "desc": desc, "toks": toks, "slots": x["slots"],
         "o": torch.zeros((T, n, H, c["dv"]), device="cuda")}
    if c["kind"] == "eager":
        s["S"] = x["S0"]
        return s
    st = D.DeltaLogState(desc, x["S0"])
    if "log" in x:
        for dst, src in zip((st.k_log, st.u_log, st.lam_log), x["log"]):
            if dst is not None:
                dst.copy_(src)
        st.len.copy_(x["live"].to(torch.int32)[:, None].expand(c["B"], H))
    s["st"] = st
    if c["kind"] == "lifecycle":
        s["q"], s["r"] = x["q"], torch.zeros((n, H, c["dv"]), device="cuda")
        s["evict"] = torch.arange(0, c["B"], 2, dtype=torch.int32, device="cuda")
    if c["kind"] == "tiled" and not c["noalloc"]:
        s["ws"] = D.tiled_workspace(desc, n)
    if c["graph"]:
        # A first call outside the capture loads the kernel; it steps a state of its own.
        D.dl_append_step(desc, D.DeltaLogState(desc), toks[0], s["o"][0], slots=s["slots"])
        s["g"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["g"]):
            _cycle(s)
    return s


def _prepare_engine(c, seed):
    d = _Draw(c, seed)
    desc = D.make_desc(c["op"], c["B"], c["H"], c["dk"], c["dv"], c["M"], c["in"], c["state"])
    eng = E.DecodeEngine(desc, c["layers"])
    u = d.bonus()
    for inp in eng.inputs:
        if u is not None:
            inp.u.copy_(u)
    active = 0
    for more in _engine_steps(c):
        S0 = [d.base(more, c["H"]) for _ in range(c["layers"])]
        for i in range(more):
            eng.admit([s[i] for s in S0])
        active += more
        _engine_write(c, d, eng, active)
        eng.schedule()
        eng.step()
    _engine_write(c, d, eng, active)
    return {"case": c, "eng": eng}


def _engine_write(c, d, eng, n):
    for inp in eng.inputs:
        x = d.tokens(1, n)
        inp.write(range(n), x["q"][0], x["k"][0], x["v"][0],
                  None if x["lam"] is None else x["lam"][0],
                  None if x["beta"] is None else x["beta"][0])


def _cycle(s):
    for tok, o in zip(s["toks"], s["o"]):
        D.dl_append_step(s["desc"], s["st"], tok, o, slots=s["slots"])


def _buffers(st):
    return {k: v for k, v in st.buffers().items() if v is not None and k != "err"}


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "engine":
        eng = s["eng"]
        eng.schedule()
        eng.step()
        return [{"o": o, **_buffers(st)} for o, st in zip(eng.outputs, eng.states)]
    desc = s["desc"]
    if kind == "eager":
        for tok, o in zip(s["toks"], s["o"]):
            D.dl_eager_step(desc, s["S"], tok, o, slots=s["slots"])
        return {"o": s["o"], "S": s["S"]}
    st, toks, o = s["st"], s["toks"], s["o"]
    if kind == "decode":
        if c["graph"]:
            s["g"].replay()
        else:
            _cycle(s)
    elif kind == "tiled":
        for tok, ot in zip(toks, o):
            if c["noalloc"]:
                D.dl_append_step_tiled_noalloc(desc, st, tok, ot, slots=s["slots"],
                                               value_tiles=c["tiles"])
            else:
                D.dl_append_step_tiled(desc, st, tok, ot, slots=s["slots"],
                                       value_tiles=c["tiles"], workspace=s["ws"])
    else:
        a = c["M"] // 2
        for t in range(a):
            D.dl_append_step(desc, st, toks[t], o[t], slots=s["slots"])
        D.dl_readout(desc, st, s["q"], s["r"], slots=s["slots"])
        D.dl_merge(desc, st, toks[a], o[a], slots=s["slots"])
        for t in range(a + 1, len(toks)):
            D.dl_append_step(desc, st, toks[t], o[t], slots=s["slots"])
        D.dl_merge(desc, st, slots=s["evict"])
        return {"o": o, "r": s["r"], **_buffers(st)}
    return {"o": o, **_buffers(st)}


def work(case):
    """Algorithmic bytes and FLOPs of one pass: a state is read once per token and
    written once per merge, a log entry is written once and read by every later token of
    its cycle."""
    c = case
    dk, dv, M, op = c["dk"], c["dv"], c["M"], c["op"]
    pin, ps, dl = (2 if c["in"] == "bf16" else 4), (2 if c["state"] == "bf16" else 4), _dl(c)
    delta = op in DELTA
    tok = pin * (2 * dk + dv) + 4 * dl + (4 if delta else 0) + 4 * dv
    S = ps * dk * dv
    entry = pin * dk + (4 if delta else pin) * dv + 4 * dl
    reads = 4 if delta else 2                                    # FLOPs per state element
    step = lambda L: (tok + S + L * entry,  # noqa: E731
                      dk * dv * reads + L * reads * (dk + dv))
    if c["kind"] == "eager":
        b, f = EAGER_STEPS * (tok + 2 * S), EAGER_STEPS * dk * dv * (reads + 3)
    elif c["kind"] == "lifecycle":
        a, e = M // 2, M // 3
        seq = [step(L) for L in range(a)] + [step(a)] + [step(L) for L in range(e)]
        b = sum(x[0] for x in seq) + (a + e) * entry + S
        f = sum(x[1] for x in seq) + dk * dv * (2 * a + 3)
        b += S + a * entry + pin * dk + 4 * dv                   # readout
        f += 2 * dk * dv + 2 * a * (dk + dv)
        b += (2 * S + e * entry) / 2                             # half the slots are flushed
        f += dk * dv * (2 * e + 1) / 2
    else:
        seq = [step(L) for L in range(M)]
        b = sum(x[0] for x in seq) + (M - 1) * entry + S
        f = sum(x[1] for x in seq) + dk * dv * (2 * (M - 1) + 3)
        if c["kind"] == "engine":                                # one token of the cycle's M
            b, f = c["layers"] * b / M, c["layers"] * f / M
    heads = c["active"] * c["H"]
    return {"bytes": heads * b, "flops": heads * f}


def tolerance(case):
    # fp32 sums over at most 128 rows and 63 log entries, carried through one cycle by the
    # delta rule.  Another order of these sums (cross-lane sums by shuffles instead of DPP,
    # the merge on the vector ALUs instead of MFMA) moved the results by rel 1.1e-7 and at
    # most 1.3e-6 of an element; against 64 bits they are within 3.5e-7.
    # A bf16 state is rounded once per merge: a difference of 1e-7 before the rounding
    # flips it for about 1e-7 / 2^-8 of the elements, each by one bf16 step (up to 2^-7 of
    # the element).
    if case["state"] == "bf16":
        return {"rel": 1e-4, "max": 2e-2}
    return {"rel": 1e-6, "max": 2e-5}


# ------------------------------------------------------------------ in 64 bits
class _Exact:
    """The recurrence in float64 (the represented state Z) beside the stored form: the base
    at the last merge, the log entries, the cumulative log-decay and the live length."""

    def __init__(self, c, S0, live=None, log=None, u=None):
        self.c, self.u = c, None if u is None else u.double()
        B, H, dk, dv, C, dl = c["B"], c["H"], c["dk"], c["dv"], c["M"] - 1, _dl(c)
        f8 = dict(dtype=torch.float64, device="cuda")
        self.C, self.dl = C, dl
        self.base = S0.double()
        self.len = torch.zeros(B, dtype=torch.long, device="cuda") if live is None else live.clone()
        self.K, self.U = torch.zeros((B, C, H, dk), **f8), torch.zeros((B, C, H, dv), **f8)
        self.Lam = torch.zeros((B, C, H, max(dl, 1)), **f8)
        self.ell = torch.zeros((B, H, max(dl, 1)), **f8)
        self.Z = self.base.clone()
        if log is not None:
            k, u_, lam = log
            self.K, self.U = k.double().transpose(1, 2).contiguous(), u_.double().transpose(1, 2).contiguous()
            if lam is not None:
                self.Lam = (lam.double()[..., None] if dl == 1 else lam.double().transpose(1, 2)).contiguous()
            has = self.len > 0
            idx = (self.len - 1).clamp(min=0)
            self.ell = self.Lam[torch.arange(B, device="cuda"), idx] * has[:, None, None]
            self.Z = torch.exp(self.ell)[..., None] * self.base
            for i in range(C):
                on = (i < self.len).double()[:, None, None]
                kd = torch.exp((self.ell - self.Lam[:, i]) * on) * self.K[:, i] * on
                self.Z += kd[..., None] * self.U[:, i][..., None, :]

    def token(self, rows, q, k, v, lam, beta, force=False, eager=False):
        q, k, v = q.double(), k.double(), v.double()
        Z = self.Z if rows is None else self.Z[rows]
        l = (torch.zeros((*k.shape[:2], 1), dtype=torch.float64, device="cuda") if lam is None
             else lam.double()[..., None] if self.dl == 1 else lam.double())
        o = None
        if self.c["op"] == "rwkv6":
            o = (q[..., None] * Z).sum(-2) + (q * self.u * k).sum(-1, keepdim=True) * v
        Z = torch.exp(l)[..., None] * Z
        b = v
        if beta is not None:
            b = beta.double()[..., None] * (v - (k[..., None] * Z).sum(-2))
        Z += k[..., None] * b[..., None, :]
        if o is None:
            o = (q[..., None] * Z).sum(-2)
        if rows is None:
            self.Z = Z
            rows = torch.arange(self.c["B"], device="cuda")
        else:
            self.Z[rows] = Z
        if eager:
            return o
        self.ell[rows] += l
        L = self.len[rows]
        full = torch.ones_like(L, dtype=torch.bool) if force else L >= self.C
        app = rows[~full]
        if app.numel():
            La = self.len[app]
            self.K[app, La], self.U[app, La], self.Lam[app, La] = k[~full], b[~full], self.ell[app]
            self.len[app] += 1
        self._materialise(rows[full])
        return o

    def _materialise(self, rows):
        if rows.numel():
            self.base[rows] = self.Z[rows]
            self.ell[rows] = 0
            self.len[rows] = 0

    def flush(self, rows):
        self._materialise(rows)

    def buffers(self):
        H = self.c["H"]
        out = {"S": self.base, "k_log": self.K.transpose(1, 2), "u_log": self.U.transpose(1, 2),
               "len": self.len.to(torch.int32)[:, None].expand(-1, H)}
        if self.dl:
            out["lam_log"] = self.Lam[..., 0] if self.dl == 1 else self.Lam.transpose(1, 2)
        return {k: v.contiguous() for k, v in out.items()}


def exact(case, seed):
    c = case
    at = lambda a, t: None if a is None else a[t]  # noqa: E731
    if c["kind"] == "engine":
        d = _Draw(c, seed)
        u = d.bonus()
        H, L = c["H"], c["layers"]
        S0 = [torch.zeros((c["B"], H, c["dk"], c["dv"]), device="cuda") for _ in range(L)]
        sims = [_Exact(c, s, u=u) for s in S0]
        o = [torch.zeros((c["B"], H, c["dv"]), dtype=torch.float64, device="cuda") for _ in range(L)]
        active = 0
        for more in _engine_steps(c) + [0]:                  # the last: the pass itself
            new = [d.base(more, H) for _ in range(L)] if more else [None] * L
            rows = torch.arange(active + more, device="cuda")
            for i, sim in enumerate(sims):
                if more:
                    sim.base[active:active + more] = new[i].double()
                    sim.Z[active:active + more] = new[i].double()
                x = d.tokens(1, active + more)
                o[i][: active + more] = sim.token(rows, x["q"][0], x["k"][0], x["v"][0],
                                                  at(x["lam"], 0), at(x["beta"], 0))
            active += more
        return [{"o": oi, **s.buffers()} for oi, s in zip(o, sims)]
    x = _inputs(c, seed)
    tk, T = x["tok"], _steps(c)
    rows = None if x["slots"] is None else x["slots"].long()
    sim = _Exact(c, x["S0"], x["live"], x.get("log"), x["u"])
    a = c["M"] // 2
    outs, r = [], None
    for t in range(T):
        if c["kind"] == "lifecycle" and t == a:
            r = (x["q"].double()[..., None] * (sim.Z if rows is None else sim.Z[rows])).sum(-2)
        outs.append(sim.token(rows, tk["q"][t], tk["k"][t], tk["v"][t], at(tk["lam"], t),
                              at(tk["beta"], t), force=c["kind"] == "lifecycle" and t == a,
                              eager=c["kind"] == "eager"))
    if c["kind"] == "eager":
        return {"o": torch.stack(outs), "S": sim.Z}
    if c["kind"] == "lifecycle":
        sim.flush(torch.arange(0, c["B"], 2, device="cuda"))
        return {"o": torch.stack(outs), "r": r, **sim.buffers()}
    return {"o": torch.stack(outs), **sim.buffers()}
