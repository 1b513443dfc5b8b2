"""The work this framework is run for, as cases that can be timed and compared.

A case is one call, or one step, of one context-parallel rank: the rank's query
block against P key/value partitions of a video-DiT sequence, some computed
fresh and the others reused from the state cache, all composed, with the
contribution weights of the partitions for the next step's selection.  Shapes
are those of the workloads the tests and the benchmark run (video-DiT,
HunyuanVideo-like head dim 64, long context, the 16,384-token reuse case, the
float32 plumbing case), and the 33K-token, 12-head shape with a
classifier-free-guidance batch of 2.

Inputs are unit-variance noise plus a smooth positional component shared by Q,
K, V and all heads, so that near partitions weigh more; cached states are what
an earlier step leaves in the cache: outputs that average many values, and
log-sum-exps near the logarithm of the key count.
"""
import math

import torch

from paper_2607_15650_amd import api
from paper_2607_15650_amd.ase import ErrorModelSelectiveAttention
from paper_2607_15650_amd.groups import GroupedSelectiveAttention, base_groups
from paper_2607_15650_amd.step import SelectiveAttention

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
_BYTES = {"f32": 4, "bf16": 2}


def _step(name, dtype, B, H, D, S, P, q, fresh, state="same"):
    return {"name": name, "kind": "step", "dtype": dtype, "state": state, "B": B, "H": H, "D": D, "S": S, "P": P,
            "q": q, "fresh": fresh}


def listed():
    return [
        # the smallest whole step, float32 inputs and states, everything
        # computed: launch latency, and a chip that few query tiles fill
        _step("step_f32_plumbing", "f32", 1, 2, 64, 4096, 4, 0, 4),
        # float32 inputs at an ordinary size: 12 heads at head dim 128, a
        # ragged sequence, the two nearest of six partitions fresh
        _step("step_f32_d128", "f32", 1, 12, 128, 12285, 6, 2, 2),
        # a short bf16 step at head dim 64: three of eight partitions fresh
        _step("step_reuse_d64", "bf16", 1, 12, 64, 16384, 8, 3, 3),
        # conditional and unconditional branch in one batch, 12 heads, a 480p
        # latent of 21 x 30 x 52 tokens
        _step("step_cfg_33k", "bf16", 2, 12, 128, 32760, 8, 3, 3),
        # the flagship step: 81 frames at 720p, 40 heads
        _step("step_videodit", "bf16", 1, 40, 128, 75600, 8, 3, 3),
        # a step that reuses nearly everything: one of sixteen partitions
        # fresh, so composition and weights count
        _step("step_longctx_reuse", "bf16", 1, 24, 128, 131072, 16, 7, 1),
        # fresh states alone at head dim 64, 129 frames at 720p, 48 heads
        {"name": "attn_hunyuan_d64", "kind": "attn", "dtype": "bf16", "state": "same", "B": 1, "H": 48, "D": 64,
         "S": 118800, "P": 8, "q": 3, "fresh": 3},
        # group-granular reuse: two groups and the local partition fresh, the
        # others' composed states from the cache
        {"name": "group_step", "kind": "group", "dtype": "bf16", "B": 1, "H": 12, "D": 128, "S": 32760, "P": 8,
         "q": 3, "g": 2, "fresh": 2},
        # the error-model planner between two anchors: local state, drift,
        # every group reused
        {"name": "planner_reuse_step", "kind": "planner", "dtype": "bf16", "B": 1, "H": 24, "D": 128, "S": 32760,
         "P": 8, "q": 3, "g": 2},
        # composition alone, states kept at full precision, a list of slots
        {"name": "merge_f32_states", "kind": "merge", "state": "f32", "out": "bf16", "B": 1, "H": 40, "D": 128,
         "L": 9450, "P": 8, "n": 5},
        # per-row contribution weights of sixteen partitions
        {"name": "weights_rows", "kind": "weights", "B": 1, "H": 24, "L": 8192, "P": 16, "rows": True},
        # drift norms of the planner: several snapshots against the current
        # local state
        {"name": "norms_drift", "kind": "norms", "state": "bf16", "B": 1, "H": 40, "D": 128, "L": 9450, "P": 6,
         "n": 4, "ref": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; no dearer than the largest listed one."""
    while True:
        kind = rng.choice(["step", "step", "step", "step", "attn", "attn", "group", "planner", "merge", "weights",
                           "norms"])
        c = {"kind": kind, "B": rng.choice([1, 1, 2]), "H": _log(rng, 2, 48), "D": rng.choice([64, 128])}
        if kind in ("step", "attn"):
            c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
            c["state"] = rng.choice(["same", "same", "same", "f32"]) if c["dtype"] == "bf16" else "same"
            c["S"], c["P"] = _log(rng, 2048, 131072), rng.randint(2, 20)
            c["q"] = rng.randrange(c["P"] - 1)
            c["fresh"] = rng.randint(1, c["P"])
        elif kind in ("group", "planner"):
            c["dtype"], c["S"], c["P"] = "bf16", _log(rng, 4096, 76000), rng.randint(4, 12)
            c["q"], c["g"] = rng.randrange(c["P"] - 1), rng.randint(2, 3)
            if kind == "group":
                c["fresh"] = rng.randint(1, 3)
        else:
            c["L"], c["P"] = _log(rng, 256, 16384), rng.randint(2, 20)
            if kind == "merge":
                c["state"], c["out"] = rng.choice(["bf16", "bf16", "f32"]), rng.choice(["bf16", "f32"])
                c["n"] = rng.randint(2, c["P"])
            elif kind == "weights":
                del c["D"]
                c["rows"] = rng.choice([True, False])
            else:
                c["state"], c["n"], c["ref"] = rng.choice(["bf16", "f32"]), rng.randint(1, min(6, c["P"])), \
                    rng.choice([True, False])
        w = work(c)
        if "S" in c:
            if min(b - a for a, b in zip(_offsets(c), _offsets(c)[1:])) < 1:
                continue
            # the whole sequence and the cache are held three times over
            if c["B"] * c["S"] * c["H"] * c["D"] > 4.2e8:
                continue
        if w["flops"] <= (4e10 if c.get("dtype") == "f32" else 4e12) and 1e6 <= w["bytes"] <= 1.2e9:
            return c


# ------------------------------------------------------------------ shapes
def _offsets(c):
    """Contiguous chunks of ceil(S/P) tokens, the last the remainder."""
    n = -(-c["S"] // c["P"])
    return [min(j * n, c["S"]) for j in range(c["P"])] + [c["S"]]


def _select(c):
    """The `fresh` partitions nearest to the query block."""
    near = sorted(range(c["P"]), key=lambda j: (abs(j - c["q"]), j))[:c["fresh"]]
    return [1 if j in near else 0 for j in range(c["P"])]


def _compute(c):
    """The `fresh` groups nearest to the query block, and all groups."""
    groups = base_groups(c["P"], c["q"], c["g"])
    near = sorted(groups, key=lambda r: (min(abs(r[0] - c["q"]), abs(r[1] - 1 - c["q"])), r[0]))
    return sorted(near[:c["fresh"]]), groups


def _q_len(c):
    o = _offsets(c)
    return o[c["q"] + 1] - o[c["q"]]


def _state_dt(c):
    return c["state"] if c["state"] != "same" else c["dtype"]


# ------------------------------------------------------------------ inputs
def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + k)
    return g


def _noise(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _qkv(c, seed):
    """Q, K, V of the whole sequence in float32."""
    B, S, H, D = c["B"], c["S"], c["H"], c["D"]
    g = _gen(seed, 0)
    freq = torch.rand(D, generator=g, device="cuda") * (2 * 2 * math.pi / S)
    phase = torch.rand(D, generator=g, device="cuda") * (2 * math.pi)
    n = torch.arange(S, device="cuda", dtype=torch.float32)
    pos = (0.5 * torch.sin(n[:, None] * freq + phase))[None, :, None, :]
    return [_noise((B, S, H, D), g).add_(pos) for _ in range(3)]


def _fill_states(out, lse, keys, seed):
    """Cached states of partitions of about `keys` keys."""
    g = _gen(seed, 1)
    for j in range(out.shape[0]):
        out[j].copy_(_noise(out.shape[1:], g).mul_(0.03))
        lse[j].copy_(_noise(lse.shape[1:], g).mul_(0.2).add_(math.log(max(keys, 1)) + 0.6))


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    st = {"case": c, "t": 1}
    if kind in ("step", "attn", "group"):
        st["q"], st["k"], st["v"] = (x.to(_DT[c["dtype"]]) for x in _qkv(c, seed))
    scale = 1.0 / math.sqrt(c["D"]) if "D" in c else 0.0
    st["scale"] = scale
    if kind == "step":
        sa = SelectiveAttention(c["B"], c["H"], c["D"], _offsets(c), scale, _DT[c["dtype"]], "cuda",
                                _DT[_state_dt(c)])
        cache = sa.cache(c["q"])
        _fill_states(cache.out, cache.lse, _q_len(c), seed)
        st["engine"], st["cache"], st["select"] = sa, cache, _select(c)
    elif kind == "attn":
        B, H, D, P, L = c["B"], c["H"], c["D"], c["P"], _q_len(c)
        a = _offsets(c)[c["q"]]
        st["q"] = st["q"][:, a:a + L].contiguous()
        st["offsets"], st["select"] = _offsets(c), _select(c)
        st["out"] = torch.zeros((P, B, L, H, D), dtype=_DT[_state_dt(c)], device="cuda")
        st["lse"] = torch.zeros((P, B, H, L), dtype=torch.float32, device="cuda")
        n = api.attn_workspace_bytes(_DT[c["dtype"]], B, H, D, L, st["offsets"], st["select"])
        st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    elif kind == "group":
        gs = GroupedSelectiveAttention(c["B"], c["H"], c["D"], _offsets(c), c["q"], c["g"], scale, _DT[c["dtype"]])
        _fill_states(gs.out, gs.lse, c["g"] * _q_len(c), seed)
        st["engine"], (st["compute"], st["groups"]) = gs, _compute(c)
    elif kind == "planner":
        # one anchor step, then the tensors of the next denoising step; with
        # a reuse ratio of 1 every group is reused until the drift limit
        em = ErrorModelSelectiveAttention(c["B"], c["H"], c["D"], _offsets(c), c["q"], c["g"], scale, 1.0, 0.5,
                                          _DT[c["dtype"]])
        now, nxt = _evolved(c, seed)
        em.step(0, *now)
        st["q"], st["k"], st["v"] = nxt
        st["engine"] = em
    else:
        B, H, P, L = c["B"], c["H"], c["P"], c["L"]
        if kind in ("merge", "norms"):
            st["out_states"] = torch.empty((P, B, L, H, c["D"]), dtype=_DT[c["state"]], device="cuda")
            lse = torch.empty((P, B, H, L), dtype=torch.float32, device="cuda")
            _fill_states(st["out_states"], lse, L, seed)
            st["lse_states"] = lse
            st["slots"] = _slots(c)
        if kind == "merge":
            st["out"] = torch.empty((B, L, H, c["D"]), dtype=_DT[c["out"]], device="cuda")
            st["lse"] = torch.empty((B, H, L), dtype=torch.float32, device="cuda")
        elif kind == "norms":
            g = _gen(seed, 2)
            st["ref"] = None
            if c["ref"]:
                # the current local state has moved a little from every snapshot
                st["ref"] = (_noise((B, L, H, c["D"]), g) * 0.01).to(_DT[c["state"]])
            n = api.norms_workspace_bytes(B, H, c["D"], L, c["n"])
            st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
            st["norms"] = torch.empty(c["n"], dtype=torch.float32, device="cuda")
        else:
            g = _gen(seed, 3)
            st["lse_states"] = _noise((P, B, H, L), g).mul_(0.3).add_(math.log(L))
            st["lse"] = torch.logsumexp(st["lse_states"].double(), dim=0).float()
            n = api.contrib_workspace_bytes(B, H, L, P)
            st["ws"] = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
            st["w"] = torch.empty(P, dtype=torch.float32, device="cuda")
            st["rows"] = torch.empty((B, H, L, P), dtype=torch.float32, device="cuda") if c["rows"] else None
    return st


def _evolved(c, seed):
    """Tensors of an anchor step and of the denoising step after it (an early
    one: its drift stands well above the rounding of bf16 states)."""
    dt = _DT[c["dtype"]]
    x = _qkv(c, seed)
    g = _gen(seed, 4)
    now = [t.to(dt) for t in x]
    nxt = [t.add_(_noise(t.shape, g), alpha=0.1).to(dt) for t in x]
    return now, nxt


def _slots(c):
    """`n` slots of the P, in an order of the planner's kind: every other
    partition first, then the rest."""
    order = list(range(0, c["P"], 2)) + list(range(1, c["P"], 2))
    return order[:c["n"]]


# --------------------------------------------------------------------- run
def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "step":
        out, lse, w = st["engine"].step(st["t"], c["q"], st["q"], st["k"], st["v"], st["select"])
        return {"out": out, "lse": lse, "w": w, "states": st["cache"].out, "state_lse": st["cache"].lse}
    if kind == "attn":
        api.attn_partition_states(st["q"], st["k"], st["v"], st["offsets"], st["select"], st["scale"], st["out"],
                                  st["lse"], st["ws"])
        return {"states": st["out"], "state_lse": st["lse"]}
    if kind == "group":
        gs = st["engine"]
        out, lse, w = gs.step(st["t"], st["q"], st["k"], st["v"], st["compute"])
        live = [grp[0] for grp in gs.groups] + [c["q"]]
        return {"out": out, "lse": lse, "w": w, "states": [gs.out[j] for j in live],
                "state_lse": [gs.lse[j] for j in live]}
    if kind == "planner":
        em = st["engine"]
        out, lse, info = em.step(st["t"], st["q"], st["k"], st["v"])
        return {"out": out, "lse": lse, "drift": float(info["drift"]), "ase": [float(x) for x in info["ase"].values()],
                "local": em.cache[c["q"]]}
    if kind == "merge":
        api.merge_states(st["out_states"], st["lse_states"], st["out"], st["lse"], slots=st["slots"])
        return {"out": st["out"], "lse": st["lse"]}
    if kind == "weights":
        api.contrib(st["lse_states"], st["lse"], st["w"], st["ws"], st["rows"])
        return {"w": st["w"], "rows": st["rows"]} if c["rows"] else {"w": st["w"]}
    api.state_norms(st["out_states"], st["norms"], st["ws"], slots=st["slots"], ref=st["ref"])
    return {"norms": st["norms"]}


# -------------------------------------------------------------------- work
def work(case):
    """Each input read once, each output written once; flops of the two
    products of the fresh partitions."""
    c = case
    kind, B, H = c["kind"], c["B"], c["H"]
    if kind in ("merge", "weights", "norms"):
        rows = B * c["L"] * H
        if kind == "weights":
            return {"bytes": rows * 4 * (c["P"] + 1 + (c["P"] if c["rows"] else 0)) + 4 * c["P"],
                    "flops": 2.0 * rows * c["P"]}
        s = _BYTES[c["state"]]
        if kind == "merge":
            return {"bytes": rows * (c["n"] * (c["D"] * s + 4) + c["D"] * _BYTES[c["out"]] + 4),
                    "flops": 2.0 * rows * c["n"] * c["D"]}
        return {"bytes": rows * c["D"] * s * (c["n"] + (1 if c["ref"] else 0)) + 4 * c["n"],
                "flops": 3.0 * rows * c["n"] * c["D"]}
    o, L, D, e = _offsets(c), _q_len(c), c["D"], _BYTES[c["dtype"]]
    rows = B * L * H
    if kind in ("step", "attn"):
        sel = [j for j, s in enumerate(_select(c)) if s]
        n_fresh = len(sel)
        keys = sum(o[j + 1] - o[j] for j in sel)
        state = rows * (D * _BYTES[_state_dt(c)] + 4)
        reused = c["P"] - n_fresh
    elif kind == "group":
        compute, groups = _compute(c)
        keys = L + sum(o[b] - o[a] for a, b in compute)
        state = rows * (D * e + 4)
        n_fresh, reused = 1 + len(compute), len(groups) - len(compute)
    else:
        keys, n_fresh = L, 1
        state = rows * (D * e + 4)
        reused = len(base_groups(c["P"], c["q"], c["g"])) + 1    # the groups, and the anchor's local state
    flops = 4.0 * rows * D * keys
    nbytes = rows * D * e + 2 * B * keys * H * D * e + n_fresh * state
    if kind != "attn":
        nbytes += reused * state + rows * (D * e + 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16 states are rounded once in the probabilities and once in the
    store; float32 paths differ by the order of their sums."""
    c = case
    f32 = c["kind"] in ("weights", "norms") or c.get("dtype") == "f32" or \
        (c["kind"] == "merge" and c["state"] == "f32" and c["out"] == "f32")
    if f32:
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 1e-1}


# ------------------------------------------------------------------- exact
def _attn64(q, k, v, a, b, scale):
    """State of keys [a, b) in 64 bits: OUT [B, L, H, D], LSE [B, H, L]."""
    B, L, H, D = q.shape
    out = torch.empty((B, L, H, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, L), dtype=torch.float64, device="cuda")
    for i in range(B):
        for h in range(H):
            kd, vd = k[i, a:b, h].double().contiguous(), v[i, a:b, h].double().contiguous()
            for r in range(0, L, 8192):
                s = torch.mm(q[i, r:r + 8192, h].double().contiguous(), kd.t()).mul_(scale)
                m = s.amax(dim=1, keepdim=True)
                s.sub_(m).exp_()
                tot = s.sum(dim=1, keepdim=True)
                out[i, r:r + 8192, h] = torch.mm(s, vd).div_(tot)
                lse[i, h, r:r + 8192] = (m + tot.log()).squeeze(1)
    return out, lse


def _merge64(states, lses):
    """Composition of lists of states: OUT, LSE."""
    stack = torch.stack([x.double() for x in lses])
    lse = torch.logsumexp(stack, dim=0)
    out = None
    for x, l in zip(states, stack):
        y = x.double() * (l - lse).exp().transpose(1, 2).unsqueeze(-1)
        out = y if out is None else out.add_(y)
    return out, lse


def exact(case, seed):
    st = prepare_inputs_only(case, seed)
    c = st["case"]
    kind = c["kind"]
    if kind == "merge":
        out, lse = _merge64([st["out_states"][j] for j in st["slots"]], [st["lse_states"][j] for j in st["slots"]])
        return {"out": out, "lse": lse}
    if kind == "weights":
        rows = (st["lse_states"].double() - st["lse"].double()).exp().permute(1, 2, 3, 0).contiguous()
        w = rows.mean(dim=(0, 1, 2))
        return {"w": w, "rows": rows} if c["rows"] else {"w": w}
    if kind == "norms":
        got = []
        for j in st["slots"]:
            x = st["out_states"][j].double()
            got.append((x if st["ref"] is None else x.sub_(st["ref"].double())).norm())
        return {"norms": torch.stack(got)}
    o, q0, L = _offsets(c), c["q"], _q_len(c)
    qb = slice(o[q0], o[q0] + L)
    scale = 1.0 / math.sqrt(c["D"])
    if kind == "planner":
        now, nxt = _evolved(c, seed)
        groups = base_groups(c["P"], q0, c["g"])
        parts = [_attn64(now[0][:, qb], now[1], now[2], o[j], o[j + 1], scale) for j in range(c["P"])]
        _, lse0 = _merge64([p[0] for p in parts], [p[1] for p in parts])
        w = [float((p[1] - lse0).exp().mean()) for p in parts]
        nrm = [float(p[0].norm()) for p in parts]
        loc = _attn64(nxt[0][:, qb], nxt[1], nxt[2], o[q0], o[q0 + 1], scale)
        d = float((loc[0] - parts[q0][0]).norm())
        ase = [sum(w[j] * nrm[j] / nrm[q0] for j in range(*g)) * d for g in groups]
        live = [_merge64([parts[j][0] for j in range(*g)], [parts[j][1] for j in range(*g)]) for g in groups] + [loc]
        out, lse = _merge64([p[0] for p in live], [p[1] for p in live])
        return {"out": out, "lse": lse, "drift": d / nrm[q0], "ase": ase, "local": loc[0]}
    q = st["q"][:, qb]
    if kind == "group":
        compute, groups = _compute(c)
        live = []
        for g in groups:
            if g in compute:
                live.append(_attn64(q, st["k"], st["v"], o[g[0]], o[g[1]], scale))
            else:
                live.append((st["states"][g[0]].double(), st["state_lse"][g[0]].double()))
        live.append(_attn64(q, st["k"], st["v"], o[q0], o[q0 + 1], scale))
        out, lse = _merge64([p[0] for p in live], [p[1] for p in live])
        w = torch.stack([(p[1] - lse).exp().mean() for p in live])
        return {"out": out, "lse": lse, "w": w, "states": [p[0] for p in live], "state_lse": [p[1] for p in live]}
    states, lses = st["states"].double(), st["state_lse"].double()
    for j, s in enumerate(_select(c)):
        if s:
            states[j], lses[j] = _attn64(q, st["k"], st["v"], o[j], o[j + 1], scale)
    if kind == "attn":
        return {"states": states, "state_lse": lses}
    out, lse = _merge64(states, lses)
    w = (lses - lse).exp().mean(dim=(1, 2, 3))
    return {"out": out, "lse": lse, "w": w, "states": states, "state_lse": lses}


def prepare_inputs_only(case, seed):
    """The inputs and cached states of `prepare`, without an engine."""
    c = dict(case)
    kind = c["kind"]
    if kind in ("merge", "weights", "norms"):
        return prepare(c, seed)
    st = {"case": c}
    if kind == "planner":
        return st
    st["q"], st["k"], st["v"] = (x.to(_DT[c["dtype"]]) for x in _qkv(c, seed))
    B, H, D, P, L = c["B"], c["H"], c["D"], c["P"], _q_len(c)
    st["states"] = torch.zeros((P, B, L, H, D), dtype=_DT[c["dtype"] if kind == "group" else _state_dt(c)],
                               device="cuda")
    st["state_lse"] = torch.zeros((P, B, H, L), dtype=torch.float32, device="cuda")
    if kind != "attn":
        _fill_states(st["states"], st["state_lse"], L * (c["g"] if kind == "group" else 1), seed)
    return st
