"""Performance cases of the expert layer: what a training program has this
framework do, through its public entry points (paper_2606_11867_amd.api and
PolicyUpdate), over the shapes of the repository's own workloads.

Routing follows the recipe of the synthetic workloads: expert popularity is a
Zipf law times a Dirichlet factor per micro-step, the recorded ids are the
top-K of noisy router logits, experts are placed on ranks by capacity-limited
LPT over 16 micro-steps, and the measured rank's heaviest experts of a
micro-step get one local replica each. Popularity and placement belong to the
case (the plan a program keeps), and so do its per-expert loads; the order of
the tokens, their values, weights and gradients come from the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2606_11867_amd import _lib, api
from paper_2606_11867_amd.policy_update import MicroStep, PolicyUpdate

MICRO_STEPS = 16
BF16, F32 = torch.bfloat16, torch.float32


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the whole layer, forward and backward, on a tiny fp32 model: the
        # smallest call, and the fp32 data path
        dict(name="layer-fp32-tiny", kind="layer", dtype="f32", T=256, d=128, F=256, E=8, K=2, P=2, reps=1,
             backward=True),
        # forward only (the recompute stage) of a short micro-step: a few
        # rows per expert, so reading the weights is the work
        dict(name="layer-fwd-short", kind="layer", dtype="bf16", T=512, d=2048, F=768, E=128, K=8, P=8, reps=4,
             backward=False),
        # the whole layer, forward and backward, at odd sizes: token count
        # and slot lengths no multiple of anything, widths that are odd
        # multiples of 128
        dict(name="layer-ragged", kind="layer", dtype="bf16", T=3001, d=1152, F=896, E=24, K=3, P=2, reps=2,
             backward=True),
        # dispatch (steps 1-3) of a Qwen3-30B-A3B EP=8 share's micro-step
        dict(name="dispatch-qwen3", kind="dispatch", dtype="bf16", T=16384, d=2048, E=128, K=8, P=8, reps=4,
             n_src=1),
        # the same micro-step as the planner places it: pairs split per
        # source rank by the water-filled counts
        dict(name="dispatch-8-sources", kind="dispatch", dtype="bf16", T=16384, d=2048, E=128, K=8, P=8, reps=4,
             n_src=8),
        # combine and the two backward gathers of a DeepSeek-V3 EP=32 share:
        # wide rows, most tokens without a local pair
        dict(name="gathers-deepseek", kind="gathers", dtype="bf16", T=32768, d=7168, E=256, K=8, P=32, reps=2),
        # expert FFN forward, activations kept for the backward, mean
        # micro-step of the Qwen3 share
        dict(name="ffn-fwd-qwen3", kind="ffn_fwd", rows=16278, d=2048, F=768, E=128, K=8, P=8, reps=4, save=True),
        # expert FFN forward of the recompute stage on a Mixtral-8x7B share
        dict(name="ffn-fwd-mixtral", kind="ffn_fwd", rows=8192, d=4096, F=14336, E=8, K=2, P=1, reps=2, save=False),
        # input gradients on a DeepSeek-V3 EP=32 share
        dict(name="ffn-dgrad-deepseek", kind="ffn_dgrad", rows=11066, d=7168, F=2048, E=256, K=8, P=32, reps=2),
        # weight gradients of four accumulated micro-steps of the Qwen3
        # share, as one update step of a program that accumulates
        dict(name="ffn-wgrad-qwen3", kind="ffn_wgrad", rows=65536, steps=4, d=2048, F=768, E=128, K=8, P=8, reps=4),
        # policy update on the Qwen3 share: eight micro-steps forward and
        # backward, pipelined, one weight-gradient group
        dict(name="policy-update-qwen3", kind="update", T=16384, steps=8, d=2048, F=768, E=128, K=8, P=8, reps=4),
        # expert transfer of the Qwen3 share: pack 20 experts with their
        # gradients, unpack them, two records accumulated into main experts
        dict(name="transfer-qwen3", kind="transfer", dtype="bf16", records=20, d=2048, F=768),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of step, spread over the logarithm of [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(max(round(v / step), -(-lo // step)), hi // step)) * step


def draw(rng):
    kind = rng.choice(["layer", "layer", "dispatch", "dispatch", "gathers", "ffn_fwd", "ffn_fwd", "ffn_dgrad",
                       "ffn_wgrad", "update", "transfer"])
    # experts in the model, top-K, EP ranks, redundant slots per rank
    E, K, P, reps = rng.choice([(8, 2, 1, 2), (24, 3, 2, 2), (64, 6, 4, 3), (128, 8, 8, 4), (256, 8, 32, 2)])
    c = dict(kind=kind, E=E, K=K, P=P, reps=reps)
    if kind == "layer":
        c["backward"] = rng.random() < 0.5
        if rng.random() < 0.4:
            c.update(dtype="f32", T=_log(rng, 64, 2048), d=_log(rng, 24, 512, 4), F=_log(rng, 40, 768), E=8, K=2,
                     P=2, reps=1)
        else:
            c.update(dtype="bf16", T=_log(rng, 100, 8192), d=_log(rng, 256, 2048, 128), F=_log(rng, 128, 1536, 128))
    elif kind == "dispatch":
        n_src = P if 1 < P <= 8 and rng.random() < 0.5 else 1
        c.update(dtype=rng.choice(["bf16", "bf16", "f32"]), T=_log(rng, 200, 32768), d=_log(rng, 128, 4096, 8),
                 n_src=n_src)
    elif kind == "gathers":
        c.update(dtype=rng.choice(["bf16", "bf16", "f32"]), T=_log(rng, 200, 32768), d=_log(rng, 128, 7168, 8))
    elif kind in ("ffn_fwd", "ffn_dgrad"):
        c.update(rows=_log(rng, 200, 40000), d=_log(rng, 512, 7168, 128), F=_log(rng, 256, 4096, 128))
        if kind == "ffn_fwd":
            c["save"] = rng.random() < 0.5
    elif kind == "ffn_wgrad":
        c.update(rows=_log(rng, 1000, 65536), steps=rng.choice([1, 2, 4, 8]), d=_log(rng, 512, 4096, 128),
                 F=_log(rng, 256, 2048, 128))
    elif kind == "update":
        c.update(T=_log(rng, 1000, 16384), steps=rng.choice([3, 5, 8]), d=_log(rng, 512, 2048, 128),
                 F=_log(rng, 256, 1024, 128))
    else:
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), records=rng.randint(4, 24),
                    d=_log(rng, 256, 4096, 8), F=_log(rng, 128, 768, 8))
    size = "rows" if "rows" in c else "T"
    while _too_large(c):
        c[size] = c[size] * 2 // 3
    return c


def _too_large(c):
    w, f32 = work(c), c.get("dtype") == "f32"
    return w["bytes"] > 1.7e9 or w["flops"] > (3e9 if f32 and c["kind"] == "layer" else 2.8e12)


# ---------------------------------------------------------------------------
# Plans: popularity, placement and slot tables of a case
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _placement(E, K, P, reps):
    """bias [MICRO_STEPS, E] of the router logits, and per micro-step the
    measured rank's slots [(expert, replica)] and expected pairs per slot and
    token; `order`: micro-steps by how close their load is to K / P."""
    rng = np.random.default_rng(1000 + E * 64 + K)
    pop = (rng.permutation(E) + 1.0) ** -1.1
    g = rng.dirichlet(np.full(E, 0.3), MICRO_STEPS)
    bias = np.log(pop) + np.log(np.maximum(E * g, 1e-30))
    n = 1024  # sampled tokens
    load = np.zeros((MICRO_STEPS, E))
    for m in range(MICRO_STEPS):
        top = np.argpartition(-(rng.standard_normal((n, E)) + bias[m]), K - 1, axis=1)[:, :K]
        load[m] = np.bincount(top.reshape(-1), minlength=E) / n
    total = load.sum(0)
    rank_load, used, rank_of = np.zeros(P), np.zeros(P, int), np.zeros(E, int)
    for e in np.argsort(-total, kind="stable"):
        r = min((r for r in range(P) if used[r] < E // P), key=lambda r: (rank_load[r], r))
        rank_of[e], rank_load[r], used[r] = r, rank_load[r] + total[e], used[r] + 1
    hosted = np.nonzero(rank_of == int(np.argmin(np.abs(rank_load - rank_load.mean()))))[0]
    slots, share = [], []
    for m in range(MICRO_STEPS):
        heavy = [int(e) for e in hosted[np.argsort(-load[m][hosted], kind="stable")[:reps]]]
        slots.append([(int(e), 0) for e in hosted] + [(e, 1) for e in heavy])
        share.append([load[m][e] / (2 if e in heavy else 1) for e, _ in slots[m]])
    order = [int(m) for m in np.argsort(np.abs(load[:, hosted].sum(1) - K / P), kind="stable")]
    return bias, hosted, slots, share, order


def _key(c):
    return c["E"], c["K"], c["P"], c["reps"]


def _steps(c):
    """The micro-steps a case runs: the one nearest the mean load, or the
    first `steps` in sequence."""
    return list(range(c["steps"])) if "steps" in c else _placement(*_key(c))[4][:1]


def _slot_rows(c):
    """Rows of every slot in each micro-step of a case that starts at the
    FFN: the expected shares scaled to c["rows"] in all."""
    share = _placement(*_key(c))[3]
    parts = [(m, j, s) for m in _steps(c) for j, s in enumerate(share[m])]
    w = np.array([s for _, _, s in parts])
    cum = np.floor(np.cumsum(w) / w.sum() * c["rows"] + 0.5).astype(np.int64)
    n = np.diff(np.concatenate([[0], cum]))
    rows = {m: [0] * len(share[m]) for m in _steps(c)}
    for (m, j, _), k in zip(parts, n):
        rows[m][j] = int(k)
    return [rows[m] for m in _steps(c)]


def _pairs(c):
    """Expected local pairs of each micro-step of a case that starts at the
    tokens."""
    share = _placement(*_key(c))[3]
    return [c["T"] * float(sum(share[m])) for m in _steps(c)]


def _i32(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _device_plan(E, slots):
    local = sorted({e for e, _ in slots})
    widx = [local.index(e) for e, _ in slots]
    nrep = np.ones(E, np.int32)
    for e, r in slots:
        nrep[e] = max(nrep[e], r + 1)
    return api.DevicePlan(E=E, S=len(slots), R_max=2, W=len(local), G=len(local),
                          slot_expert=_i32([e for e, _ in slots]), slot_replica=_i32([r for _, r in slots]),
                          expert_nrep=torch.from_numpy(nrep).cuda(), expert_rep_weight=None, slot_widx=_i32(widx),
                          slot_gidx=_i32(widx))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(gen):
    return lambda *shape, scale=1.0, dtype=BF16: torch.randn(*shape, generator=gen, device="cuda").mul_(scale).to(dtype)


def _weights(rand, W, d, F, dtype):
    gu = torch.empty((W, 2 * F, d), dtype=dtype, device="cuda")
    dn = torch.empty((W, d, F), dtype=dtype, device="cuda")
    for w in range(W):
        gu[w] = rand(2 * F, d, scale=d ** -0.5, dtype=dtype)
        dn[w] = rand(d, F, scale=F ** -0.5, dtype=dtype)
    return gu, dn


def _routing(gen, c, m):
    """Ids and gates of micro-step m: the case's routing, its tokens in an
    order of the seed's own within every source rank (so that the plan's
    foreseen loads hold)."""
    T, S = c["T"], c.get("n_src", 1)
    bias = torch.from_numpy(_placement(*_key(c))[0][m]).to("cuda", F32)
    logits = _rand(_generator(100 + m))(T, c["E"], dtype=F32) + bias
    order = [torch.randperm(T * (s + 1) // S - T * s // S, generator=gen, device="cuda") + T * s // S for s in range(S)]
    top, ids = logits[torch.cat(order)].topk(c["K"], dim=1)
    return ids.to(torch.int32).contiguous(), torch.softmax(top, dim=1).contiguous()


def _slot_pairs(ids, slots):
    """Pair indices of every slot: an expert's pairs in ascending order, split
    in contiguous blocks floor(n r / R) over its replicas."""
    flat = ids.reshape(-1)
    nrep = {}
    for e, _ in slots:
        nrep[e] = nrep.get(e, 0) + 1
    pairs = {e: torch.nonzero(flat == e).reshape(-1) for e in nrep}
    return [pairs[e][len(pairs[e]) * r // nrep[e]:len(pairs[e]) * (r + 1) // nrep[e]] for e, r in slots]


def _local(ids, slots):
    return int(torch.isin(ids, _i32(sorted({e for e, _ in slots}))).sum())


def _dtype(c):
    return F32 if c.get("dtype") == "f32" else BF16


def _inputs(c, seed):
    """The tensors of a case, without any of the framework's handles."""
    gen, dt, kind = _generator(seed), _dtype(c), c["kind"]
    rand = _rand(gen)
    d, F = c["d"], c.get("F", 0)
    if kind == "transfer":
        n = c["records"]
        gu, dn = _weights(rand, n, d, F, dt)
        # n experts leave with parameters and gradients; they arrive in the
        # slots of their mirror images, the last two as replicas' partial
        # gradients of the first two
        return dict(gu=gu, dn=dn, ggu=rand(n, 2 * F, d, dtype=F32), gdn=rand(n, d, F, dtype=F32),
                    gu2=torch.zeros_like(gu), dn2=torch.zeros_like(dn))
    slots = _placement(*_key(c))[2]
    if kind in ("layer", "dispatch", "gathers", "update"):
        steps = []
        for m in _steps(c):
            ids, gates = _routing(gen, c, m)
            s = dict(ids=ids, gates=gates, slots=slots[m])
            if kind != "gathers":
                s["x"] = rand(c["T"], d, dtype=dt)
            if kind in ("gathers", "update") or c.get("backward"):
                s["dy"] = rand(c["T"], d, dtype=dt)
            steps.append(s)
        W = len({e for e, _ in slots[0]})
        out = dict(steps=steps)
        if kind == "gathers":
            n = _local(steps[0]["ids"], steps[0]["slots"])
            out.update(yp=rand(n, d, dtype=dt), dxp=rand(n, d, dtype=dt))
        if kind in ("layer", "update"):
            out.update(zip(("gu", "dn"), _weights(rand, W, d, F, dt)))
        return out
    # the FFN on rows already in slot order
    W = len({e for e, _ in slots[0]})
    out = dict(steps=[])
    for m, rows in zip(_steps(c), _slot_rows(c)):
        n = sum(rows)
        local = sorted({e for e, _ in slots[m]})
        s = dict(rows=rows, widx=[local.index(e) for e, _ in slots[m]])
        if kind in ("ffn_fwd", "ffn_wgrad"):
            s["x"] = rand(n, d)
        if kind in ("ffn_dgrad", "ffn_wgrad"):
            s["dy"] = rand(n, d, scale=0.3)
        if kind == "ffn_dgrad":
            s["au"] = rand(n, 2 * F)
        if kind == "ffn_wgrad":
            s["h"], s["dau"] = rand(n, F, scale=0.5), rand(n, 2 * F, scale=0.3)
        out["steps"].append(s)
    if kind != "ffn_wgrad":
        out.update(zip(("gu", "dn"), _weights(rand, W, d, F, dt)))
    return out


# ---------------------------------------------------------------------------
# Preparation: plans, workspaces and gradient buffers a program keeps
# ---------------------------------------------------------------------------
def _source_plan(c, ids):
    """The planner's placement of one micro-step and the last rank's slot
    table with the water-filled counts as per-source weights."""
    S, E, T = c["n_src"], c["E"], c["T"]
    tb = [T * s // S for s in range(S + 1)]
    host = ids.cpu().numpy()
    w = np.stack([np.bincount(host[tb[s]:tb[s + 1]].reshape(-1), minlength=E) for s in range(S)]).astype(np.int32)
    base = api.plan_base(w, 1, S, E // S)
    copy_rank, counts, _ = api.plan_micro_step(w, base, 1, S, E // S, c["reps"], S)
    t = api.plan_rank_slots(copy_rank, S - 1)
    n_local = int(sum(counts[:, e, r].sum() for e, r in zip(t["slot_expert"], t["slot_replica"])))
    plan = api.DevicePlan(E=E, S=len(t["slot_expert"]), R_max=counts.shape[2], W=len(t["local_experts"]),
                          G=len(t["local_experts"]), slot_expert=_i32(t["slot_expert"]),
                          slot_replica=_i32(t["slot_replica"]), expert_nrep=_i32(t["expert_nrep"]),
                          expert_rep_weight=None, slot_widx=_i32(t["slot_widx"]), slot_gidx=_i32(t["slot_widx"]),
                          n_src=S, src_token_begin=_i32(tb), src_rep_weight=_i32(counts.reshape(-1)))
    return plan, n_local


def prepare(c, seed):
    st, kind, dev = _inputs(c, seed), c["kind"], torch.device("cuda")
    st["case"] = c
    d, F = c["d"], c.get("F", 0)
    if kind == "transfer":
        n = c["records"]
        st["widx"], st["gidx"] = list(range(n)), list(range(n))
        st["arrive"] = list(range(n))[::-1]
        st["target"] = st["arrive"][:-2] + st["arrive"][:2]
        st["mode"] = [_lib.XFER_ASSIGN] * (n - 2) + [_lib.XFER_ADD] * 2
        st["ggu2"], st["gdn2"] = torch.zeros_like(st["ggu"]), torch.zeros_like(st["gdn"])
        st["what"] = _lib.XFER_PARAMS | _lib.XFER_GRADS
        st["buf"] = torch.empty(n * api.xfer_record_bytes(d, F, _dtype(c), st["what"]), dtype=torch.uint8, device=dev)
        return st
    if kind == "update":
        S = max(len(s["slots"]) for s in st["steps"])
        W = st["gu"].shape[0]
        st["pu"] = PolicyUpdate(c["T"], c["K"], d, F, c["E"], W, S, st["gu"], st["dn"], dev,
                                wgrad_group=min(8, c["steps"]))
        st["micro"] = [MicroStep(s["ids"], s["gates"], s["x"], s["dy"], _device_plan(c["E"], s["slots"]))
                       for s in st["steps"]]
        return st
    if kind in ("layer", "dispatch", "gathers"):
        s = st["steps"][0]
        if c.get("n_src", 1) > 1:
            st["plan"], st["n"] = _source_plan(c, s["ids"])
        else:
            # the routing is foreseen, so its local pairs are known: they
            # size the permuted buffers
            st["plan"], st["n"] = _device_plan(c["E"], s["slots"]), _local(s["ids"], s["slots"])
        st["ws"] = api.workspace(c["T"], c["K"], c["E"] * c.get("n_src", 1), dev)
    if kind == "gathers":
        s = st["steps"][0]
        _, rep_begin, _, slot_offset = api.histogram_assign(s["ids"], st["plan"], st["ws"])
        x = torch.zeros((c["T"], 8), dtype=BF16, device=dev)
        st["p2r"] = api.permute(x, s["ids"], st["plan"], rep_begin, slot_offset, st["n"], st["ws"])[2]
    if kind.startswith("ffn"):
        for s in st["steps"]:
            s["off"] = _i32(np.concatenate([[0], np.cumsum(s["rows"])]))
            s["widx"] = _i32(s["widx"])
    if kind in ("layer", "ffn_fwd", "ffn_dgrad"):
        st["rws"] = api.ffn_workspace(dev)
    if kind == "ffn_wgrad" or c.get("backward"):
        W = len({e for e, _ in _placement(*_key(c))[2][0]})
        st["dwgu"] = torch.zeros((W, 2 * F, d), dtype=F32, device=dev)
        st["dwdn"] = torch.zeros((W, d, F), dtype=F32, device=dev)
        st["wws"] = api.wgrad_workspace(d, F, dev)
    if kind == "ffn_wgrad":
        st["records"] = [dict(x_perm=s["x"], h=s["h"], dy_perm=s["dy"], d_au=s["dau"], slot_offset=s["off"],
                              slot_gidx=s["widx"]) for s in st["steps"]]
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _run_layer(st, c):
    s, plan, n = st["steps"][0], st["plan"], st["n"]
    out_dtype = _dtype(c)
    _, rep_begin, _, off = api.histogram_assign(s["ids"], plan, st["ws"])
    xp, _, p2r = api.permute(s["x"], s["ids"], plan, rep_begin, off, n, st["ws"])
    h, yp, au = api.grouped_ffn_fwd(xp, off, plan.slot_widx, st["gu"], st["dn"], save=c["backward"], ws=st["rws"])
    y = api.combine(yp, p2r, s["gates"], out_dtype=out_dtype)
    if not c["backward"]:
        return dict(y=y, pair_to_row=p2r)
    dyp, dgates = api.combine_bwd(s["dy"], yp, p2r, s["gates"])
    dau, dxp = api.grouped_ffn_dgrad(dyp, au, off, plan.slot_widx, st["gu"], st["dn"], ws=st["rws"])
    st["dwgu"].zero_()
    st["dwdn"].zero_()
    api.grouped_ffn_wgrad(xp, h, dyp, dau, off, plan.slot_gidx, st["dwgu"], st["dwdn"], ws=st["wws"])
    dx = api.permute_bwd(dxp, p2r, c["T"], c["K"], out_dtype=out_dtype)
    return dict(y=y, pair_to_row=p2r, dgates=dgates, dx=dx, dw_gate_up=st["dwgu"], dw_down=st["dwdn"])


def _run_update(st):
    pu, micro = st["pu"], st["micro"]
    pu.dw_gate_up.zero_()
    pu.dw_down.zero_()
    pu.start()
    for i, ms in enumerate(micro):
        pu.run(i, ms, pipelined=True, side_gathers=2, early_hist=True,
               next_ms=micro[i + 1] if i + 1 < len(micro) else None)
    pu.finish()
    # the last two micro-steps' token outputs are still in their buffers
    last = [pu.set_of(i, True) for i in (len(micro) - 2, len(micro) - 1)]
    return dict(dw_gate_up=pu.dw_gate_up, dw_down=pu.dw_down, y=[b["y"] for b in last],
                dgates=[b["dgates"] for b in last], dx=[b["dx"] for b in last])


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "layer":
        return _run_layer(st, c)
    if kind == "update":
        return _run_update(st)
    if kind == "dispatch":
        s, plan = st["steps"][0], st["plan"]
        counts, rep_begin, slot_count, off = api.histogram_assign(s["ids"], plan, st["ws"])
        xp, r2p, p2r = api.permute(s["x"], s["ids"], plan, rep_begin, off, st["n"], st["ws"])
        return [counts, rep_begin, slot_count, off, xp, r2p, p2r]
    if kind == "gathers":
        s, dt = st["steps"][0], _dtype(c)
        y = api.combine(st["yp"], st["p2r"], s["gates"], out_dtype=dt)
        dyp, dgates = api.combine_bwd(s["dy"], st["yp"], st["p2r"], s["gates"])
        dx = api.permute_bwd(st["dxp"], st["p2r"], c["T"], c["K"], out_dtype=dt)
        return dict(y=y, dy_perm=dyp, dgates=dgates, dx=dx)
    if kind == "ffn_fwd":
        s = st["steps"][0]
        h, yp, au = api.grouped_ffn_fwd(s["x"], s["off"], s["widx"], st["gu"], st["dn"], save=c["save"], ws=st["rws"])
        return dict(h=h, y=yp, au=au)
    if kind == "ffn_dgrad":
        s = st["steps"][0]
        dau, dxp = api.grouped_ffn_dgrad(s["dy"], s["au"], s["off"], s["widx"], st["gu"], st["dn"], ws=st["rws"])
        return dict(d_au=dau, dx=dxp)
    if kind == "ffn_wgrad":
        st["dwgu"].zero_()
        st["dwdn"].zero_()
        api.grouped_ffn_wgrad_steps(st["records"], st["dwgu"], st["dwdn"], ws=st["wws"])
        return dict(dw_gate_up=st["dwgu"], dw_down=st["dwdn"])
    # transfer: out of one set of expert arrays, into another
    api.copy_out(st["gu"], st["dn"], st["ggu"], st["gdn"], st["widx"], st["gidx"], st["what"], buf=st["buf"])
    api.copy_in(st["buf"], st["arrive"], st["target"], st["mode"], st["what"], st["gu2"], st["dn2"], st["ggu2"],
                st["gdn2"])
    return [st["gu2"], st["dn2"], st["ggu2"], st["gdn2"]]


# ---------------------------------------------------------------------------
# Algorithmic work: every input read once, every output written once
# ---------------------------------------------------------------------------
def work(c):
    kind, d, F = c["kind"], c["d"], c.get("F", 0)
    b = 4 if c.get("dtype") == "f32" else 2
    if kind == "transfer":
        n, par, grad = c["records"], 3 * d * F * b, 12 * d * F
        # copy-out reads and writes n records; copy-in reads them and writes
        # every parameter slot and the n - 2 gradient targets
        return dict(bytes=n * (par + grad) * 3 + n * par + (n - 2) * grad, flops=0)
    share = _placement(*_key(c))[3]
    W = len({e for e, _ in _placement(*_key(c))[2][0]})
    if kind in ("ffn_fwd", "ffn_dgrad", "ffn_wgrad"):
        n = c["rows"]
        if kind == "ffn_wgrad":
            return dict(bytes=n * (2 * d + 3 * F) * b + W * 12 * d * F, flops=6.0 * n * d * F)
        used = _used(c, _steps(c)[0], _slot_rows(c)[0])
        per_row = 2 * d + F + (2 * F if c.get("save") else 0) if kind == "ffn_fwd" else 2 * d + 4 * F
        return dict(bytes=n * per_row * b + used * 3 * d * F * b, flops=6.0 * n * d * F)
    T, K = c["T"], c["K"]
    n = sum(_pairs(c))
    if kind == "dispatch":
        n = n if c["n_src"] == 1 else T * K / c["P"]  # the planned share is balanced
        rows = T * (1 - (1 - n / (T * K)) ** K)  # tokens with a local pair, at least
        return dict(bytes=(rows + n) * d * b + 4 * n + 8 * T * K, flops=0)
    if kind == "gathers":
        # y_perm and dx_perm read, dy_perm written; dy read; y and dx written
        return dict(bytes=(3 * n + 3 * T) * d * b + 16 * T * K, flops=6.0 * n * d)
    steps = _steps(c)
    used = max(_used(c, m, [s * T for s in share[m]]) for m in steps)
    per_step = 2 * T * d * b + 12 * T * K
    if kind == "layer" and not c["backward"]:
        return dict(bytes=per_step + used * 3 * d * F * b, flops=6.0 * n * d * F)
    return dict(bytes=len(steps) * 2 * per_step + used * 3 * d * F * b + W * 12 * d * F, flops=18.0 * n * d * F)


def _used(c, m, rows):
    """Experts with rows to compute in micro-step m."""
    return len({e for (e, _), k in zip(_placement(*_key(c))[2][m], rows) if k >= 1})


# ---------------------------------------------------------------------------
# Tolerances and 64-bit results
# ---------------------------------------------------------------------------
def tolerance(c):
    """About four times the relative error against `exact` that the path shows
    over the ranges of draw()."""
    kind = c["kind"]
    if kind in ("dispatch", "transfer"):
        return "exact"  # integer maps, copies, and fp32 sums in a stated order
    if c.get("dtype") == "f32":
        return {"rel": 4e-6} if kind == "layer" else {"rel": 1e-6}  # measured up to 5e-7 and 2e-7
    if kind == "ffn_wgrad":
        return {"rel": 4e-6}  # bf16 operands, fp32 sums over up to 65536 rows: up to 6e-7
    if kind in ("layer", "update"):
        return {"rel": 1.5e-2}  # several bf16 intermediates: up to 4e-3
    return {"rel": 1e-2}  # one or two bf16 roundings: up to 2.4e-3


def _ffn64(x, gu, dn):
    a, u = (x @ gu.T).chunk(2, dim=1)
    h = torch.nn.functional.silu(a) * u
    return a, u, h, h @ dn.T


def _dgrad64(dy, a, u, gu, dn):
    s = torch.sigmoid(a)
    dh = dy @ dn
    dau = torch.cat([dh * u * (s + a * s * (1 - s)), dh * a * s], dim=1)
    return dau, dau @ gu


def _layer64(s, gu, dn, T, K, backward, dwgu=None, dwdn=None):
    d, local = gu.shape[2], sorted({e for e, _ in s["slots"]})
    gates = s["gates"].double().reshape(-1)
    zeros = lambda *shape: torch.zeros(shape, dtype=torch.float64, device="cuda")  # noqa: E731
    y, dx, dgates = zeros(T, d), zeros(T, d), zeros(T * K)
    p2r = torch.full((T * K,), -1, dtype=torch.int32, device="cuda")
    row = 0
    for (e, _), pairs in zip(s["slots"], _slot_pairs(s["ids"], s["slots"])):
        p2r[pairs] = torch.arange(row, row + len(pairs), dtype=torch.int32, device="cuda")
        row += len(pairs)
        w, tok = local.index(e), pairs // K
        gu64, dn64 = gu[w].double(), dn[w].double()
        x = s["x"][tok].double()
        a, u, h, yp = _ffn64(x, gu64, dn64)
        g = gates[pairs][:, None]
        y.index_add_(0, tok, g * yp)
        if backward:
            dy = s["dy"][tok].double()
            dgates[pairs] = (dy * yp).sum(1)
            dau, dxp = _dgrad64(g * dy, a, u, gu64, dn64)
            dx.index_add_(0, tok, dxp)
            dwgu[w] += dau.T @ x
            dwdn[w] += (g * dy).T @ h
    return y, p2r, dgates.reshape(T, K), dx


def exact(c, seed):
    kind = c["kind"]
    if kind in ("dispatch", "transfer"):
        return None  # bitwise outputs
    st = _inputs(c, seed)
    d, F = c["d"], c.get("F", 0)
    W = len({e for e, _ in _placement(*_key(c))[2][0]})
    dw = lambda: (torch.zeros((W, 2 * F, d), dtype=torch.float64, device="cuda"),  # noqa: E731
                  torch.zeros((W, d, F), dtype=torch.float64, device="cuda"))
    if kind == "layer":
        s = st["steps"][0]
        dwgu, dwdn = dw() if c["backward"] else (None, None)
        y, p2r, dgates, dx = _layer64(s, st["gu"], st["dn"], c["T"], c["K"], c["backward"], dwgu, dwdn)
        if not c["backward"]:
            return dict(y=y, pair_to_row=p2r)
        return dict(y=y, pair_to_row=p2r, dgates=dgates, dx=dx, dw_gate_up=dwgu, dw_down=dwdn)
    if kind == "update":
        dwgu, dwdn = dw()
        got = []
        for s in st["steps"]:
            y, _, dgates, dx = _layer64(s, st["gu"], st["dn"], c["T"], c["K"], True, dwgu, dwdn)
            got = (got + [(y, dgates, dx)])[-2:]
        return dict(dw_gate_up=dwgu, dw_down=dwdn, y=[g[0] for g in got], dgates=[g[1] for g in got],
                    dx=[g[2] for g in got])
    if kind == "gathers":
        s = st["steps"][0]
        T, K = c["T"], c["K"]
        gates = s["gates"].double().reshape(-1)
        y, dx = (torch.zeros((T, d), dtype=torch.float64, device="cuda") for _ in range(2))
        dyp, dgates = torch.zeros(st["yp"].shape, dtype=torch.float64, device="cuda"), torch.zeros_like(gates)
        row = 0
        for pairs in _slot_pairs(s["ids"], s["slots"]):
            tok, rows = pairs // K, slice(row, row + len(pairs))
            row += len(pairs)
            yp, dy, g = st["yp"][rows].double(), s["dy"][tok].double(), gates[pairs][:, None]
            y.index_add_(0, tok, g * yp)
            dx.index_add_(0, tok, st["dxp"][rows].double())
            dyp[rows] = g * dy
            dgates[pairs] = (dy * yp).sum(1)
        return dict(y=y, dy_perm=dyp, dgates=dgates.reshape(T, K), dx=dx)
    out, (dwgu, dwdn) = [], dw() if kind == "ffn_wgrad" else (None, None)
    for s in st["steps"]:
        row = 0
        for w, n in zip(s["widx"], s["rows"]):
            r = slice(row, row + n)
            row += n
            if kind == "ffn_wgrad":
                dwgu[w] += s["dau"][r].double().T @ s["x"][r].double()
                dwdn[w] += s["dy"][r].double().T @ s["h"][r].double()
                continue
            gu64, dn64 = st["gu"][w].double(), st["dn"][w].double()
            if kind == "ffn_fwd":
                a, u, h, yp = _ffn64(s["x"][r].double(), gu64, dn64)
                out.append((h, yp, torch.cat([a, u], dim=1) if c["save"] else None))
            else:
                au = s["au"][r].double()
                out.append(_dgrad64(s["dy"][r].double(), au[:, :F], au[:, F:], gu64, dn64))
    if kind == "ffn_wgrad":
        return dict(dw_gate_up=dwgu, dw_down=dwdn)
    cols = [None if v[0] is None else torch.cat(v) for v in zip(*out)]
    return dict(zip(("h", "y", "au") if kind == "ffn_fwd" else ("d_au", "dx"), cols))
