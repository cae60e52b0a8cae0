"""The work a program that serves MoE layers through this framework has it do.

Three kinds of call, each through the public binding:

  route   easybalance_route: RMSNorm, router and top-k of one micro-batch
  step    easybalance_moe_step + easybalance_combine: the expert FFNs of a set
          of micro-batches (each at its own layer) and the weighted combine
  pass    Stack.run_native: a whole Algorithm-1 pass through every layer

A case fixes the model's shape, the micro-batches and the storage type; the
inputs follow from the case and a seed alone.
"""
import math

import numpy as np
import torch

from paper_2608_07964_amd import binding as B
from paper_2608_07964_amd.driver import Stack, pack_expert_weights

DEV = "cuda:0"
EPS = 1e-6


def _case(name, kind, *, H, F, E, k, S, L, n, T, dtype="bf16", ragged=False, norm_topk=0, skew=1.0, D=1, m=1):
    """n micro-batches of up to T tokens, spread over L layers."""
    return dict(name=name, kind=kind, H=H, F=F, E=E, k=k, S=S, L=L, n=n, T=T, dtype=dtype, ragged=ragged,
                norm_topk=norm_topk, skew=skew, D=D, m=m)


def listed():
    return [
        # Routing of a decode micro-batch (16 sequences, one token each) on
        # DeepSeek-V2-Lite-shaped layers: latency and launches.
        _case("route_decode_dsv2_lite", "route", H=2048, F=1408, E=64, k=6, S=2, L=1, n=1, T=16),
        # Routing of a prefill micro-batch on Mixtral-shaped layers (few experts).
        _case("route_prefill_mixtral", "route", H=4096, F=14336, E=8, k=2, S=0, L=1, n=1, T=2048, norm_topk=1),
        # Routing of a prefill micro-batch on DeepSeek-V3-shaped layers (256 experts).
        _case("route_prefill_dsv3", "route", H=7168, F=2048, E=256, k=8, S=1, L=1, n=1, T=4096, norm_topk=1,
              skew=1.3),
        # The smallest expert call: one sequence decoding.
        _case("step_decode_one_dsv2_lite", "step", H=2048, F=1408, E=64, k=6, S=2, L=1, n=1, T=1),
        # Batched decode, micro-batches of a few sequences at three layers at once.
        _case("step_decode_qwen", "step", H=2048, F=1408, E=60, k=4, S=4, L=3, n=6, T=16, ragged=True, skew=1.1),
        # Batched decode on large experts: weight streaming.
        _case("step_decode_mixtral", "step", H=4096, F=14336, E=8, k=2, S=0, L=1, n=4, T=16),
        # Small micro-batches at five layers: many groups of few rows.
        _case("step_cross_dsv2_lite", "step", H=2048, F=1408, E=64, k=6, S=2, L=5, n=12, T=256),
        # A cross-layer step of three prefill micro-batches on large experts.
        _case("step_cross_mixtral", "step", H=4096, F=14336, E=8, k=2, S=0, L=2, n=3, T=512),
        # Prefill of prompts of different lengths, shared experts in every row.
        _case("step_prefill_qwen", "step", H=2048, F=1408, E=60, k=4, S=4, L=2, n=6, T=1024, ragged=True, skew=1.1),
        # The largest call: long prompts on 256 experts (one GPU's share).
        _case("step_prefill_dsv3", "step", H=7168, F=2048, E=256, k=8, S=1, L=1, n=2, T=4096, skew=1.3),
        # fp32 storage: a small model kept in full precision.
        _case("step_f32", "step", H=1024, F=2816, E=16, k=2, S=1, L=2, n=4, T=256, dtype="f32", ragged=True),
        # A whole device-scheduled pass: eight micro-batches through four layers.
        _case("pass_qwen", "pass", H=2048, F=1408, E=60, k=4, S=4, L=4, n=8, T=128, skew=1.1, D=4, m=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges: sizes between the listed ones, odd ones included."""
    top = work(listed()[9])
    while True:
        kind = rng.choice(["route", "step", "step", "step", "pass"])
        f32 = rng.random() < 0.2
        H = 256 * _log_int(rng, 2, 28)
        F = 128 * _log_int(rng, 3, 112)
        E = _log_int(rng, 4, 256)
        k = rng.randint(1, min(8, E))
        S = rng.randint(0, 4)
        n, L, T, D, m = 1, 1, _log_int(rng, 1, 4096), 1, 1
        if kind == "step":
            n = _log_int(rng, 1, 16)
            L = rng.randint(1, min(5, n))
            T = _log_int(rng, 1, 4096)
        elif kind == "pass":
            n, L, T = rng.randint(2, 10), rng.randint(2, 5), _log_int(rng, 8, 512)
            D = rng.choice([d for d in (1, 2, 4, 8) if E % d == 0])
            m = max(1, (3 * n) // 4)
            f32 = f32 and E <= 64
        c = dict(kind=kind, H=H, F=F, E=E, k=k, S=S, L=L, n=n, T=T, dtype="f32" if f32 else "bf16",
                 ragged=rng.random() < 0.5 and kind == "step", norm_topk=rng.randint(0, 1),
                 skew=round(rng.uniform(0.8, 1.3), 2), D=D, m=m)
        weights = L * (E + S) * 3 * H * F * (4 if f32 else 2)
        if kind != "route" and weights > (2e9 if kind == "pass" else 12e9):
            continue
        w = work(c)
        if w["flops"] > (0.03 if f32 else 0.5) * top["flops"] or w["bytes"] > 0.5 * top["bytes"]:
            continue
        return c


# ---- inputs -----------------------------------------------------------------

def _lens(c):
    """Tokens of each micro-batch; ragged ones run from T down to about T / 2."""
    if not c["ragged"]:
        return [c["T"]] * c["n"]
    return [max(1, c["T"] - (37 * i) % (c["T"] // 2 + 1)) for i in range(c["n"])]


def _layers(c):
    return [i * c["L"] // c["n"] for i in range(c["n"])]


def _tdt(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _desc(c):
    return B.make_desc(c["L"], c["H"], c["F"], c["E"], c["k"], c["S"], c["D"], c["dtype"], EPS, c["norm_topk"])


def _gen(seed, what):
    return torch.Generator(device=DEV).manual_seed((seed * 16 + what) & 0x7FFFFFFFFFFF)


def _randn(g, *shape, dtype=torch.float32, scale=1.0):
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype).mul_(scale)


def _bias(c, seed):
    """Router bias ln p of a Zipf law in an order of its own per layer: hot and cold experts."""
    rng = np.random.default_rng(seed)
    p = (1.0 + np.arange(c["E"])) ** -c["skew"]
    p /= p.sum()
    b = np.stack([np.log(p)[rng.permutation(c["E"])] for _ in range(c["L"])])
    return torch.from_numpy(b.astype(np.float32)).to(DEV)


def _router(c, seed):
    g = _gen(seed, 1)
    return [_randn(g, c["E"], c["H"], dtype=_tdt(c), scale=c["H"] ** -0.5) for _ in range(c["L"])]


def _gain(c, seed):
    return 1.0 + _randn(_gen(seed, 2), c["L"], c["H"], scale=0.1)


def _experts(c, seed):
    """Row-major expert weights of every layer: [E+S][2F][H] and [E+S][H][F]."""
    g, ES = _gen(seed, 3), c["E"] + c["S"]
    gu = [_randn(g, ES, 2 * c["F"], c["H"], dtype=_tdt(c), scale=0.02) for _ in range(c["L"])]
    dn = [_randn(g, ES, c["H"], c["F"], dtype=_tdt(c), scale=0.02) for _ in range(c["L"])]
    return gu, dn


def _hidden(c, seed):
    g = _gen(seed, 4)
    return [_randn(g, T, c["H"]) for T in _lens(c)]


def _picks(c, seed):
    """Routing results of each micro-batch: activations, expert ids and weights."""
    g, bias = _gen(seed, 5), _bias(c, seed)
    out = []
    for T, l in zip(_lens(c), _layers(c)):
        a = _randn(g, T, c["H"], dtype=_tdt(c))
        z = _randn(g, T, c["E"]) + bias[l]
        idx = torch.topk(z, c["k"], dim=1).indices
        w = torch.gather(torch.softmax(z, 1), 1, idx)
        if c["norm_topk"]:
            w = w / w.sum(1, keepdim=True)
        out.append((a, idx.to(torch.int32).contiguous(), w.contiguous()))
    return out


def _aligned(nbytes):
    t = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)
    return t, t.data_ptr() + (-t.data_ptr()) % 256


def prepare(case, seed):
    c, desc, kind = case, _desc(case), case["kind"]
    s = dict(case=c, desc=desc)
    if kind == "route":
        T, H = c["T"], c["H"]
        s.update(x=_hidden(c, seed)[0], gain=_gain(c, seed)[0], Wg=_router(c, seed)[0], bias=_bias(c, seed)[0],
                 a=torch.empty(T, H, dtype=_tdt(c), device=DEV), z=torch.empty(T, c["E"], device=DEV),
                 idx=torch.empty(T, c["k"], dtype=torch.int32, device=DEV), w=torch.empty(T, c["k"], device=DEV),
                 counts=torch.empty(c["E"], dtype=torch.int32, device=DEV))
        return s
    gu, dn = _experts(c, seed)
    pack_expert_weights(desc, gu, dn)
    if kind == "pass":
        x0 = torch.stack(_hidden(c, seed))
        s["x0"] = x0
        s["stack"] = Stack(L=c["L"], H=c["H"], F=c["F"], E=c["E"], k=c["k"], S=c["S"], D=c["D"], N=c["n"], T=c["T"],
                           dtype=c["dtype"], x=x0.clone(), gain=_gain(c, seed), Wg=_router(c, seed),
                           bias=_bias(c, seed), W_gu=gu, W_dn=dn, eps=EPS, norm_topk=c["norm_topk"], device=DEV)
        return s
    lens, picks = _lens(c), _picks(c, seed)
    P = sum(lens) * (c["k"] + c["S"])
    ws_bytes = B.easybalance_moe_step_workspace_size(desc, lens)
    ws, ws_ptr = _aligned(ws_bytes)
    s.update(gu=gu, dn=dn, picks=picks, x=_hidden(c, seed), ws=ws, ws_ptr=ws_ptr, ws_bytes=ws_bytes,
             o=torch.empty(P, c["H"], dtype=_tdt(c), device=DEV), inv=torch.empty(P, dtype=torch.int32, device=DEV),
             run=B.work_array((i, l, T, a, idx, w) for i, (l, T, (a, idx, w)) in
                              enumerate(zip(_layers(c), lens, picks))))
    return s


def run(s):
    c, stream = s["case"], torch.cuda.current_stream().cuda_stream
    if c["kind"] == "route":
        B.easybalance_route(s["desc"], 0, c["T"], s["x"], s["gain"], s["Wg"], s["bias"], s["a"], s["z"], s["idx"],
                            s["w"], s["counts"], stream)
        return {k: s[k] for k in ("a", "z", "idx", "w", "counts")}
    if c["kind"] == "pass":
        s["stack"].x.copy_(s["x0"])  # the micro-batches' residual streams, in place
        s["stack"].run_native("maxutil", m=c["m"], record=False, device_schedule=True)
        return {"x": s["stack"].x}
    # the residual streams take the experts' sums in place, call after call
    B.easybalance_moe_step(s["desc"], s["run"], c["n"], s["gu"], s["dn"], s["ws_ptr"], s["ws_bytes"], s["o"], s["inv"],
                           None, stream)
    B.easybalance_combine(s["desc"], s["run"], c["n"], s["x"], s["o"], s["inv"], stream)
    return {"o": s["o"], "inv": s["inv"], "x": s["x"]}


# ---- what the calls cannot do without ---------------------------------------

def _distinct(c, lens, layers):
    """Distinct (layer, expert) groups with rows, for one draw of the routing."""
    rng = np.random.default_rng(1)
    p = (1.0 + np.arange(c["E"])) ** -c["skew"]
    ln_p = np.log(p / p.sum())
    perms = [rng.permutation(c["E"]) for _ in range(c["L"])]
    seen = set()
    for T, l in zip(lens, layers):
        z = rng.standard_normal((T, c["E"])) + ln_p[perms[l]]
        for e in np.unique(np.argpartition(-z, c["k"] - 1, axis=1)[:, :c["k"]]):
            seen.add((l, int(e)))
    return len(seen) + c["S"] * len(set(layers))


def work(case):
    c = case
    b = 2 if c["dtype"] == "bf16" else 4
    H, F, E, k, S = c["H"], c["F"], c["E"], c["k"], c["S"]

    def route(T):
        return T * H * (4 + b) + E * H * b + T * E * 4 + T * k * 8 + E * 4, 2 * T * H * E + 4 * T * H

    def step(lens, layers):
        tok = sum(lens)
        P = tok * (k + S)
        weights = _distinct(c, lens, layers) * 3 * H * F * b
        return weights + tok * H * (b + 8) + P * (H * b + 4) + tok * k * 8, 6 * P * H * F + 2 * P * H

    if c["kind"] == "route":
        by, fl = route(c["T"])
    elif c["kind"] == "step":
        by, fl = step(_lens(c), _layers(c))
    else:
        by = fl = 0
        for l in range(c["L"]):
            r, st = route(c["n"] * c["T"]), step([c["T"]] * c["n"], [l] * c["n"])
            by, fl = by + r[0] + st[0], fl + r[1] + st[1]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times the error seen against exact(): bf16 2.3e-3 (the rounding
    of h and o; a router's near-tie may fall the other way), a whole pass 4.6e-3
    over its four layers (a pick that flips moves its token by the size of the
    residual), fp32 1.5e-6 from the order of the sums."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.002}
    if case["kind"] == "pass":
        return {"rel": 2e-2, "max": 0.5, "differ": 0.002}
    return {"rel": 5e-3, "max": 0.05, "differ": 0.002}


# ---- the same in 64 bits ----------------------------------------------------

def _ffn(a, gu, dn):
    """One expert's FFN on rows a, in 64 bits: silu(a gate^T) * (a up^T), then down."""
    F = dn.shape[1]
    z = a @ gu.double().t()
    return (torch.nn.functional.silu(z[:, :F]) * z[:, F:]) @ dn.double().t()


def _experts_of(c, gu, dn, ents):
    """ents: (layer, a [T][H] f64, idx [T][k], w [T][k] f64).  The grouped expert
    outputs, each pair's grouped position and every entry's weighted sum."""
    ES, slots = c["E"] + c["S"], c["k"] + c["S"]
    keys, rows, base = [], [], 0
    for l, a, idx, _ in ents:
        shared = torch.arange(c["E"], ES, device=DEV).expand(a.shape[0], c["S"])
        keys.append((l * ES + torch.cat([idx.long(), shared], 1)).reshape(-1))
        rows.append(base + torch.arange(a.shape[0], device=DEV).repeat_interleave(slots))
        base += a.shape[0]
    keys, rows = torch.cat(keys), torch.cat(rows)
    a_all = torch.cat([e[1] for e in ents])
    order = torch.argsort(keys, stable=True)
    inv = torch.empty_like(order)
    inv[order] = torch.arange(order.numel(), device=DEV)
    o = torch.empty(order.numel(), c["H"], dtype=torch.float64, device=DEV)
    cnt = torch.bincount(keys, minlength=c["L"] * ES).tolist()
    at = 0
    for key, n in enumerate(cnt):
        if n:
            l, e = divmod(key, ES)
            o[at:at + n] = _ffn(a_all[rows[order[at:at + n]]], gu[l][e], dn[l][e])
            at += n
    sums, q = [], 0
    for _, a, idx, w in ents:
        T = a.shape[0]
        ww = torch.cat([w, torch.ones(T, c["S"], dtype=torch.float64, device=DEV)], 1)
        y = torch.zeros(T, c["H"], dtype=torch.float64, device=DEV)
        for r in range(slots):
            y += ww[:, r:r + 1] * o[inv[q:q + T * slots].reshape(T, slots)[:, r]]
        sums.append(y)
        q += T * slots
    return o, inv, sums


def _route64(c, x, gain, Wg, bias):
    """a in 64 bits, the logits of a as it is stored, the picks and their weights."""
    x = x.double()
    a = x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * gain.double()
    stored = a.to(_tdt(c)).double()
    z = stored @ Wg.double().t() + bias.double()
    idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :c["k"]]
    w = torch.gather(torch.softmax(z, 1), 1, idx)
    if c["norm_topk"]:
        w = w / w.sum(1, keepdim=True)
    return a, stored, z, idx, w


def exact(case, seed):
    c = case
    if c["kind"] == "route":
        a, _, z, idx, w = _route64(c, _hidden(c, seed)[0], _gain(c, seed)[0], _router(c, seed)[0], _bias(c, seed)[0])
        counts = torch.bincount(idx.reshape(-1), minlength=c["E"])
        return {"a": a, "z": z, "idx": idx.int(), "w": w, "counts": counts.int()}
    gu, dn = _experts(c, seed)
    if c["kind"] == "step":
        ents = [(l, a.double(), idx, w.double()) for l, (a, idx, w) in zip(_layers(c), _picks(c, seed))]
        o, inv, sums = _experts_of(c, gu, dn, ents)
        return {"o": o, "inv": inv.int(), "x": [x.double() + y for x, y in zip(_hidden(c, seed), sums)]}
    x = torch.stack(_hidden(c, seed)).double().reshape(-1, c["H"])
    gain, Wg, bias = _gain(c, seed), _router(c, seed), _bias(c, seed)
    for l in range(c["L"]):
        _, stored, _, idx, w = _route64(c, x, gain[l], Wg[l], bias[l])
        x = x + _experts_of(c, gu, dn, [(l, stored, idx, w)])[2][0]
    return {"x": x.reshape(c["n"], c["T"], c["H"])}
