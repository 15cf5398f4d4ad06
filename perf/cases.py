"""The work that users of this package have it do, as timed cases.

A case is a plain dict. ``kind`` says which public entry points one pass goes through:

* ``step``: attention_forward and attention_backward, one training step of the layer;
* ``forward``: attention_forward alone (prefill, evaluation);
* ``indexed``: the same step through attention_forward_indexed / attention_backward_indexed,
  the option for callers short of memory;
* ``wrap_forward`` and ``wrap_backward``: the stages around an attention of the caller's own
  (the method leaves the inner attention stock): pool_score, select, gather and scatter, and
  scatter_bwd and gather_bwd.

``exact`` gives the same outputs in 64 bits from plain torch. Only the scores (fp32 by
definition) and, with them, the selected entries are rounded there.
"""
from __future__ import annotations

import math

import torch

import paper_2605_06554_amd as lh

SHARED, STRATIFIED = lh.LH_FLAG_GQA_SHARED, lh.LH_FLAG_STRATIFIED


def _case(kind, B, N, Hq, Hkv, D, p, L, k, dtype="bf16", flags=0, data="iid", name=None):
    c = dict(kind=kind, B=B, N=N, Hq=Hq, Hkv=Hkv, D=D, p=p, L=L, k=k, dtype=dtype, flags=flags, data=data)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a unit-test or debugging sized layer in fp32, bound by latency
        _case("step", 1, 1024, 2, 2, 64, 4, 3, 128, "fp32", name="step_1k_fp32"),
        # fp32 with grouped heads at a length where the attention itself counts: reference runs
        # and numerics studies; S = 2257 is ragged in every tile
        _case("step", 1, 4112, 8, 2, 128, 4, 3, 250, "fp32", name="step_4k_fp32_gqa"),
        # both ends of the paper's range for one layer (8 heads of 128, p = 4, L = 3, a 64th of
        # the sequence per level): the shortest sequence it benchmarks, ...
        _case("step", 1, 8192, 8, 8, 128, 4, 3, 128, name="step_8k_h8"),
        # ... the length it trains at, ...
        _case("step", 1, 98304, 8, 8, 128, 4, 3, 1536, name="step_96k_h8"),
        # ... and the longest, forward only: prefill of a long context
        _case("forward", 1, 524288, 8, 8, 128, 4, 3, 8192, name="forward_512k_h8"),
        # a 16-head layer with planted large keys
        _case("step", 1, 16384, 16, 16, 128, 4, 4, 2048, data="spikes", name="step_16k_h16"),
        # the benchmark's layer: 256K tokens, 32 query heads over 8 KV heads (the largest case)
        _case("step", 1, 262144, 32, 8, 128, 4, 5, 4096, data="spikes", name="step_256k_gqa"),
        # one selection per KV group, two sequences, at a common training length
        _case("step", 2, 32768, 16, 4, 128, 4, 4, 1024, flags=SHARED, name="step_32k_shared"),
        # the option that never materialises gathered rows, with heads of 64, p = 2 and dense near-ties
        _case("indexed", 1, 24576, 12, 4, 64, 2, 6, 768, data="subspace", name="indexed_24k_p2_d64"),
        # the chunked top-k with p = 3: ragged in every tile, forward only
        _case("forward", 1, 45 * 729, 6, 3, 64, 3, 5, 500, flags=STRATIFIED, name="forward_33k_p3_strat"),
        # the stages around a caller's own attention: a budget large enough that a level no longer
        # fits one workgroup's LDS (65,536 candidates)
        _case("wrap_forward", 1, 524288, 8, 8, 128, 4, 3, 16384, name="wrap_forward_512k"),
        # their adjoints at the benchmark's shape
        _case("wrap_backward", 1, 262144, 32, 8, 128, 4, 5, 4096, name="wrap_backward_256k_gqa"),
    ]


def _levels(c):
    """(rows of each level, candidates of each level, parents of each level, S)."""
    rows = [c["N"] // c["p"] ** l for l in range(c["L"])]
    cand, par = [0] * c["L"], [0] * c["L"]
    cand[-1] = rows[-1]
    for l in range(c["L"] - 1, 0, -1):
        par[l] = min(c["k"], cand[l])
        cand[l - 1] = c["p"] * par[l]
    return rows, cand, par, sum(cand)


def draw(rng):
    """One more case: lengths of 1K to 512K (odd multiples among them), 1 to 32 heads, budgets of
    a 256th to a 16th of the sequence, every kind, type and option."""
    while True:
        kind = rng.choice(["step"] * 8 + ["forward"] * 3 + ["indexed"] * 2 + ["wrap_forward"] * 2 + ["wrap_backward"] * 2)
        dtype = "fp32" if kind != "indexed" and rng.random() < 0.2 else "bf16"
        D = rng.choice([64, 128, 128])
        p = rng.choice([2, 3, 4, 4, 4])
        L = rng.choice([1] + [2, 3, 3, 4, 4, 5, 6] * 2)
        P = p ** (L - 1)
        N = P * max(1, round(math.exp(rng.uniform(math.log(1024), math.log(524288))) / P))
        Hkv = rng.choice([1, 2, 3, 4, 8, 8, 16])
        G = rng.choice([1, 1, 2, 4])
        B = rng.choice([1, 1, 1, 2])
        k = 0 if L == 1 else max(8, int(N * 2 ** rng.uniform(-8, -4)))
        flags = 0
        if L > 1 and G > 1 and rng.random() < 0.3:
            flags |= SHARED
        if L > 1 and rng.random() < 0.15:
            flags |= STRATIFIED
        data = rng.choice(["iid", "iid", "spikes", "subspace"])
        c = _case(kind, B, N, Hkv * G, Hkv, D, p, L, k, dtype, flags, data)
        if Hkv * G > 32 or N < 1024 or B * N * Hkv * G * D > 2 ** 30:
            continue
        # no dearer than the largest listed case: in bf16 half its operations; fp32 is used for far
        # smaller problems (the larger of the listed ones)
        if _flops(c) > (4e10 if dtype == "fp32" else 4e13) or _levels(c)[3] > 2 ** 18:
            continue
        return c


# ------------------------------------------------------------------ inputs

def _dtype(c):
    return torch.float32 if c["dtype"] == "fp32" else torch.bfloat16


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 + seed)
    return g


def _inputs(c, seed):
    """q, k, v, dout: standard normal; some key positions 8 times larger ("spikes"), or q and k of
    a head in one 48-dimensional subspace with a little noise ("subspace", dense near-ties)."""
    g = _gen(seed)
    B, N, Hq, Hkv, D, dt = c["B"], c["N"], c["Hq"], c["Hkv"], c["D"], _dtype(c)
    f = dict(dtype=torch.float32, device="cuda", generator=g)
    if c["data"] == "subspace":
        basis = torch.randn(Hkv, 48, D, **f) / math.sqrt(48)
        q = torch.empty(B, N, Hq, D, dtype=dt, device="cuda")
        k = torch.empty(B, N, Hkv, D, dtype=dt, device="cuda")
        for x, H in ((q, Hq), (k, Hkv)):
            for h in range(H):
                z = torch.randn(B * N, 48, **f) @ basis[h // (H // Hkv)]
                x[:, :, h] = (z + 0.1 * torch.randn(B * N, D, **f)).view(B, N, D).to(dt)
    else:
        q = torch.randn(B, N, Hq, D, **f).to(dt)
        k = torch.randn(B, N, Hkv, D, **f)
        if c["data"] == "spikes":
            k[:, torch.randperm(N, generator=g, device="cuda")[: max(1, N // 200)]] *= 8.0
        k = k.to(dt)
    v = torch.randn(B, N, Hkv, D, **f).to(dt)
    dout = torch.randn(B, N, Hq, D, **f).to(dt) if c["kind"] in ("step", "indexed") else None
    return q, k, v, dout


def _heads(c):
    """(selection heads, query heads per selection head, query heads per KV head)."""
    G = c["Hq"] // c["Hkv"]
    return (c["Hkv"], G, G) if c["flags"] & SHARED else (c["Hq"], 1, G)


def _gathered(c, seed):
    """Gathered rows (or their gradients) as a caller's attention returns them."""
    g = _gen(seed + 7919)
    S, Hs = _levels(c)[3], _heads(c)[0]
    f = dict(dtype=torch.float32, device="cuda", generator=g)
    return [torch.randn(c["B"], H, S, c["D"], **f).to(_dtype(c)) for H in (c["Hq"], Hs, Hs)]


def prepare(case, seed):
    c = case
    if c["kind"] == "wrap_backward":
        dout = torch.randn(c["B"], c["N"], c["Hq"], c["D"], device="cuda", generator=_gen(seed)).to(_dtype(c))
        pr = _problem(c)
        return dict(c=c, pr=pr, dout=dout, grads=_gathered(c, seed), slot=_slots(c, seed))
    q, k, v, dout = _inputs(c, seed)
    s = dict(c=c, q=q, k=k, v=v, dout=dout)
    if c["kind"] == "wrap_forward":
        s["pr"] = _problem(c)
        s["os"] = _gathered(c, seed)[0]
        s["ws"] = lh.workspace(s["pr"], lh.LH_OP_SELECT)
    return s


def _problem(c):
    return lh.problem(c["B"], c["N"], c["Hq"], c["Hkv"], c["D"], c["p"], c["L"], c["k"], _dtype(c), 0.0, c["flags"])


def run(state):
    s, c = state, state["c"]
    args = (c["p"], c["L"], c["k"])
    if c["kind"] == "forward":
        _, st = lh.attention_forward(s["q"], s["k"], s["v"], *args, flags=c["flags"])
        return dict(o=st["o"], idx=st["idx"], slot=st["slot"], os=st["os"], lse=st["lse"])
    if c["kind"] == "step":
        pr, st = lh.attention_forward(s["q"], s["k"], s["v"], *args, flags=c["flags"])
        dq, dk, dv = lh.attention_backward(pr, st, s["dout"])
        return dict(o=st["o"], idx=st["idx"], lse=st["lse"], dq=dq, dk=dk, dv=dv)
    if c["kind"] == "indexed":
        pr, st = lh.attention_forward_indexed(s["q"], s["k"], s["v"], *args, flags=c["flags"])
        dq, dk, dv = lh.attention_backward_indexed(pr, s["q"], s["k"], s["v"], st, s["dout"])
        return dict(o=st["o"], idx=st["idx"], lse=st["lse"], dq=dq, dk=dk, dv=dv)
    pr = s["pr"]
    B, N, Hq, Hkv, D, S, Ptot = (c["B"], c["N"], c["Hq"], c["Hkv"], c["D"], lh.lh_subseq_len(pr),
                                 lh.lh_pyramid_rows(pr))
    Hs, dt = lh.selection_heads(pr), _dtype(c)
    new = lambda *shape, dtype=dt: torch.empty(*shape, dtype=dtype, device="cuda")  # noqa: E731
    if c["kind"] == "wrap_forward":
        R = max(Ptot - N, 1)
        qp, kp, vp = new(B, R, Hq, D), new(B, R, Hkv, D), new(B, R, Hkv, D)
        s_qk, s_kq = new(B, Hq, Ptot, dtype=torch.float32), new(B, Hkv, Ptot, dtype=torch.float32)
        idx, slot = new(B, Hs, S, dtype=torch.int32), new(B, Hs, Ptot, dtype=torch.int32)
        qs, ks, vs, o = new(B, Hq, S, D), new(B, Hs, S, D), new(B, Hs, S, D), new(B, N, Hq, D)
        lh.lh_pool_score(pr, s["q"], s["k"], s["v"], qp, kp, vp, s_qk, s_kq)
        lh.lh_select_topk(pr, s_qk, s_kq, idx, slot, s["ws"])
        lh.lh_gather(pr, s["q"], s["k"], s["v"], qp, kp, vp, idx, qs, ks, vs)
        lh.lh_scatter(pr, s["os"], slot, o)
        return dict(s_qk=s_qk, s_kq=s_kq, idx=idx, slot=slot, qs=qs, ks=ks, vs=vs, o=o)
    dos = new(B, Hq, S, D)
    dq, dk, dv = new(B, N, Hq, D), new(B, N, Hkv, D), new(B, N, Hkv, D)
    lh.lh_scatter_bwd(pr, s["dout"], s["slot"], dos)
    lh.lh_gather_bwd(pr, *s["grads"], s["slot"], dq, dk, dv)
    return dict(dos=dos, dq=dq, dk=dk, dv=dv)


# ------------------------------------------------------------------ what a pass cannot do without

def _flops(c):
    """Two products of a causal pair forward; backward five (the forward keeps no weights, so the
    logits are formed again)."""
    S = _levels(c)[3]
    per = {"forward": 4, "step": 14, "indexed": 14}.get(c["kind"], 0)
    return per * c["D"] * c["B"] * c["Hq"] * (S * (S + 1) // 2)


def work(case):
    c = case
    rows, _, _, S = _levels(c)
    e = 4 if c["dtype"] == "fp32" else 2
    B, N, Hq, Hkv, Hs, D, Ptot = c["B"], c["N"], c["Hq"], c["Hkv"], _heads(c)[0], c["D"], sum(rows)
    q, kv, gq, gkv = (B * x * D * e for x in (N * Hq, N * Hkv, S * Hq, S * Hs))
    sel = 4 * B * Hs * (S + Ptot)
    if c["kind"] == "forward":
        b = 2 * q + 2 * kv + sel + gq + 4 * B * Hq * S
    elif c["kind"] in ("step", "indexed"):
        b = 4 * q + 4 * kv + 4 * B * S * (Hs + Hq)
    elif c["kind"] == "wrap_forward":
        b = 2 * q + 2 * kv + 4 * B * Ptot * (Hq + Hkv) + sel + 2 * gq + 2 * gkv
    else:
        b = q + q + 2 * kv + 2 * gq + 2 * gkv + 4 * B * Hs * Ptot
    return {"bytes": b, "flops": _flops(c)}


def tolerance(case):
    if case["kind"] == "wrap_forward":
        # pooled rows and scores are rounded once from exact sums, the gather copies; the scatter
        # adds at most L values in 32 bits
        return {"rel": 4e-3, "max": 0.04} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    # measured against 64 bits: up to 1.2e-6 in fp32, and in bf16 (P, dS and the gathered rows and
    # gradients are rounded) 0.0024 for o to 0.0063 for dq and dk with planted keys
    if case["dtype"] == "fp32":
        return {"rel": 5e-6, "max": 1e-3}
    return {"rel": 1.5e-2, "max": 0.5}


# ------------------------------------------------------------------ 64 bits, plain torch

def _select(c, scores):
    """(idx [H, S], slot [H, Ptot]) of the per-level descent over scores [H, Ptot]: the k best
    candidates of a level (ties to the lower index) are parents, their children the next level's
    candidates; every candidate is kept, ordered by window end, coarser first."""
    rows, cand, par, S = _levels(c)
    p, L, H, dev = c["p"], c["L"], scores.shape[0], scores.device
    off = [sum(rows[:l]) for l in range(L)]
    ids, keys = [], []
    cur = torch.arange(rows[-1], device=dev).expand(H, -1)
    for l in range(L - 1, -1, -1):
        ids.append(off[l] + cur)
        keys.append(((cur + 1) * p ** l - 1) * L + (L - 1 - l))
        if l == 0:
            break
        n, k = cand[l], par[l]
        if k < n:
            sc = scores.gather(1, off[l] + cur)
            step = 2048 if c["flags"] & STRATIFIED else n
            best = []
            for a in range(0, n, step):
                b = min(a + step, n)
                quota = k * b // n - k * a // n if step < n else k
                order = torch.sort(sc[:, a:b], dim=1, descending=True, stable=True).indices[:, :quota]
                best.append(a + order)
            cur = cur.gather(1, torch.cat(best, 1).sort(1).values)
        cur = (cur[:, :, None] * p + torch.arange(p, device=dev)).reshape(H, -1)
    ids, keys = torch.cat(ids, 1), torch.cat(keys, 1)
    idx = ids.gather(1, keys.argsort(1))
    slot = torch.full((H, sum(rows)), -1, dtype=torch.int64, device=dev)
    slot.scatter_(1, idx, torch.arange(S, device=dev).expand(H, -1).contiguous())
    return idx, slot


def _slots(c, seed):
    """slot [B, Hs, Ptot] of a selection by norms of standard normal rows."""
    g = _gen(seed + 104729)
    rows, Hs = _levels(c)[0], _heads(c)[0]
    out = []
    for _ in range(c["B"]):
        s0 = torch.randn(Hs, c["N"], device="cuda", generator=g).mul_(0.5).add_(math.sqrt(c["D"]))
        out.append(_select(c, _max_up(c, s0))[1].to(torch.int32))
    return torch.stack(out)


def _max_up(c, s0):
    lev = [s0] + [s0.view(s0.shape[0], -1, c["p"] ** l).amax(2) for l in range(1, c["L"])]
    return torch.cat(lev, 1)


def _norms(x):
    """fp32 norms [H, N] of x [N, H, D], a head at a time."""
    return torch.stack([x[:, h].double().square().sum(1).sqrt().float() for h in range(x.shape[1])])


def _pyramid(c, x):
    """Rows of every level, in 64 bits, of one head x [N, D]."""
    x = x.double()
    return torch.cat([x] + [x.view(-1, c["p"] ** l, c["D"]).mean(1) for l in range(1, c["L"])])


def _windows(c, slot, shifted):
    """(position, slot, 1 / p^l) of every level's contributions to base positions: entry
    floor(j / p^l), or floor((j + 1) / p^l) - 1 where the ranges are shifted."""
    rows = _levels(c)[0]
    j = torch.arange(c["N"], device=slot.device)
    for l in range(c["L"] - 1, -1, -1):
        e = (j + 1) // c["p"] ** l - 1 if shifted else j // c["p"] ** l
        m = torch.where((e >= 0) & (e < rows[l]), slot[sum(rows[:l]) + e.clamp(0, rows[l] - 1)].long(), -1)
        at = (m >= 0).nonzero()[:, 0]
        yield at, m[at], 1.0 / c["p"] ** l


def _spread(c, rows, slot):
    o = torch.zeros(c["N"], c["D"], dtype=torch.float64, device=rows.device)
    for at, m, _ in _windows(c, slot, True):
        o[at] += rows[m].double()
    return o


def _spread_adjoint(c, dout, slot, S):
    d = torch.zeros(S, c["D"], dtype=torch.float64, device=dout.device)
    for at, m, _ in _windows(c, slot, True):
        d.index_add_(0, m, dout[at].double())
    return d


def _gather_adjoint(c, g, slot, out):
    for at, m, w in _windows(c, slot, False):
        out[at] += g[m].double() * w


def _attention(c, q, k, v, do):
    """o, lse (and dq, dk, dv given do) of causal attention over [S, D] rows, by blocks of rows."""
    S, sc = q.shape[0], 1.0 / math.sqrt(c["D"])
    o, lse = torch.empty_like(q), torch.empty(S, dtype=q.dtype, device=q.device)
    dq, dk, dv = (torch.zeros_like(q) for _ in range(3)) if do is not None else (None, None, None)
    step = 2048
    for a in range(0, S, step):
        b = min(a + step, S)
        s = (q[a:b] @ k[:b].T).mul_(sc)
        s[:, a:b].masked_fill_(torch.ones(b - a, b - a, dtype=torch.bool, device=q.device).triu_(1), -math.inf)
        lse[a:b] = torch.logsumexp(s, 1)
        pr = s.sub_(lse[a:b, None]).exp_()
        o[a:b] = pr @ v[:b]
        if do is None:
            continue
        dv[:b] += pr.T @ do[a:b]
        ds = (do[a:b] @ v[:b].T).sub_((do[a:b] * o[a:b]).sum(1, keepdim=True)).mul_(pr).mul_(sc)
        dq[a:b] = ds @ k[:b]
        dk[:b] += ds.T @ q[a:b]
    return o, lse, dq, dk, dv


def exact(case, seed):
    c = case
    B, N, Hq, Hkv, D = c["B"], c["N"], c["Hq"], c["Hkv"], c["D"]
    rows, _, _, S = _levels(c)
    Hs, Gq, G = _heads(c)
    f64 = dict(dtype=torch.float64, device="cuda")
    if c["kind"] == "wrap_backward":
        s = prepare(c, seed)
        out = dict(dos=torch.empty(B, Hq, S, D, **f64), dq=torch.zeros(B, N, Hq, D, **f64),
                   dk=torch.zeros(B, N, Hkv, D, **f64), dv=torch.zeros(B, N, Hkv, D, **f64))
        for b in range(B):
            for h in range(Hq):
                slot = s["slot"][b, h // Gq]
                out["dos"][b, h] = _spread_adjoint(c, s["dout"][b, :, h], slot, S)
                _gather_adjoint(c, s["grads"][0][b, h], slot, out["dq"][b, :, h])
            for x in range(Hs):
                for name, src in (("dk", s["grads"][1]), ("dv", s["grads"][2])):
                    _gather_adjoint(c, src[b, x], s["slot"][b, x], out[name][b, :, x * Hkv // Hs])
        return out
    q, k, v, dout = _inputs(c, seed)
    given = _gathered(c, seed)[0] if c["kind"] == "wrap_forward" else None
    out = dict(o=torch.empty(B, N, Hq, D, **f64), idx=[], slot=[], lse=torch.empty(B, Hq, S, **f64),
               os=torch.empty(B, Hq, S, D, **f64), s_qk=[], s_kq=[])
    for name, H in (("qs", Hq), ("ks", Hs), ("vs", Hs)):
        out[name] = torch.empty(B, H, S, D, **f64) if given is not None else None
    for name, H in (("dq", Hq), ("dk", Hkv), ("dv", Hkv)):
        out[name] = torch.zeros(B, N, H, D, **f64) if dout is not None else None
    for b in range(B):
        s_qk, s_kq = _max_up(c, _norms(q[b])), _max_up(c, _norms(k[b]))
        both = torch.maximum(s_qk.view(Hs, Gq, -1).amax(1), s_kq.repeat_interleave(Hs // Hkv, 0))
        idx, slot = _select(c, both)
        for name, x in (("idx", idx), ("slot", slot), ("s_qk", s_qk), ("s_kq", s_kq)):
            out[name].append(x.to(torch.int32) if name in ("idx", "slot") else x.double())
        for h in range(Hq):
            x, g = h // Gq, h // G
            qs, ks, vs = (_pyramid(c, y)[idx[x]] for y in (q[b, :, h], k[b, :, g], v[b, :, g]))
            if given is not None:
                out["qs"][b, h], out["ks"][b, x], out["vs"][b, x] = qs, ks, vs
                out["o"][b, :, h] = _spread(c, given[b, h], slot[x])
                continue
            do = _spread_adjoint(c, dout[b, :, h], slot[x], S) if dout is not None else None
            os_, lse, dqs, dks, dvs = _attention(c, qs, ks, vs, do)
            out["o"][b, :, h], out["os"][b, h], out["lse"][b, h] = _spread(c, os_, slot[x]), os_, lse
            if do is not None:
                _gather_adjoint(c, dqs, slot[x], out["dq"][b, :, h])
                _gather_adjoint(c, dks, slot[x], out["dk"][b, :, g])
                _gather_adjoint(c, dvs, slot[x], out["dv"][b, :, g])
    for name in ("idx", "slot", "s_qk", "s_kq"):
        out[name] = torch.stack(out[name])
    names = {"forward": ("o", "idx", "slot", "os", "lse"),
             "wrap_forward": ("s_qk", "s_kq", "idx", "slot", "qs", "ks", "vs", "o")}
    return {n: out[n] for n in names.get(c["kind"], ("o", "idx", "lse", "dq", "dk", "dv"))}
