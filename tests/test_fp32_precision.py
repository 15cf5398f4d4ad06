"""The fp32 SDPA keeps fp32's precision: every column of o, dQ, dK and dV within COL_TOL of 64 bits,
relative to the column (parity.py), on plain data and on operands of mixed magnitude.

The kernels form an fp32 product from six of the nine products of bf16 parts (high, middle, low). That
the bar can see a lost part is shown on the CPU: the same arithmetic with six products meets it, as
plain fp32 does, and without the low parts (16 bits of each operand) it does not, on any of the data."""
import numpy as np
import pytest
import torch

import paper_2605_06554_amd as lh
from parity import COL_TOL, check_columns, column_error

DATA = ["normal", "columns", "spikes", "rows"]
NAMES = ("os", "dqs", "dks", "dvs")
SIX = ("mm", "lh", "hl", "mh", "hm", "hh")
FOUR = ("mm", "mh", "hm", "hh")  # no low parts
THREE = ("mh", "hm", "hh")


def operands(S, D, data):
    """q, k, v, do [S, D]. columns: the products q k and do v are sums of terms of one size whose factors
    differ by up to 2^12 each way; spikes: a few keys with logits of 10 and more; rows: dO and V rows of
    mixed magnitude."""
    r = np.random.default_rng(S + D)
    q, k, v, do = (r.standard_normal((S, D)) for _ in range(4))
    if data == "columns":
        c, e = 2.0 ** r.integers(-12, 13, D), 2.0 ** r.integers(-12, 13, D)
        q, k, v, do = q * c, k / c, v * e, do / e
    elif data == "spikes":
        k[r.permutation(S)[:max(1, S // 20)]] *= 4
    elif data == "rows":
        do *= 2.0 ** r.integers(-3, 4, S)[:, None]
        v *= 2.0 ** r.integers(-3, 4, S)[:, None]
    return [x.astype(np.float32) for x in (q, k, v, do)]


def exact(q, k, v, do, scale):
    q, k, v, do = (x.astype(np.float64) for x in (q, k, v, do))
    s = np.where(np.tril(np.ones((len(q),) * 2, bool)), q @ k.T * scale, -np.inf)
    p = np.exp(s - s.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    o = p @ v
    ds = p * (do @ v.T - (o * do).sum(1)[:, None])
    return o, ds @ k * scale, ds.T @ q * scale, p.T @ do


def split(x):
    """An fp32 array as its high, middle and low bf16 parts."""
    x = np.ascontiguousarray(x, np.float32)
    bf = lambda y: torch.from_numpy(y).to(torch.bfloat16).float().numpy()  # noqa: E731
    h = (x.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    m = bf(x - h)
    return {"h": h.astype(np.float64), "m": m.astype(np.float64), "l": bf(x - h - m).astype(np.float64)}


def emulated(q, k, v, do, scale, terms):
    """Forward and backward with products of the given parts, 16 columns at a time (exact), summed in fp32."""
    f = np.float32

    def mm(a, b):
        A, B = split(a), split(b)
        out = np.zeros((a.shape[0], b.shape[1]), f)
        for c in range(0, a.shape[1], 16):
            for x, y in terms:
                out = (out + A[x][:, c:c + 16] @ B[y][c:c + 16]).astype(f)
        return out

    mask = np.tril(np.ones((len(q),) * 2, bool))
    s = mm(q, k.T)
    m = np.where(mask, s, -np.inf).max(1).astype(f)
    w = np.where(mask, np.exp2((s - m[:, None]) * f(scale * np.log2(np.e))), 0).astype(f)
    l = w.sum(1, dtype=f)
    o = mm(w, v) / l[:, None]
    p = np.where(mask, np.exp(s * f(scale) - (m * f(scale) + np.log(l))[:, None]), 0).astype(f)
    ds = p * (mm(do, v.T) - (o * do).sum(1, dtype=f)[:, None])
    return o, mm(ds, k) * f(scale), mm(ds.T, q) * f(scale), mm(p.T, do)


@pytest.mark.parametrize("data", DATA)
@pytest.mark.parametrize("S,D", [(33, 128), (257, 64)])
def test_bar_sees_a_lost_part(S, D, data):
    x = operands(S, D, data)
    ref = exact(*x, D ** -0.5)
    err = {t: [column_error(a, b) for a, b in zip(emulated(*x, D ** -0.5, t), ref)] for t in (SIX, FOUR, THREE)}
    assert max(err[SIX]) <= COL_TOL / 2
    assert min(err[FOUR]) > 2 * COL_TOL and min(err[THREE]) > 2 * COL_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("data", DATA)
@pytest.mark.parametrize("S,D,H", [(33, 64, 1), (257, 64, 2), (700, 64, 30), (33, 128, 1), (257, 128, 2), (1000, 128, 2)])
def test_fp32_kernels(S, D, H, data):
    """D = 64 with 8 waves a workgroup and, from 545 row blocks (641 in the backward, which has twice as
    many), 4; D = 128."""
    print(f"[fp32 precision] S={S} D={D} H={H} {data}", flush=True)
    x = operands(S, D, data)
    ref = exact(*x, D ** -0.5)
    pr = lh.problem(1, S, H, H, D, 2, 1, 0, torch.float32)
    qs, ks, vs, dos = (torch.from_numpy(t).cuda().expand(1, H, S, D).contiguous() for t in x)
    out = [torch.full_like(qs, float("nan")) for _ in range(4)]
    lse = torch.empty(1, H, S, device="cuda")
    lh.lh_sdpa_fwd(pr, qs, ks, vs, out[0], lse)
    lh.lh_sdpa_bwd(pr, qs, ks, vs, out[0], lse, dos, *out[1:], lh.workspace(pr, lh.LH_OP_SDPA_BWD))
    torch.cuda.synchronize()
    for name, o, r in zip(NAMES, out, ref):
        assert torch.equal(o, o[:, :1].expand_as(o)), f"{name}: equal heads differ"
        check_columns(name, o[0, 0], r)
