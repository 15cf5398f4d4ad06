"""SDPA forward and backward at the edges of the kernels' tiles and splits, against the oracle.

L = 1 gives S = N, so every S can be asked for. The sizes sit on both sides of a 32-row block
and of the blocks that the waves of a workgroup share out, and reach every split of the rows. With LH_FLAG_GQA_SHARED two query heads share a K, V head, whose
gradients sum over them."""
import numpy as np
import pytest
import torch

import bf16_floor
import oracle
import paper_2605_06554_amd as lh
from parity import check_close, check_columns, emulated_floor

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_case(S, D, dt, Hq, Hkv, shared, rng, B=1, sample=False):
    """sample: the first, a middle and the last selection head (of B Hs) against the oracle, all of
    them finite; else every head."""
    print(f"[sdpa edges] B={B} S={S} D={D} {dt} Hq={Hq} Hkv={Hkv} shared={shared}", flush=True)
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    pr = lh.problem(B, S, Hq, Hkv, D, 2, 1, 0, tdt, flags=lh.LH_FLAG_GQA_SHARED if shared else 0)
    Hs = lh.selection_heads(pr)
    x = [torch.from_numpy(rng.standard_normal((B, H, S, D))).to(tdt) for H in (Hq, Hs, Hs, Hq)]
    qs, ks, vs, dos = (t.to(DEV) for t in x)
    os_, dqs, dks, dvs = (torch.full_like(t, float("nan")) for t in (qs, qs, ks, vs))
    lse = torch.full((B, Hq, S), float("nan"), device=DEV)
    lh.lh_sdpa_fwd(pr, qs, ks, vs, os_, lse)
    lh.lh_sdpa_bwd(pr, qs, ks, vs, os_, lse, dos, dqs, dks, dvs, lh.workspace(pr, lh.LH_OP_SDPA_BWD))
    torch.cuda.synchronize()
    for name, t in (("os", os_), ("lse", lse), ("dqs", dqs), ("dks", dks), ("dvs", dvs)):
        assert bool(torch.isfinite(t).all()), f"{name}: non-finite values"
    sc, G, bf = 1.0 / np.sqrt(D), Hq // Hs, dt == "bf16"
    todo = [0, B * Hs // 2 + 1, B * Hs - 1] if sample else range(B * Hs)
    for b in range(B):
        for hs in range(Hs):
            if b * Hs + hs not in todo:
                continue
            k, v = x[1][b, hs].double().numpy(), x[2][b, hs].double().numpy()
            rk, rv = np.zeros((S, D)), np.zeros((S, D))
            ek, ev = np.zeros((S, D)), np.zeros((S, D))
            for hq in range(hs * G, hs * G + G):
                q, do = x[0][b, hq].double().numpy(), x[3][b, hq].double().numpy()
                ro, rl = oracle.sdpa_fwd(q, k, v, sc)
                rq, dk, dv = oracle.sdpa_bwd(q, k, v, ro, rl, do, sc)
                rk += dk
                rv += dv
                fo = fq = None
                if bf:
                    eo, _ = bf16_floor.sdpa_fwd(q, k, v, sc)
                    eq, dk, dv = bf16_floor.sdpa_bwd(q, k, v, eo, rl, do, sc)
                    ek += dk
                    ev += dv
                    fo, fq = emulated_floor(eo, ro), emulated_floor(eq, rq)
                check_close(f"os[{b},{hq}]", os_[b, hq], ro, dt, fo)
                check_close(f"lse[{b},{hq}]", lse[b, hq], rl, "fp32")
                check_close(f"dqs[{b},{hq}]", dqs[b, hq], rq, dt, fq)
                if not bf and S >= 32:  # (a row alone has dS = 0: nothing to be relative to)
                    check_columns(f"os[{b},{hq}]", os_[b, hq], ro)
                    check_columns(f"dqs[{b},{hq}]", dqs[b, hq], rq)
            fk = emulated_floor(bf16_floor.round_bf16(ek), rk) if bf else None
            fv = emulated_floor(bf16_floor.round_bf16(ev), rv) if bf else None
            check_close(f"dks[{b},{hs}]", dks[b, hs], rk, dt, fk)
            check_close(f"dvs[{b},{hs}]", dvs[b, hs], rv, dt, fv)
            if not bf and S >= 32:
                check_columns(f"dks[{b},{hs}]", dks[b, hs], rk)
                check_columns(f"dvs[{b},{hs}]", dvs[b, hs], rv)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S", [1, 32, 33, 128, 129, 255, 257])
def test_fp32_edges(S, D, rng):
    """A workgroup is 32 rows, its 4 or 8 waves take every 4th or 8th 32-row tile."""
    run_case(S, D, "fp32", 2, 2, False, rng)


@pytest.mark.parametrize("B", [1, 2])
@pytest.mark.parametrize("S,D,Hq,Hkv", [(161, 64, 4, 2), (97, 128, 6, 2), (545, 64, 32, 16)])
def test_fp32_shared(S, D, Hq, Hkv, B, rng):
    """dK, dV over the query heads of a shared selection; at (545, 64, 32) the row blocks fill the
    chip and the 4-wave split runs at D = 64."""
    run_case(S, D, "fp32", Hq, Hkv, True, rng, B, sample=Hq > 8)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("S,j,Hq", [(97, 0, 2), (97, 40, 2), (97, 96, 2), (545, 301, 32)])
def test_fp32_nonfinite_stays_causal(S, j, Hq, value, D):
    """One non-finite element in row j of K, V, Q or dO: rows before j of o and dQ, and for Q and dO the
    other rows and the keys after j of dK and dV, keep their bits; what depends on it is not finite."""
    print(f"[sdpa edges non-finite] S={S} D={D} j={j} value={value}", flush=True)
    Hs, col = Hq // 2, 37
    pr = lh.problem(1, S, Hq, Hs, D, 2, 1, 0, torch.float32, flags=lh.LH_FLAG_GQA_SHARED)
    g = torch.Generator(device=DEV)
    g.manual_seed(S + D)
    x = [torch.randn(1, H, S, D, device=DEV, generator=g) for H in (Hq, Hs, Hs, Hq)]
    ws = lh.workspace(pr, lh.LH_OP_SDPA_BWD)

    def step(q, k, v, do):
        o, dq, dk, dv = (torch.full_like(t, float("nan")) for t in (q, q, k, v))
        lse = torch.empty(1, Hq, S, device=DEV)
        lh.lh_sdpa_fwd(pr, q, k, v, o, lse)
        lh.lh_sdpa_bwd(pr, q, k, v, o, lse, do, dq, dk, dv, ws)
        torch.cuda.synchronize()
        return o, dq, dk, dv

    clean = step(*x)
    assert all(bool(torch.isfinite(t).all()) for t in clean)
    for n, name in enumerate(("q", "k", "v", "do")):
        y = list(x)
        y[n] = x[n].clone()
        y[n][0, -1, j, col] = value  # the last head (of Q, dO: the last of its group)
        o, dq, dk, dv = step(*y)
        query = n in (0, 3)
        for a, b, what in zip((o, dq, dk, dv), clean, ("o", "dq", "dk", "dv")):
            H = a.shape[1]
            hit = slice(H - 1, H) if query or what in ("dk", "dv") else slice(H - 2, H)
            assert torch.equal(a[:, :hit.start], b[:, :hit.start]), (name, what, "another head")
            a, b = a[0, hit], b[0, hit]
            if what in ("o", "dq"):
                assert torch.equal(a[:, :j], b[:, :j]), (name, what)
                if query:
                    assert torch.equal(a[:, j + 1:], b[:, j + 1:]), (name, what)
            elif query:
                assert torch.equal(a[:, j + 1:], b[:, j + 1:]), (name, what)
        bad = lambda t: not bool(torch.isfinite(t).any())  # noqa: E731
        if name == "v":
            assert bad(o[0, -2:, j:, col]) and bad(dq[0, -2:, j:])
        elif name == "do":
            assert bad(dv[0, -1, :j + 1, col]) and bad(dq[0, -1, j]) and bad(dk[0, -1, :j + 1])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S", [1, 33, 64, 65, 127, 128, 129, 257])
def test_bf16_few_blocks(S, D, rng):
    """Few row blocks: a workgroup owns 64 rows, each 32-row block shared by 4 waves that take 32
    rows each of every 128-row tile (up to 64 rows no block is shared)."""
    run_case(S, D, "bf16", 2, 2, False, rng)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,S,Hq,Hkv", [(2, 193, 2, 2), (1, 1313, 16, 16), (2, 1313, 8, 8), (1, 1313, 32, 32),
                                        (2, 1313, 16, 16), (1, 1377, 92, 92), (2, 1377, 46, 46), (1, 161, 4, 2),
                                        (2, 161, 4, 2), (1, 1313, 40, 20), (2, 1313, 20, 10), (1, 1377, 96, 48),
                                        (2, 1377, 48, 24), (2, 161, 96, 96)])
def test_bf16_splits(B, S, Hq, Hkv, D, rng):
    """Shapes on which a row block is shared by 4 waves (193 and 161 rows of few heads; forward: 1313 of 16),
    by 2 (forward: 1313 of 32 and 40; backward: of 16 and of 20 selections) and by none (1377; 161 of
    192 heads), with and without shared selections, in one batch and two."""
    run_case(S, D, "bf16", Hq, Hkv, Hkv != Hq, rng, B, sample=B * Hkv > 4)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S,Hq,Hkv", [(321, 4, 4), (1313, 16, 16), (1313, 32, 32), (1377, 92, 92), (161, 4, 2), (1313, 40, 20), (1377, 96, 48)])
def test_indexed_equals_gathered(S, Hq, Hkv, D):
    """The index-driven kernels give the bits of the gather followed by the plain ones, whichever
    split runs (rows in any order, some taken twice)."""
    print(f"[sdpa edges indexed] S={S} D={D} Hq={Hq} Hkv={Hkv}", flush=True)
    shared = Hkv != Hq
    pr = lh.problem(1, S, Hq, Hkv, D, 2, 1, 0, torch.bfloat16, flags=lh.LH_FLAG_GQA_SHARED if shared else 0)
    g = torch.Generator(device=DEV)
    g.manual_seed(S + D)
    new = lambda *s: torch.randn(*s, device=DEV, generator=g).to(torch.bfloat16)  # noqa: E731
    q, k, v = new(1, S, Hq, D), new(1, S, Hkv, D), new(1, S, Hkv, D)
    idx = torch.randint(0, S, (1, Hkv, S), device=DEV, generator=g).to(torch.int32)
    qs, ks, vs, dos = new(1, Hq, S, D), new(1, Hkv, S, D), new(1, Hkv, S, D), new(1, Hq, S, D)
    lh.lh_gather(pr, q, k, v, None, None, None, idx, qs, ks, vs)
    ws = lh.workspace(pr, lh.LH_OP_SDPA_BWD)
    got = []
    for indexed in (False, True):
        o, dqs, dks, dvs = (torch.full_like(t, float("nan")) for t in (qs, qs, ks, vs))
        lse = torch.full((1, Hq, S), float("nan"), device=DEV)
        if indexed:
            lh.lh_sdpa_fwd_indexed(pr, q, k, v, None, None, None, idx, o, lse)
            lh.lh_sdpa_bwd_indexed(pr, q, k, v, None, None, None, idx, o, lse, dos, dqs, dks, dvs, ws)
        else:
            lh.lh_sdpa_fwd(pr, qs, ks, vs, o, lse)
            lh.lh_sdpa_bwd(pr, qs, ks, vs, o, lse, dos, dqs, dks, dvs, ws)
        got.append((o, lse, dqs, dks, dvs))
    torch.cuda.synchronize()
    for name, a, b in zip(("os", "lse", "dqs", "dks", "dvs"), *got):
        assert bool(torch.isfinite(a).all()), f"{name}: non-finite values"
        assert torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                           b.view(torch.int16 if b.dtype == torch.bfloat16 else torch.int32)), name


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("data", ["growing", "spikes", "ramp"])
def test_bf16_splits_round_alike(data, D, rng):
    """A row's softmax weights are rounded to bf16 at one scale, whichever split of its keys runs: a
    head alone (4 waves a row block), among 60 (2 waves) and among 200 (one) gives the same rows
    but for the order of fp32 sums. The maxima of the rows' logits grow by far more than the 2^8 at
    which the accumulators are rescaled. Bound: sums of up to 700 products differ by 2^-20 of the sum
    of their sizes, so one element in 2^12 rounds to the other neighbour, 2^-8 away: 2^-14 of the
    2-norm; four times that for sums that cancel."""
    S = 700
    print(f"[sdpa edges] splits round alike S={S} D={D} {data}", flush=True)
    q, k, v = (rng.standard_normal((S, D)) for _ in range(3))
    if data == "growing":
        k *= np.linspace(0.5, 16, S)[:, None]
    elif data == "spikes":
        k[rng.permutation(S)[:S // 20]] *= 8.0
        k[:S // 2] *= 0.25
    else:  # every row's logits climb along the sequence, and fall again for the other half of the rows
        u = rng.standard_normal(D) / np.sqrt(D)
        k += np.linspace(0, 24, S)[:, None] * u * np.sqrt(D)
        q += np.where(rng.random(S) < 0.5, 1.0, -1.0)[:, None] * u * np.sqrt(D)
    got = []
    for H in (1, 60, 200):
        pr = lh.problem(1, S, H, H, D, 2, 1, 0, torch.bfloat16)
        x = [torch.from_numpy(t).to(torch.bfloat16).to(DEV).expand(1, H, S, D).contiguous() for t in (q, k, v)]
        o = torch.full_like(x[0], float("nan"))
        lse = torch.full((1, H, S), float("nan"), device=DEV)
        lh.lh_sdpa_fwd(pr, *x, o, lse)
        torch.cuda.synchronize()
        assert bool((o == o[:, :1]).all()) and bool((lse == lse[:, :1]).all()), "equal heads differ"
        got.append((o[0, 0].double(), lse[0, 0].double()))
    for o, lse in got[:2]:
        d = ((o - got[2][0]).norm() / got[2][0].norm()).item()
        print(f"  2-norm of the difference {d:.2e}, lse {(lse - got[2][1]).abs().max().item():.2e}", flush=True)
        assert d <= 2.0 ** -12
        assert (lse - got[2][1]).abs().max().item() <= 1e-5 * max(1.0, got[2][1].abs().max().item())
