"""Pooling and scores at the edges of the kernel's row groups, bit for bit against the oracle:
leaves cut by the end of the sequence, pyramids as deep as a workgroup holds (one head slot per
workgroup, leaves of 16 and of 64 rows), the walk that serves p > 4, head counts that leave slots
of a workgroup empty."""
import pytest
import torch

import oracle
import paper_2605_06554_amd as lh
from parity import check_equal, to64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,Hq,Hkv,D,p,L,dt", [
    (20, 5, 5, 128, 4, 2, "bf16"), (4 * 17, 3, 1, 64, 4, 2, "fp32"), (16 * 33, 2, 1, 128, 4, 3, "bf16"),
    (1024 * 2, 1, 1, 128, 4, 6, "bf16"), (1024, 3, 1, 64, 4, 6, "fp32"), (1024 * 2, 1, 1, 128, 4, 6, "fp32"),
    (4096, 1, 1, 128, 4, 7, "bf16"), (9 * 7, 3, 3, 64, 3, 3, "fp32"), (243 * 3, 2, 1, 128, 3, 6, "bf16"),
    (6, 1, 1, 64, 2, 2, "bf16"), (128 * 3, 3, 1, 64, 2, 8, "bf16"), (125 * 3, 2, 2, 64, 5, 4, "bf16"),
    (49 * 3, 1, 1, 128, 7, 3, "fp32"), (77, 2, 1, 64, 4, 1, "bf16")])
def test_pool_score_edges(N, Hq, Hkv, D, p, L, dt):
    print(f"[pool edges] N={N} Hq={Hq} Hkv={Hkv} D={D} p={p} L={L} {dt}", flush=True)
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    B = 2
    pr = lh.problem(B, N, Hq, Hkv, D, p, L, 1, tdt)
    Ptot = lh.lh_pyramid_rows(pr)
    R = Ptot - N
    g = torch.Generator()
    g.manual_seed(N + D)
    q, k, v = (torch.randn(B, N, H, D, generator=g).to(tdt) for H in (Hq, Hkv, Hkv))
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    nan = float("nan")
    pyr = [torch.full((B, max(R, 1), H, D), nan, dtype=tdt, device=DEV) for H in (Hq, Hkv, Hkv)]
    sqk, skq = (torch.full((B, H, Ptot), nan, device=DEV) for H in (Hq, Hkv))
    lh.lh_pool_score(pr, qd, kd, vd, *pyr, sqk, skq)
    alone = [torch.full_like(x, nan) for x in pyr]
    s2 = [torch.full_like(x, nan) for x in (sqk, skq)]
    lh.lh_pyramid_pool(pr, qd, kd, vd, *alone)
    lh.lh_score(pr, qd, kd, *s2)
    torch.cuda.synchronize()
    assert torch.equal(sqk, s2[0]) and torch.equal(skq, s2[1])
    if R:
        assert all(torch.equal(a, b) for a, b in zip(pyr, alone))
    h = oracle.Head(N, D, p, L, 1, oracle.BF16 if dt == "bf16" else oracle.F32)
    for b in range(B):
        for x, py, s, H in ((q, pyr[0], sqk, Hq), (k, pyr[1], skq, Hkv), (v, pyr[2], None, Hkv)):
            for hh in range(H):
                rows = x[b, :, hh].double().numpy()
                if s is not None:
                    check_equal(f"scores[{b},{hh}]", s[b, hh], oracle.scores(h, rows))
                if R:
                    check_equal(f"pyramid[{b},{hh}]", to64(py[b, :, hh]), oracle.pool(h, rows)[N:])


@pytest.mark.parametrize("B", [44, 45])
def test_walk_and_leaves_agree(B):
    """p = 4, L = 6, D = 128, 16 head slots: batches of 45 give the walk 720 workgroups, from which it is
    launched; one batch alone runs in leaves. Bit for bit alike, and against the oracle."""
    N, Hq, Hkv, D, p, L = 16384, 12, 2, 128, 4, 6
    print(f"[pool edges walk] B={B}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(B)
    x = [torch.randn(B, N, H, D, device=DEV, generator=g).to(torch.bfloat16) for H in (Hq, Hkv, Hkv)]

    def run(B, x):
        pr = lh.problem(B, N, Hq, Hkv, D, p, L, 1, torch.bfloat16)
        Ptot = lh.lh_pyramid_rows(pr)
        nan = float("nan")
        pyr = [torch.full((B, Ptot - N, H, D), nan, dtype=torch.bfloat16, device=DEV) for H in (Hq, Hkv, Hkv)]
        s = [torch.full((B, H, Ptot), nan, device=DEV) for H in (Hq, Hkv)]
        lh.lh_pool_score(pr, *x, *pyr, *s)
        torch.cuda.synchronize()
        return pyr + s

    all_ = run(B, x)
    for b in range(B):
        for a, one in zip(all_, run(1, [t[b:b + 1] for t in x])):
            assert torch.equal(a[b:b + 1], one), b
    h = oracle.Head(N, D, p, L, 1, oracle.BF16)
    rows = x[0][B - 1, :, Hq - 1].double().cpu().numpy()
    check_equal("scores", all_[3][B - 1, Hq - 1], oracle.scores(h, rows))
    check_equal("pyramid", to64(all_[0][B - 1, :, Hq - 1]), oracle.pool(h, rows)[N:])
