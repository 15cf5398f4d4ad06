"""Scatter adjoint and gather + pool adjoint at the edges of the kernels' runs and row groups,
against the oracle: positions cut by the end of the sequence, pyramids as deep as a workgroup
holds (a head over several column slots among them), the walk that serves p > 4, head counts that
leave slots of a workgroup empty, and dQ, dK, dV in one launch or more."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_06554_amd as lh
from parity import check_close, rounding_floor

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,Hq,Hkv,D,p,L,k,dt,flags", [
    (20, 5, 5, 128, 4, 2, 3, "bf16", 0), (4 * 17, 3, 1, 64, 4, 2, 5, "fp32", 0), (16 * 33, 2, 1, 128, 4, 3, 9, "bf16", 4),
    (1024 * 2, 1, 1, 128, 4, 6, 2, "bf16", 0), (1024 * 2, 2, 1, 128, 4, 6, 2, "fp32", 0), (4096, 1, 1, 128, 4, 7, 1, "bf16", 0),
    (9 * 7, 3, 3, 64, 3, 3, 4, "fp32", 0), (243 * 3, 2, 1, 128, 3, 6, 3, "bf16", 0), (6, 1, 1, 64, 2, 2, 1, "bf16", 0),
    (128 * 3, 3, 1, 64, 2, 8, 2, "bf16", 4), (125 * 3, 2, 2, 64, 5, 4, 3, "bf16", 0), (77, 2, 2, 64, 4, 1, 0, "bf16", 0),
    (50, 4, 2, 64, 4, 1, 0, "fp32", 0)])
def test_adjoint_edges(N, Hq, Hkv, D, p, L, k, dt, flags):
    print(f"[adjoint edges] N={N} Hq={Hq} Hkv={Hkv} D={D} p={p} L={L} k={k} {dt} flags={flags}", flush=True)
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    B = 2
    pr = lh.problem(B, N, Hq, Hkv, D, p, L, k, tdt, flags=flags)
    S, Ptot, Hs = lh.lh_subseq_len(pr), lh.lh_pyramid_rows(pr), lh.selection_heads(pr)
    g = torch.Generator()
    g.manual_seed(N + D)
    sq, sk = (torch.rand(B, H, Ptot, generator=g).to(DEV) for H in (Hq, Hkv))
    idx = torch.empty(B, Hs, S, dtype=torch.int32, device=DEV)
    slot = torch.empty(B, Hs, Ptot, dtype=torch.int32, device=DEV)
    lh.lh_select_topk(pr, sq, sk, idx, slot, lh.workspace(pr, lh.LH_OP_SELECT))
    dout = torch.randn(B, N, Hq, D, generator=g).to(tdt)
    gs = [torch.randn(B, H, S, D, generator=g).to(tdt) for H in (Hq, Hs, Hs)]
    nan = float("nan")
    dos = torch.full((B, Hq, S, D), nan, dtype=tdt, device=DEV)
    dq, dk, dv = (torch.full((B, N, H, D), nan, dtype=tdt, device=DEV) for H in (Hq, Hkv, Hkv))
    lh.lh_scatter_bwd(pr, dout.to(DEV), slot, dos)
    lh.lh_gather_bwd(pr, *(x.to(DEV) for x in gs), slot, dq, dk, dv)
    torch.cuda.synchronize()
    h = oracle.Head(N, D, p, L, k, oracle.BF16 if dt == "bf16" else oracle.F32)
    ii = idx.cpu().numpy()
    fl = (lambda r: rounding_floor(r)) if dt == "bf16" else (lambda r: None)
    for b in range(B):
        for hq in range(Hq):
            sel = ii[b, hq * Hs // Hq]
            ref = oracle.scatter_bwd(h, sel, np.ascontiguousarray(dout[b, :, hq].double().numpy()))
            check_close(f"dos[{b},{hq}]", dos[b, hq], ref, dt, fl(ref))
            ref = oracle.gather_pool_bwd(h, sel, gs[0][b, hq].double().numpy())
            check_close(f"dq[{b},{hq}]", dq[b, :, hq], ref, dt, fl(ref))
        for kv in range(Hkv):
            for name, out, src in (("dk", dk, gs[1]), ("dv", dv, gs[2])):
                ref = np.zeros((N, D))
                for x in range(kv * Hs // Hkv, (kv + 1) * Hs // Hkv):
                    oracle.gather_pool_bwd(h, ii[b, x], src[b, x].double().numpy(), ref)
                check_close(f"{name}[{b},{kv}]", out[b, :, kv], ref, dt, fl(ref))
