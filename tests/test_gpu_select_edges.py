"""The selection where the radix select changes course: a first digit whose bin holds just as many
keys as are ranked outright (256), one more, or nearly all keys (further digits follow), with and
without ties at the threshold, in every key store (LDS with the lists, LDS, global) and in chunks;
and the order kernel on both sides of the line between its ranges of 1024 and 8192 window ends, where
the ranges' edges split coarse windows. Exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_06554_amd as lh
from parity import check_equal

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("inbin", [1, 255, 256, 257, 0.9])
@pytest.mark.parametrize("N,p,L,k,flags", [(2048, 4, 2, 300, 0), (32768, 4, 3, 1500, 0), (65536, 2, 2, 5000, 2),
                                           (81920, 4, 2, 9000, 0), (163840, 4, 2, 20000, 0)])
def test_bin_sizes(N, p, L, k, flags, inbin, ties, rng):
    print(f"[select edges] N={N} p={p} L={L} k={k} flags={flags} bin={inbin} ties={ties}", flush=True)
    pr = lh.problem(1, N, 1, 1, 64, p, L, k, lh.LH_F32, 0.0, flags)
    S, Ptot, off = lh.lh_subseq_len(pr), lh.lh_pyramid_rows(pr), lh.lh_level_offset(pr, L - 1)
    n = Ptot - off
    s = (rng.random(Ptot) * 0.25).astype(np.float32)
    # the top level: `m` keys close together at 2 (one bin of 2^13 steps), the rest of them below or
    # above so that the k-th key lies among the m
    m = min(int(inbin * n) if inbin < 1 else int(inbin), n - 2)
    above = max(0, k - (m + 1) // 2)
    lev = (rng.random(n) * 0.5).astype(np.float32)
    order = rng.permutation(n)
    steps = rng.integers(0, 3 if ties else 8192, m).astype(np.uint32)
    lev[order[:m]] = (np.float32(2.0).view(np.uint32) + steps).view(np.float32)
    lev[order[m:m + min(above, n - m - 1)]] = 3.0 + rng.random(min(above, n - m - 1)).astype(np.float32)
    s[off:] = lev
    sq = torch.from_numpy(s).view(1, 1, Ptot).to(DEV)
    sk = torch.zeros_like(sq)
    idx = torch.empty(1, 1, S, dtype=torch.int32, device=DEV)
    slot = torch.empty(1, 1, Ptot, dtype=torch.int32, device=DEV)
    lh.lh_select_topk(pr, sq, sk, idx, slot, lh.workspace(pr, lh.LH_OP_SELECT))
    torch.cuda.synchronize()
    ri, rs = oracle.select(oracle.Head(N, 64, p, L, k, oracle.F32, flags), s, np.zeros(Ptot, np.float32))
    check_equal("idx", idx[0, 0].cpu().numpy(), ri)
    check_equal("slot", slot[0, 0].cpu().numpy(), rs)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("N,p,L,k,H", [(20000, 5, 3, 300, 42), (20000, 5, 3, 300, 43), (9999, 3, 3, 200, 64),
                                       (9999, 3, 3, 200, 65), (19683, 3, 5, 50, 43), (16400, 2, 5, 40, 43)])
def test_order_ranges(N, p, L, k, H, flags, rng):
    """Selections x ranges of 8192 window ends: 126 and 128 (ranges of 1024 run), 129 and 130; with p = 3 and
    5 a range's edge lies inside windows of every level; at N = 16,400 the last range holds one window."""
    print(f"[select edges order] N={N} p={p} L={L} k={k} H={H} flags={flags}", flush=True)
    N -= N % p ** (L - 1)
    pr = lh.problem(1, N, H, H, 64, p, L, k, lh.LH_F32, 0.0, flags)
    S, Ptot = lh.lh_subseq_len(pr), lh.lh_pyramid_rows(pr)
    s = rng.random((H, Ptot)).astype(np.float32)
    sq = torch.from_numpy(s).view(1, H, Ptot).to(DEV)
    idx = torch.empty(1, H, S, dtype=torch.int32, device=DEV)
    slot = torch.empty(1, H, Ptot, dtype=torch.int32, device=DEV)
    lh.lh_select_topk(pr, sq, torch.zeros_like(sq), idx, slot, lh.workspace(pr, lh.LH_OP_SELECT))
    torch.cuda.synchronize()
    head = oracle.Head(N, 64, p, L, k, oracle.F32, flags)
    for h in range(H):
        ri, rs = oracle.select(head, s[h], np.zeros(Ptot, np.float32))
        check_equal(f"idx[{h}]", idx[0, h].cpu().numpy(), ri)
        check_equal(f"slot[{h}]", slot[0, h].cpu().numpy(), rs)
