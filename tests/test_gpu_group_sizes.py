"""Grouped FFN on expert groups whose sizes sit on the edges of the kernels' row tiles
(empty, one row, a tile less one, a tile, a tile and one, several tiles and a ragged
rest), with F and H at their smallest and at odd multiples of the column tiles, against
the same values in float64 on the CPU."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2606_21712_amd as moe
from gpu_util import log

pytestmark = pytest.mark.gpu

# rows per expert: edges of 16-, 32- and 64-row tiles
COUNTS = {
    "edges": [0, 1, 15, 16, 17, 0, 31, 32, 33, 63, 64, 65, 0],
    "one_expert": [129],
    "many_empty": [0] * 70 + [3] + [0] * 60 + [64, 1],
}


def ffn_bound(x, wg, wu, wd, eps_store, eps_sum):
    """y in float64 and a bound on another summation's distance from it.  eps_sum: the
    relative error of one product or addition; a sum of n terms is within (n + 4) eps_sum of
    the sum of its terms' magnitudes.  eps_store: the relative rounding of h and of y as
    stored (0: not rounded further).  |silu'| <= 1.1; silu and its product add a few
    roundings of h itself."""
    H, F = x.shape[1], wg.shape[0]
    g, u = x @ wg.T, x @ wu.T
    dg = (H + 4) * eps_sum * (x.abs() @ wg.abs().T)
    du = (H + 4) * eps_sum * (x.abs() @ wu.abs().T)
    s = g * torch.sigmoid(g)
    h = s * u
    dh = 1.1 * dg * u.abs() + s.abs() * du + 1.1 * dg * du + (8 * eps_sum + eps_store) * h.abs()
    y = h @ wd.T
    dy = dh @ wd.abs().T + (F + 4) * eps_sum * (h.abs() @ wd.abs().T)
    return y, dy + eps_store * (y.abs() + dy)


def make(counts, H, F, dt, seed):
    g = torch.Generator().manual_seed(seed)
    E, R = len(counts), sum(counts)
    T = max(1, R // 2)
    x = torch.randn(T, H, generator=g).to(dt)
    w = [(torch.randn(E, F, H, generator=g) * H ** -0.5).to(dt), (torch.randn(E, F, H, generator=g) * H ** -0.5).to(dt),
         (torch.randn(E, H, F, generator=g) * F ** -0.5).to(dt)]
    tok = torch.randint(0, T, (R,), generator=g, dtype=torch.int32)
    off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32)
    return x, w, tok, off


@pytest.mark.parametrize("counts", list(COUNTS))
@pytest.mark.parametrize("H,F", [(64, 64), (192, 320), (576, 64), (64, 448)])
def test_f32_groups(counts, H, F):
    c = COUNTS[counts]
    log(f"[gpu] f32 groups {counts} H={H} F={F}")
    x, w, tok, off = make(c, H, F, torch.float32, 5)
    dx, dw, dtok, doff = x.cuda(), [t.cuda() for t in w], tok.cuda(), off.cuda()
    y = moe.moe_grouped_ffn_gather(dx, dtok, doff, *dw)
    y2 = moe.moe_grouped_ffn(dx[dtok.long()].contiguous(), doff, *dw)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    y = y.cpu().double()
    for e in range(len(c)):
        lo, hi = int(off[e]), int(off[e + 1])
        if hi > lo:
            ref, bound = ffn_bound(x[tok[lo:hi].long()].double(), *(t[e].double() for t in w), 0.0, 2.0 ** -24)
            assert ((y[lo:hi] - ref).abs() <= bound).all(), (e, hi - lo)
