"""Small batches: the one-block grouping on and around its 64-assignment groups and its
largest size, and the combine's column splits."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2606_21712_amd as moe
from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,E", [(1, 1, 1), (63, 1, 3), (64, 1, 256), (65, 1, 7), (21, 3, 5), (512, 2, 64),
                                   (513, 2, 64), (1023, 1, 2), (341, 3, 8), (1025, 1, 256), (8191, 2, 9),
                                   (8192, 2, 64), (1024, 16, 17), (1025, 16, 256),
                                   (2049, 1, 5), (4097, 1, 256), (3072, 2, 8), (6145, 1, 31), (2049, 4, 64),
                                   (6144, 2, 8), (12289, 1, 3)])
def test_permute_small(T, k, E):
    """Exactly the oracle's maps, below, at and above the single-block limit of 16384 and the
    sizes at which its wavefronts take one, 2, 4, 6, 8 and 12 groups of 64."""
    log(f"[gpu] permute maps T={T} k={k} E={E}")
    rng = np.random.default_rng(T * 31 + E)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    x = torch.zeros((T, 64), dtype=torch.bfloat16, device="cuda")
    out = moe.moe_permute(torch.from_numpy(ids).cuda(), x, E, gather_rows=False)
    torch.cuda.synchronize()
    counts, offsets, dest, tok, _ = oracle.permute(ids, np.zeros((T, 1), np.float32), E)
    for name, want in (("counts", counts), ("offsets", offsets), ("dest_rows", dest), ("sorted_token_ids", tok)):
        assert np.array_equal(out[name].cpu().numpy(), want), name


@pytest.mark.parametrize("T,k,H,dt", [(1, 1, 64, torch.bfloat16), (1, 8, 7168, torch.bfloat16),
                                      (97, 8, 7168, torch.bfloat16), (255, 2, 4096, torch.bfloat16),
                                      (1000, 3, 4160, torch.bfloat16), (2049, 4, 1088, torch.bfloat16),
                                      (4095, 2, 2112, torch.bfloat16), (300, 2, 8256, torch.float32),
                                      (33, 16, 320, torch.float32)])
def test_combine_small(T, k, H, dt):
    """Each output in float64, within k roundings of the fp32 sum and one of the store."""
    log(f"[gpu] combine T={T} k={k} H={H} {dt}")
    g = torch.Generator().manual_seed(T + k)
    yp = torch.randn(T * k, H, generator=g).to(dt)
    dest = torch.randperm(T * k, generator=g).to(torch.int32).reshape(T, k)
    w = torch.rand(T, k, generator=g)
    ys = torch.randn(T, H, generator=g).to(dt)
    y = moe.moe_combine(yp.cuda(), dest.cuda(), w.cuda(), ys.cuda()).cpu().double()
    rows = yp[dest.long()].double() * w.double()[..., None]
    ref = rows.sum(1) + ys.double()
    mag = rows.abs().sum(1) + ys.double().abs()
    bound = (k + 2) * 2.0 ** -24 * mag + (2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -23) * ref.abs()
    assert ((y - ref).abs() <= bound).all()
