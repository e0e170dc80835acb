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
@pytest.mark.parametrize("tiles", ["by_size", "64x64"])
def test_f32_groups(counts, H, F, tiles):
    """A budget of two compute units leaves all but the smallest grids to the 64 x 64 tiles."""
    c = COUNTS[counts]
    log(f"[gpu] f32 groups {counts} H={H} F={F} {tiles}")
    x, w, tok, off = make(c, H, F, torch.float32, 5)
    dx, dw, dtok, doff = x.cuda(), [t.cuda() for t in w], tok.cuda(), off.cuda()
    moe.set_cu_budget(2 if tiles == "64x64" else 0)
    try:
        y = moe.moe_grouped_ffn_gather(dx, dtok, doff, *dw)
        y2 = moe.moe_grouped_ffn(dx[dtok.long()].contiguous(), doff, *dw)
        torch.cuda.synchronize()
    finally:
        moe.set_cu_budget(0)
    assert torch.equal(y, y2)
    y = y.cpu().double()
    for e in range(len(c)):
        lo, hi = int(off[e]), int(off[e + 1])
        if hi > lo:
            ref, bound = ffn_bound(x[tok[lo:hi].long()].double(), *(t[e].double() for t in w), 0.0, 2.0 ** -24)
            assert ((y[lo:hi] - ref).abs() <= bound).all(), (e, hi - lo)


# The streaming kernels pick tiles of 32, 64, 128 or 160 rows, one to four k groups and 64 to
# 256 weight rows by the average group size and the number of tiles, and bypass the caches
# (nt) for weights of 128 MB and more: (counts, H, F), with groups on and around the tile edges
# and F, H off the column tiles.  STREAM_TILES says which kernels each reaches.
W32 = [1, 0, 16, 9, 31, 32, 33, 2]
W64 = [63, 64, 65, 1, 0, 40, 20, 30]
W128 = [127, 128, 129, 1, 0, 64, 32, 33]
W160 = [159, 160, 161, 95, 96, 97, 129, 128]
STREAM = {
    "decode_few": ([0, 1, 3, 0, 32, 33, 1], 192, 320),
    "decode_k_groups": ([2, 1, 0, 5], 4160, 64),
    "decode_many": ([1, 0, 16, 17, 31, 32, 33, 2] * 8, 2304, 576),
    "mid64": ([63, 64, 65, 1, 0, 40, 20, 30] * 8, 2112, 960),
    "mid64_few": ([63, 64, 65, 1, 0, 40], 320, 192),
    "mid64_wide": ([30, 33, 64, 65, 20, 25, 31, 28] * 8, 4096, 2048),
    "mid128": ([127, 128, 129, 1, 0, 64, 96, 97], 4160, 4160),
    "mid128_half": ([127, 128, 129, 1, 0, 64, 96, 97], 4160, 1216),
    "mid160": ([159, 160, 161, 95, 96, 97, 129, 128], 4160, 4160),
    "mid160_half": ([159, 160, 161, 320, 321, 1, 100, 128], 3136, 1664),
    "one_expert": ([577], 448, 320),
    "w32": (W32 * 8, 1152, 1088),
    "w32_gate": (W32 * 8, 192, 576),
    "w32_down": (W32 * 8, 1152, 64),
    "w32_k2": (W32 * 2, 2304, 1984),
    "w32_k2_small": (W32 * 8, 320, 192),
    "w32_k4": ([9], 8320, 8128),
    "w64_gate": (W64 * 8, 128, 576),
    "w64_down": (W64 * 8, 1152, 64),
    "w64_k2": (W64 * 2, 2304, 1984),
    "w64_k2_small": (W64 * 8, 320, 192),
    "w64_k4": ([33], 8320, 8128),
    "w128": (W128 * 8, 1088, 1088),
    "w128_gate": (W128 * 8, 512, 576),
    "w128_down": (W128 * 8, 1088, 64),
    "w128_narrow": (W128 * 8, 512, 256),
    "w128_narrow_nt": (W128 * 8, 2112, 256),
    "w160": (W160 * 8, 1088, 1088),
    "w160_gate": (W160 * 8, 512, 576),
    "w160_down": (W160 * 8, 1088, 64),
    "w160_narrow_nt": (W160 * 8, 2112, 256),
    # one GEMM on the streaming kernels, the other on the large-batch ones
    "down_streams": ([150, 160, 161, 128, 129, 257, 100, 127] * 8, 128, 640),
    "gate_streams": ([63, 64, 65, 1, 0, 96, 97, 33] * 8, 2304, 384),
}
# MXFP8 weights of 128 MB and more where the shapes above have less
STREAM_MX = {
    "mx_w32": (W32 * 8, 1152, 2304),
    "mx_w32_k2": (W32 * 2, 3968, 2176),
    "mx_w32_k4": ([9], 8448, 8064),
    "mx_w64_k2": (W64 * 2, 3968, 2176),
    "mx_w64_k4": ([33], 8448, 8064),
    "mx_w128": (W128 * 8, 1152, 1920),
    "mx_w128_narrow": (W128 * 8, 4224, 256),
}
# the kernels of (bf16 gate/up, bf16 down, MXFP8 gate/up, MXFP8 down) on 256 compute units: "weight
# rows / 64, activation rows, k groups, stages, nt" or "0", a large-batch kernel
STREAM_TILES = {
    "decode_few": ("1 32 4 3 0", "1 32 4 3 0", "1 32 4 3 0", "1 32 4 3 0"),
    "decode_k_groups": ("1 32 4 3 0", "1 32 4 3 0", "1 32 4 3 0", "1 32 4 3 0"),
    "decode_many": ("2 64 1 3 1", "2 64 1 3 1", "2 64 1 3 1", "2 64 1 3 0"),
    "mid64": ("2 64 1 3 1", "2 64 1 3 1", "2 64 1 3 1", "2 64 1 3 1"),
    "mid64_few": ("1 64 2 4 0", "1 64 2 4 0", "1 64 2 4 0", "1 64 2 4 0"),
    "mid64_wide": ("2 64 1 3 1", "2 64 1 3 1", "2 64 1 3 1", "2 64 1 3 1"),
    "mid128": ("4 128 1 3 1", "2 128 1 4 1", "4 128 1 3 1", "2 128 1 4 1"),
    "mid128_half": ("2 64 2 3 0", "2 128 1 4 0", "2 64 2 3 0", "2 128 1 4 0"),
    "mid160": ("4 160 1 3 1", "2 160 1 4 1", "0", "4 128 1 3 0"),
    "mid160_half": ("2 160 1 4 0", "2 160 1 4 0", "2 128 1 4 0", "2 128 1 4 0"),
    "one_expert": ("1 64 2 4 0", "1 64 2 4 0", "1 64 2 4 0", "1 64 2 4 0"),
    "w32": ("2 32 1 3 1", "2 32 1 3 1", "2 32 1 3 1", "2 32 1 3 0"),
    "w32_gate": ("2 32 1 3 0", "1 32 4 3 0", "2 32 1 3 0", "1 32 4 3 0"),
    "w32_down": ("1 32 4 3 0", "2 32 1 3 0", "1 32 4 3 0", "2 32 1 3 0"),
    "w32_k2": ("2 32 2 3 1", "2 32 2 3 1", "2 32 2 3 1", "2 32 2 3 0"),
    "w32_k2_small": ("2 32 2 3 0", "2 32 2 3 0", "2 32 2 3 0", "2 32 2 3 0"),
    "w32_k4": ("1 32 4 3 1", "1 32 4 3 1", "2 32 2 3 1", "1 32 4 3 0"),
    "w64_gate": ("2 64 1 3 0", "1 64 2 4 0", "2 64 1 3 0", "1 64 2 4 0"),
    "w64_down": ("1 64 2 4 0", "2 64 1 3 0", "1 64 2 4 0", "2 64 1 3 0"),
    "w64_k2": ("2 64 2 3 1", "2 64 2 3 1", "2 64 2 3 1", "2 64 2 3 0"),
    "w64_k2_small": ("2 64 2 3 0", "2 64 2 3 0", "2 64 2 3 0", "2 64 2 3 0"),
    "w64_k4": ("1 64 2 4 1", "1 64 2 4 1", "2 64 2 3 1", "1 64 2 4 0"),
    "w128": ("4 128 1 3 1", "4 128 1 3 1", "4 128 1 3 1", "4 128 1 3 0"),
    "w128_gate": ("4 128 1 3 0", "2 128 1 4 0", "4 128 1 3 0", "2 128 1 4 0"),
    "w128_down": ("2 64 2 3 0", "4 128 1 3 0", "2 64 2 3 0", "4 128 1 3 0"),
    "w128_narrow": ("2 128 1 4 0", "2 128 1 4 0", "2 128 1 4 0", "2 128 1 4 0"),
    "w128_narrow_nt": ("2 128 1 4 1", "0", "2 128 1 4 0", "0"),
    "w160": ("4 160 1 3 1", "4 160 1 3 1", "0", "0"),
    "w160_gate": ("4 160 1 3 0", "2 160 1 4 0", "0", "4 128 1 3 0"),
    "w160_down": ("2 64 2 3 0", "4 160 1 3 0", "2 128 1 4 0", "0"),
    "w160_narrow_nt": ("2 160 1 4 1", "0", "4 128 1 3 0", "0"),
    "down_streams": ("0", "2 64 2 3 0", "0", "2 64 2 3 0"),
    "gate_streams": ("2 128 1 4 1", "0", "2 128 1 4 0", "0"),
    "mx_w32": (None, None, "2 32 1 3 1", "2 32 1 3 1"),
    "mx_w32_k2": (None, None, "2 32 1 3 1", "2 32 2 3 1"),
    "mx_w32_k4": (None, None, "1 32 4 3 1", "1 32 4 3 0"),
    "mx_w64_k2": (None, None, "2 64 1 3 1", "2 64 2 3 1"),
    "mx_w64_k4": (None, None, "1 64 2 4 1", "1 64 2 4 0"),
    "mx_w128": (None, None, "4 128 1 3 1", "4 128 1 3 1"),
    "mx_w128_narrow": (None, None, "2 128 1 4 1", "0"),
}


def mx_dims(H, F):
    return (H + 127) // 128 * 128, (F + 127) // 128 * 128


@pytest.mark.parametrize("name", list(STREAM))
def test_bf16_stream(name):
    check_bf16(name, *STREAM[name])


def check_bf16(name, c, H, F):
    log(f"[gpu] bf16 groups {name} H={H} F={F}")
    x, w, tok, off = make(c, H, F, torch.bfloat16, 7)
    dx, dw, dtok, doff = x.cuda(), [t.cuda() for t in w], tok.cuda(), off.cuda()
    y = moe.moe_grouped_ffn_gather(dx, dtok, doff, *dw)
    y2 = moe.moe_grouped_ffn(dx[dtok.long()].contiguous(), doff, *dw)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    y = y.cpu().double()
    experts = [e for e in range(len(c)) if c[e]]
    for e in experts[:24]:
        lo, hi = int(off[e]), int(off[e + 1])
        ref, bound = ffn_bound(x[tok[lo:hi].long()].double(), *(t[e].double() for t in w), 2.0 ** -9, 2.0 ** -24)
        assert ((y[lo:hi] - ref).abs() <= bound).all(), (e, hi - lo)


@pytest.mark.parametrize("name", [n for n in STREAM | STREAM_MX if n not in ("mid64_wide", "mid160")])
def test_mxfp8_stream(name):
    c, H, F = (STREAM | STREAM_MX)[name]
    check_mxfp8(name, c, *mx_dims(H, F))


# Groups on the edges of the large-batch kernels' m-tiles (256 and 320 rows).  On a device's
# own compute units shapes this small take the streaming kernels; planned for four compute
# units they take the large-batch ones.
LARGE = [1, 64, 65, 256, 257, 300, 320, 321, 512, 576, 577, 0]


@pytest.mark.parametrize("dtype", ["bf16", "mxfp8"])
def test_large_kernel_edges(dtype):
    moe.set_cu_budget(4)
    try:
        if dtype == "bf16":
            check_bf16("large edges", LARGE, 320, 448)
        else:
            check_mxfp8("large edges", LARGE, 384, 640)
    finally:
        moe.set_cu_budget(0)


@pytest.mark.parametrize("dtype", ["bf16", "mxfp8"])
def test_budget_keeps_persistent_kernels(dtype):
    """Under a compute-unit budget small groups, too, run on the kernels whose grids hold to it
    (they find their tiles through a prefix launch; the streaming kernels have none)."""
    x, w, tok, off = make([5, 9], 128, 128, torch.bfloat16, 3)
    dx, dtok, doff = x.cuda(), tok.cuda(), off.cuda()
    if dtype == "bf16":
        dw = [t.cuda() for t in w]
        call = lambda: moe.moe_grouped_ffn_gather(dx, dtok, doff, *dw)
    else:
        dw = [moe.quantize_weights_mxfp8(t.cuda()) for t in w]
        xq = moe.moe_quantize_mxfp8(dx)
        call = lambda: moe.moe_grouped_ffn_mxfp8_gather(xq, dtok, doff, *dw)
    for budget, prefix in ((0, False), (8, True)):
        log(f"[gpu] {dtype} small groups, budget {budget}")
        moe.set_cu_budget(budget)
        try:
            call()
            moe.profiler_start(16)
            call()
            torch.cuda.synchronize()
            moe.profiler_stop()
            names = [n for n, _ in moe.profiler_records()]
        finally:
            moe.set_cu_budget(0)
        assert any("prefix" in n for n in names) == prefix, names


def check_mxfp8(name, c, H, F):
    """The reference is dequantized in float64; the MFMA's fp8 sums are within 2^-12 of the sum
    of the products' magnitudes, and a code of h that rounds the other way moves it by at most
    one part in eight (a scale by two)."""
    log(f"[gpu] mxfp8 groups {name} H={H} F={F}")
    x, w, tok, off = make(c, H, F, torch.bfloat16, 9)
    dx, dtok, doff = x.cuda(), tok.cuda(), off.cuda()
    dw = [moe.quantize_weights_mxfp8(t.cuda()) for t in w]
    xq = moe.moe_quantize_mxfp8(dx)
    y = moe.moe_grouped_ffn_mxfp8_gather(xq, dtok, doff, *dw)
    y2 = moe.moe_grouped_ffn_mxfp8(moe.moe_quantize_mxfp8(dx, row_map=dtok), doff, *dw)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    y = y.cpu().double()
    X = dequantize(xq)
    W = [dequantize(q).reshape(len(c), -1, q.codes.shape[-1]) for q in dw]
    experts = [e for e in range(len(c)) if c[e]]
    for e in experts[:24]:
        lo, hi = int(off[e]), int(off[e + 1])
        xe = X[tok[lo:hi].long()]
        g, u = xe @ W[0][e].T, xe @ W[1][e].T
        h = g * torch.sigmoid(g) * u
        y64 = quantize64(h) @ W[2][e].T
        # as a whole: rounding differences of h are rare and independent
        rel = (y[lo:hi] - y64).norm() / y64.norm()
        assert rel <= 1e-2, (e, hi - lo, float(rel))
        # and no single value off by more than every h code moving one step, each way at random
        # (six sigma), plus the sums' and the store's rounding
        step = (h.abs().square() @ W[2][e].square().T).sqrt() / 8
        bound = 6 * step * 0.25 + 2.0 ** -12 * (h.abs() @ W[2][e].abs().T) + 2.0 ** -8 * y64.abs() + 1e-6
        assert ((y[lo:hi] - y64).abs() <= bound).all(), (e, hi - lo)


def dequantize(q):
    """float64 values of an MXFP8 matrix (codes E4M3, scales [K / 128][rows][4])."""
    codes = q.codes.reshape(-1, q.codes.shape[-1]).cpu()
    rows, K = codes.shape
    v = codes.view(torch.float8_e4m3fn).double()
    s = q.scales[: rows * K // 32].cpu().reshape(K // 128, rows, 4).permute(1, 0, 2).reshape(rows, K // 32).double()
    return (v.reshape(rows, K // 32, 32) * torch.exp2(s - 127.0)[..., None]).reshape(rows, K)


def quantize64(v):
    """v rounded to MXFP8 and back, in float64."""
    b = v.reshape(-1, 32)
    amax = b.abs().amax(1, keepdim=True)
    s = torch.exp2(torch.where(amax > 0, (torch.frexp(amax)[1].double() - 9.0).clamp(-127, 127),
                               torch.full_like(amax, -127.0)))
    q = b / s
    step = torch.exp2((torch.frexp(q)[1].double() - 1.0).clamp_min(-6.0) - 3.0)
    return ((torch.round(q / step) * step).clamp(-448.0, 448.0) * s).reshape(v.shape)


def test_f32_grid_past_2_32_threads():
    """So many gate/up tiles (2^24 of 64 x 32, h of 137 GB) that one grid dimension would pass
    2^32 threads.  Every row repeats one of 1024 tokens, so a call on those alone, checked
    against float64, gives every row's bits (a budget of one compute unit leaves it, too, to
    the 64 x 64 tiles: the same k order)."""
    H, F, T, E, R = 64, 16384, 1024, 2, (1 << 21) + 100
    if torch.cuda.mem_get_info()[0] < 150e9:
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < 150e9:
            pytest.skip("needs 150 GB of free device memory")
    log(f"[gpu] f32 grid H={H} F={F} R={R}")
    g = torch.Generator().manual_seed(3)
    x = torch.randn(T, H, generator=g)
    w = [torch.randn(E, F, H, generator=g) * H ** -0.5, torch.randn(E, F, H, generator=g) * H ** -0.5,
         torch.randn(E, H, F, generator=g) * F ** -0.5]
    dx, dw = x.cuda(), [t.cuda() for t in w]
    tok = torch.arange(T, dtype=torch.int32, device="cuda")
    moe.set_cu_budget(1)
    try:
        few = moe.moe_grouped_ffn_gather(dx, tok.repeat(E),
                                         torch.tensor([0, T, 2 * T], dtype=torch.int32, device="cuda"), *dw)
    finally:
        moe.set_cu_budget(0)
    many = (torch.arange(R, device="cuda") * 37 % T).to(torch.int32)
    split = R // 3
    ws = torch.empty(moe.moe_grouped_ffn_workspace_bytes(R, E, H, F, torch.float32), dtype=torch.uint8, device="cuda")
    y = moe.moe_grouped_ffn_gather(dx, many, torch.tensor([0, split, R], dtype=torch.int32, device="cuda"), *dw, ws=ws)
    torch.cuda.synchronize()
    del ws
    torch.cuda.empty_cache()
    assert torch.equal(y[:split], few[many[:split].long()])
    assert torch.equal(y[split:], few[T + many[split:].long()])
    for e in range(E):
        ref, bound = ffn_bound(x[:16].double(), *(t[e].double() for t in w), 0.0, 2.0 ** -24)
        assert ((few[e * T:e * T + 16].cpu().double() - ref).abs() <= bound).all()
