"""The rules that pick a launch's form (csrc/launch_rules.h), evaluated on the host: where
they were measured to be right, they stay.  CPU only."""
import os
import shutil
import subprocess

import pytest

from test_gpu_group_sizes import STREAM, STREAM_MX, STREAM_TILES, mx_dims

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_21712_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="session")
def rules(tmp_path_factory):
    """rules(lines) -> the choice for each line "rule arg arg ..."."""
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                    os.path.join(HERE, "native", "launch_rules.cpp"), "-o", exe], check=True)

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        out = r.stdout.splitlines()
        assert len(out) == len(lines)
        return out
    return ask


def test_permute_groups(rules):
    """Every size fits its groups; the largest sizes get no more than they fill by a third."""
    sizes = [1, 64, 1024, 1025, 2048, 2049, 4096, 4097, 6144, 6145, 8192, 8193, 12288, 12289, 16384]
    for R, n in zip(sizes, map(int, rules([f"permute {R}" for R in sizes]))):
        assert n <= 16 and n * 1024 >= R, (R, n)
        assert R <= 4096 or n * 1024 < 1.5 * R + 1024, (R, n)


def test_combine_splits(rules):
    """Every lane of a part has a vector; parts only where they were measured faster: not for
    rows of one pass (8 vectors per lane with k = 1, 2, 4) from 640 tokens, and up to 4096
    wavefronts for rows of several."""
    cases = [(T, k, H * 2 // 16) for T in (1, 96, 509, 640, 1024, 2048, 2049, 4095, 4096, 8191, 8192, 131072)
             for k in (1, 2, 3, 4, 8, 16) for H in (64, 1024, 2048, 4096, 7168, 16384)]
    for (T, k, nvec), s in zip(cases, map(int, rules(["combine %d %d %d" % c for c in cases]))):
        assert s in (1, 2, 4, 8, 16) and (s == 1 or nvec // s >= 64), (T, k, nvec, s)
        one_pass = nvec <= 64 * (8 if k in (1, 2, 4) else 2)
        if T < 4096:
            assert s == 1 or T * s <= (2800 if one_pass else 4096), (T, k, nvec, s)
            assert s == 1 or not one_pass or T < 640, (T, k, nvec, s)
        elif T < 8192:
            assert s == 1
    got = rules(["combine 96 8 896", "combine 509 4 512", "combine 2048 2 512", "combine 2048 8 896",
                 "combine 131072 4 512"])
    assert got == ["8", "4", "1", "2", "2"]


def test_tile_grid(rules):
    """Every tile has a workgroup, in launches that the runtime takes (under 2^32 threads along
    a dimension with workgroups of 512, at most 65535 along y), up to R x F of 2^37 in fp32
    gate/up tiles of 64 x 32."""
    tiles = [1, 7, 8, 9, 1000, (1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 24) - 8, 1 << 24, (1 << 24) + 511, 1 << 26]
    for n, out in zip(tiles, rules([f"grid {n}" for n in tiles])):
        x, y = map(int, out.split())
        assert x % 8 == 0 and x * y >= n and x * 512 < 1 << 32 and 1 <= y <= 65535, (n, x, y)
        assert y > 1 or x < n + 8


def stream_choices(rules, c, H, F, fp8):
    E, R = len(c), sum(c)
    return rules([f"stream {R} {E} {H} {F} 1 {fp8} 256", f"stream {R} {E} {F} {H} 0 {fp8} 256"])


def test_stream_cases_reach_their_kernels(rules):
    """The cases that the GPU tests run the streaming kernels on launch what their table says,
    and together every tile in both GEMMs and data types: bf16 with both cache policies."""
    seen = set()
    for name, tiles in STREAM_TILES.items():
        c, H, F = (STREAM | STREAM_MX)[name]
        for fp8 in (0, 1):
            want = list(tiles[2 * fp8:2 * fp8 + 2])
            if want == [None, None]:
                continue
            got = stream_choices(rules, c, *(mx_dims(H, F) if fp8 else (H, F)), fp8)
            assert got == want, (name, fp8)
            seen |= {(fp8, g, t) for g, t in enumerate(got)}
    assert set(STREAM_TILES) == set(STREAM | STREAM_MX)
    both = ["4 128 1 3", "2 128 1 4", "2 64 1 3", "2 64 2 3", "1 64 2 4", "2 32 1 3", "2 32 2 3", "1 32 4 3"]
    for g in (0, 1):
        for t in both + ["4 160 1 3", "2 160 1 4"]:
            assert {(0, g, t + " 0"), (0, g, t + " 1")} <= seen, (g, t)
        for t in both:
            assert {(1, g, t + " 0"), (1, g, t + " 1")} & seen, (g, t)
            if g == 0 or not t.startswith("1 "):       # (MXFP8 down on 64 weight rows: only small weights)
                assert (1, g, t + " 1") in seen, (g, t)


# (mean rows, H, F, experts, MXFP8, GEMM, streams): both sides of the lines, where they were measured
LINES = [
    # the shapes of the repository's workloads
    (3, 4096, 14336, 8, 0, "gate", 1), (128, 4096, 14336, 8, 0, "gate", 1), (160, 4096, 14336, 8, 0, "gate", 0),
    (128, 4096, 14336, 8, 0, "down", 1), (220, 4096, 14336, 8, 0, "down", 1), (300, 4096, 14336, 8, 0, "down", 0),
    (12, 7168, 2048, 64, 0, "gate", 1), (112, 7168, 2048, 64, 0, "gate", 1), (128, 7168, 2048, 64, 0, "gate", 0),
    (80, 7168, 2048, 64, 0, "down", 1), (96, 7168, 2048, 64, 0, "down", 0),
    (112, 4096, 4096, 64, 0, "down", 1), (128, 4096, 4096, 64, 0, "down", 0),
    (96, 4096, 14336, 8, 1, "gate", 1), (128, 4096, 14336, 8, 1, "gate", 0),
    (25, 7168, 2048, 64, 1, "down", 1), (96, 7168, 2048, 64, 1, "down", 0),
    # MXFP8 tiles of the large-batch kernel are 256 rows: a grid that it fills, and ones that it does not
    (256, 4096, 14336, 8, 1, "down", 1), (300, 4096, 14336, 8, 1, "down", 1), (330, 4096, 14336, 8, 1, "down", 0),
    (400, 5120, 1536, 4, 1, "down", 1), (640, 4096, 14336, 4, 1, "down", 1), (500, 4096, 14336, 8, 1, "down", 0),
    # bf16: few tiles, but more of the streaming kernel's than run at once
    (400, 4096, 14336, 4, 0, "down", 1), (500, 4096, 14336, 4, 0, "down", 0), (640, 5120, 1536, 4, 0, "gate", 0),
    # short k loops, and many rounds of large tiles
    (40, 2048, 768, 128, 0, "down", 1), (52, 2048, 768, 128, 0, "down", 0), (24, 2048, 768, 128, 1, "down", 1),
    (40, 2048, 768, 128, 1, "down", 0), (64, 2816, 1408, 60, 1, "down", 1), (96, 2816, 1408, 60, 1, "down", 0),
    (24, 7168, 2048, 256, 0, "down", 1), (40, 7168, 2048, 256, 0, "down", 0),
]


@pytest.mark.parametrize("mean,H,F,E,fp8,gemm,streams", LINES)
def test_stream_lines(rules, mean, H, F, E, fp8, gemm, streams):
    got = stream_choices(rules, [mean] * E, H, F, fp8)[gemm == "down"]
    assert (got != "0") == bool(streams), got
