"""bench.py's host-side helpers that the committed measurements rely on: the
expert-batch runtime-model fit, the kernel labels of rocprofv3 traces and the
algorithmic work per launch.  CPU only."""
import numpy as np
import pytest

import bench
import moegen


def test_fit_ffn_model_recovers_its_parameters():
    # times generated by the model itself, on both sides of the ridge
    t0, bw, pf, w = 300e-6, 5e12, 1.3e15, 6.4e9
    rows = []
    for T in (256, 512, 1024, 2048, 4096, 8192, 16384, 32768):
        fl = 6.0 * 4096 * 4096 * T * 4
        rows.append({"ffn_ms": (t0 + max(w / bw, fl / pf)) * 1e3, "flops": fl})
    fit = bench.fit_ffn_model(rows, w)
    assert fit["t0_us"] == pytest.approx(300, rel=1e-3)
    assert fit["weight_GBps"] == pytest.approx(5000, rel=1e-3)
    assert fit["tflops"] == pytest.approx(1300, rel=1e-3)
    assert fit["max_abs_residual_pct"] < 0.01


def test_kernel_labels():
    # demangled names as rocprofv3 traces print them
    lab = bench.kernel_label
    assert lab("void moe::(anonymous namespace)::grouped_gemm_bf16_kernel<true, 1>"
               "(moe::(anonymous namespace)::GemmArgs)") == "gemm1"
    assert lab("void moe::(anonymous namespace)::grouped_gemm_bf16_kernel<false, 0>"
               "(moe::(anonymous namespace)::GemmArgs)") == "gemm2"
    assert lab("void moe::(anonymous namespace)::grouped_gemm_fp8_kernel<true, true>"
               "(moe::(anonymous namespace)::GemmArgsF8)") == "gemm1"
    # the kernels for small groups: MXFP8 first, then gate/up; fp32 on 32 x 32 tiles
    for mx in ("false", "true"):
        for swiglu, want in (("true", "gemm1"), ("false", "gemm2")):
            assert lab(f"void moe::(anonymous namespace)::stream_gemm_kernel<{mx}, {swiglu}, 2, 32, 1, 3, true>"
                       "(moe::(anonymous namespace)::StreamArgs)") == want
    assert lab("void moe::(anonymous namespace)::grouped_gemm_f32_small_kernel<true>"
               "(moe::(anonymous namespace)::GemmArgsF)") == "gemm1"
    assert lab("void moe::(anonymous namespace)::grouped_gemm_f32_kernel<false>"
               "(moe::(anonymous namespace)::GemmArgsF)") == "gemm2"
    assert lab("void moe::(anonymous namespace)::permute_small_kernel<4>(int const*, long, int, int, int, int*, int*, "
               "int*, int*)") == "permute_small"
    assert lab("void moe::(anonymous namespace)::combine_kernel<true, 4, 8>(unsigned char const*, int const*, "
               "float const*, unsigned char const*, long, int, long, int, unsigned char*)") == "combine"
    assert lab("void moe::(anonymous namespace)::route_kernel<8, 8, true, 4>(float const*, long, int, int, int, "
               "int*, float*)") == "route"
    assert lab("moe::(anonymous namespace)::permute_rank_kernel(int const*, long, int, int, int, long, long, "
               "int const*, int*, int*, int*, int*)") == "permute_rank"
    assert lab("moe::(anonymous namespace)::tile_prefix_kernel(int const*, int, int, int, int*, int*)") == \
        "tile_prefix"


def test_workload_tokens():
    assert bench.workload("mixtral4k") is moegen.CONFIGS["mixtral4k"]
    c = bench.workload("mixtral4k", 24)
    assert (c.T, c.R, c.H, c.F, c.E, c.k) == (24, 48, 4096, 14336, 8, 2)
    assert bench.measured_traffic(c.name) is None          # no other batch's counters


def test_algorithmic_work():
    c = moegen.CONFIGS["memconstrained"]
    T, H, E, k, F, R = c.T, c.H, c.E, c.k, c.F, c.R
    fl, by = bench.algorithmic_work(c, "gemm1", gather=True)
    assert fl == 4.0 * H * F * R
    assert by == 2 * E * F * H * 2 + T * H * 2 + R * 4 + R * F * 2
    fl2, _ = bench.algorithmic_work(c, "gemm2")
    assert fl2 == 2.0 * H * F * R
    # MXFP8: one-byte codes plus one scale byte per 32 elements for the GEMM operands
    fl8, by8 = bench.algorithmic_work(c, "gemm1", gather=True, mx=True)
    assert fl8 == fl
    q = 1 + 1 / 32
    assert by8 == pytest.approx(2 * E * F * H * q + T * H * q + R * 4 + R * F * q)
    assert by8 < 0.55 * by
    _, byc = bench.algorithmic_work(c, "combine")
    assert byc == R * H * 2 + T * H * 2 + T * k * 8


def test_summarize_dense(tmp_path, capsys):
    """The --dense counter table: per kernel, the dispatches within 80% of its longest,
    vendor kernels labelled by macro tile, this library's by template instance."""
    import csv
    vendor = "Cijk_Alik_Bljk_F8BS_UserArgs_MT256x256x128_MI16x16x1_gfx950"
    ours = "void moe::(anonymous namespace)::grouped_gemm_fp8_kernel<true, true>(moe::(anonymous namespace)::GemmArgsF8)"
    rows = []
    # vendor: one long dispatch (1000 us) and one short per-expert one (100 us, left out)
    for disp, name, us, busy in ((1, vendor, 1000.0, 0.8), (2, vendor, 100.0, 0.1), (3, ours, 2000.0, 0.6)):
        cyc = 1.8e3 * us                                    # 1.8 GHz
        for cn, v in (("GRBM_GUI_ACTIVE", cyc * 8), ("SQ_VALU_MFMA_BUSY_CYCLES", busy * cyc * 1024),
                      ("TCC_HIT", 3.0), ("TCC_MISS", 1.0)):
            rows.append({"Dispatch_Id": disp, "Kernel_Name": name, "Counter_Name": cn, "Counter_Value": v,
                         "Start_Timestamp": 0, "End_Timestamp": int(us * 1e3)})
    d = tmp_path / "sq8"
    d.mkdir()
    with open(d / "run_counter_collection.csv", "w", newline="") as f:
        w = csv.DictWriter(f, fieldnames=list(rows[0]))
        w.writeheader()
        w.writerows(rows)
    bench.summarize_dense(str(tmp_path))
    out = capsys.readouterr().out.splitlines()
    by = {ln.split("|")[1].strip(): [c.strip() for c in ln.split("|")[2:-1]] for ln in out[2:]}
    assert set(by) == {"`hipBLASLt MT256x256x128`", "`grouped_gemm_fp8_kernel<true, true>`"}
    v = by["`hipBLASLt MT256x256x128`"]
    assert v[0] == "1" and v[1] == "1000.0" and v[2] == "1.800" and v[3] == "80.0" and v[-1] == "75.0"
    assert by["`grouped_gemm_fp8_kernel<true, true>`"][3] == "60.0"
