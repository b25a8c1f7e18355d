"""Host-side checks of the benchmark's accounting (no GPU): the algorithmic bytes and operations
that the roofline line is built from, which bound is reported for which workload, and that a run
on more than one GPU is refused."""
import os
import subprocess
import sys

import pytest

import bench
from paper_2605_00422_amd import binding as B
from paper_2605_00422_amd import inputs as syn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def _library():
    """The kernels' names come from the library's dispatch, which needs no GPU."""
    if not os.path.exists(B.LIB_PATH):
        from paper_2605_00422_amd.build import build_library
        build_library()


def test_linear_forward_bytes_of_the_default_workload():
    """cfg1 (one token, 4096 -> 11008, rank 32): sign bits 5.64 MB + fp16 alpha and V + the codes,
    scale and code sum of one token + T + the fp32 output row = 6.41 MB, counted term by term."""
    cfg = syn.CONFIGS["cfg1_decode7b"]
    assert (cfg.M, cfg.K, cfg.N, cfg.r) == (1, 4096, 11008, 32)
    bits, alpha, V = 11008 * 4096 // 8, 2 * 11008, 2 * 11008 * 32
    codes, scale_qsum, T, Y = 4096, 8, 4 * 32, 4 * 11008
    assert bench.linear_forward_bytes(cfg) == bits + alpha + V + codes + scale_qsum + T + Y == 6410888
    assert bench.gemm_ops(cfg) == 2 * 11008 * 4096


def test_roofline_fields_and_bound_selection():
    cfg1 = syn.CONFIGS["cfg1_decode7b"]
    traffic = bench.measured_traffic()
    # two launches per layer: the dominant kernel is the GEMM of bwla_linear_forward, the layer beside it
    r = bench.roofline_for(cfg1, 2, 13.0, 5.0, None, traffic)
    assert r["bound"] == "hbm" and r["unit"] == "GB/s" and r["peak"] == 8000.0
    assert r["kernel"] == "gemm_decode_bs_kernel"
    assert abs(r["achieved"] - 6410888 / 5e-6 / 1e9) < 1e-6 and abs(r["frac"] - r["achieved"] / 8000.0) < 1e-12
    assert abs(r["layer"]["achieved"] - bench.layer_bytes(cfg1) / 13e-6 / 1e9) < 1e-6 and r["layer"]["launches"] == 2
    # the measured traffic comes from the tracked counter summary, and is no less than the algorithmic bytes
    assert r["traffic"] == traffic[("cfg1_decode7b", "gemm_decode_bs_kernel")] >= 6410888
    # one launch per layer: the kernel is the layer
    r1 = bench.roofline_for(cfg1, 1, 7.0, 5.0, None, traffic)
    assert r1["kernel"] == "decode_layer_kernel" and r1["bytes_per_launch"] == bench.layer_bytes(cfg1)
    assert abs(r1["achieved"] - bench.layer_bytes(cfg1) / 7e-6 / 1e9) < 1e-6 and r1["layer"]["frac"] == r1["frac"]
    assert r1["traffic"] == traffic[("cfg1_decode7b", "decode_layer_kernel")] >= bench.layer_bytes(cfg1)
    cfg3 = syn.CONFIGS["cfg3_qwen32b_down_m2048"]
    r3 = bench.roofline_for(cfg3, 2, 450.0, 200.0, None, traffic)
    assert r3["bound"] == "mfma" and r3["unit"] == "TOP/s" and r3["peak"] == 5000.0
    assert abs(r3["achieved"] - 2 * 2048 * cfg3.N * cfg3.K / 200e-6 / 1e12) < 1e-9
    assert abs(r3["layer"]["achieved"] - 2 * 2048 * cfg3.N * cfg3.K / 450e-6 / 1e12) < 1e-9
    # the same rule at the crossover: bytes / 8 TB/s against ops / 5 POP/s
    for cfg in (cfg1, cfg3, syn.CONFIGS["cfg2_qwen32b_up_m16"]):
        hbm_t = bench.layer_bytes(cfg) / 8e12
        mfma_t = bench.gemm_ops(cfg) / 5e15
        assert bench.roofline_for(cfg, 2, 20.0, 10.0, None, traffic)["bound"] == ("hbm" if hbm_t >= mfma_t else "mfma")


def test_the_kernels_named_are_the_ones_that_run():
    """roofline.kernel of the prefill workloads against the table the library picks the tile from, and the kernels of the
    counter summary against the sources: a figure measured on a kernel that is gone would be printed beside a
    time of another."""
    import glob
    import re
    import tempfile
    csrc = os.path.join(ROOT, "paper_2605_00422_amd", "csrc")
    cfgs = [c for M in (64, 4096) for c in syn.block70b_configs(M)] + [syn.CONFIGS["cfg3_qwen32b_down_m2048"]]
    with tempfile.TemporaryDirectory() as tmp:
        src = "#include <cstdio>\n#include \"gemm_tiles.h\"\nint main() {\n" + "".join(
            f'printf("%d\\n", GD_TILES[gd_pick({c.M}, {c.K}, {c.N}, {c.r}, 256, {a4})].wn);\n'
            for c in cfgs for a4 in ("false", "true")) + "}\n"
        with open(os.path.join(tmp, "wn.cpp"), "w") as f:
            f.write(src)
        subprocess.run(["g++", "-std=c++17", "-I", csrc, "-o", os.path.join(tmp, "wn"), os.path.join(tmp, "wn.cpp")], check=True)
        wn = subprocess.run([os.path.join(tmp, "wn")], capture_output=True, text=True, check=True).stdout.split()
    for c, w in zip([c for c in cfgs for _ in (0, 1)], map(int, wn)):
        assert bench.gemm_kernel(c) == ("gemm_prefill_shared_kernel" if w > 1 else "gemm_prefill_direct_kernel"), c.name
    sources = "".join(open(f).read() for f in glob.glob(os.path.join(csrc, "*.h*")))
    traffic = bench.measured_traffic()
    for _, kernel in traffic:
        assert re.search(rf"__global__[^;{{]*\b{kernel}\(", sources), kernel
    for c in (syn.CONFIGS["cfg3_qwen32b_down_m2048"], next(c for c in cfgs if c.name == "cfg4_70b_gate_m4096")):
        r = bench.roofline_for(c, 2, 450.0, 200.0, None, traffic)
        assert r["traffic"] == traffic[(c.name, bench.gemm_kernel(c))] >= bench.linear_forward_bytes(c)


def test_layer_bytes_are_both_calls_bytes():
    cfg = syn.CONFIGS["cfg1_decode7b"]
    rq = 2 * 4096 + 4 * (64 * 64 + 64 * 64) + 2 * 4096 * 32 + 4096 + 8 + 4 * 32
    assert bench.rotate_quant_bytes(cfg) == rq
    assert bench.layer_bytes(cfg) == 6410888 + rq == 6718224


def test_more_than_one_gpu_is_refused_with_a_message():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert p.returncode == 2
    assert "one GPU" in p.stderr and p.stdout.strip() == ""


def test_the_kernels_named_for_narrow_codes():
    """The same with codes of at most seven bits, against the table of the GEMM on the sparse instructions."""
    import tempfile
    csrc = os.path.join(ROOT, "paper_2605_00422_amd", "csrc")
    cfgs = [c for M in (64, 4096) for c in syn.block70b_configs(M)] + [syn.CONFIGS["cfg3_qwen32b_down_m2048"]]
    with tempfile.TemporaryDirectory() as tmp:
        src = "#include <cstdio>\n#include \"gemm_tiles.h\"\nint main() {\n" + "".join(
            f'printf("%d\\n", gs_pick({c.M}, {c.K}, {c.N}, {c.r}, 256) >= 0);\n' for c in cfgs) + "}\n"
        with open(os.path.join(tmp, "gs.cpp"), "w") as f:
            f.write(src)
        subprocess.run(["g++", "-std=c++17", "-I", csrc, "-o", os.path.join(tmp, "gs"), os.path.join(tmp, "gs.cpp")], check=True)
        sparse = subprocess.run([os.path.join(tmp, "gs")], capture_output=True, text=True, check=True).stdout.split()
    for c, s in zip(cfgs, sparse):
        assert (bench.gemm_kernel(c, 6) == "gemm_sparse_kernel") == (s == "1"), c.name


def test_the_kernels_named_are_the_dispatch_s_own():
    """Beside the listed configurations too, at the widths of codes that decide: (tokens, columns, channels, rank, bits,
    nibbles), the kernel."""
    import dataclasses
    base = syn.CONFIGS["cfg3_qwen32b_down_m2048"]
    for M, K, N, r, bits, nibbles, kernel in (
            (512, 8192, 28672, 64, 6, False, "gemm_sparse_kernel"), (512, 8192, 28672, 64, 8, False, "gemm_prefill_shared_kernel"),
            (2048, 4096, 22016, 64, 6, False, "gemm_sparse_kernel"), (2048, 4096, 22016, 64, 4, True, "gemm_prefill_shared_kernel"),
            (2048, 8192, 64, 64, 6, False, "gemm_prefill_direct_kernel"), (64, 8192, 28672, 64, 6, False, "gemm_prefill_direct_kernel"),
            (2048, 4128, 4096, 64, 6, False, "gemm_prefill_kernel"), (16, 4096, 11008, 32, 6, False, "gemm_decode_bs_kernel")):
        c = dataclasses.replace(base, M=M, K=K, N=N, r=r)
        assert bench.gemm_kernel(c, bits, nibbles) == kernel, (M, K, N, r, bits, nibbles)


def test_share_of_the_peak_says_which_peak():
    """Operations of the dense product over the dense instructions' peak, for every kernel; the one on the sparse
    instructions says beside it what share of theirs that is."""
    cfg = syn.CONFIGS["cfg3_qwen32b_down_m2048"]
    r = bench.roofline_for(cfg, 4, 318.0, 175.0, None, {}, act_bits=6)
    assert r["kernel"] == "gemm_sparse_kernel" and r["peak"] == 5000.0
    assert abs(r["frac"] - bench.gemm_ops(cfg) / 175e-6 / 5e15) < 1e-9
    assert abs(r["frac_of_sparse_peak"] - r["frac"] / 2) < 1e-12
    assert "frac_of_sparse_peak" not in bench.roofline_for(cfg, 3, 318.0, 195.0, None, {}, act_bits=8)


def test_the_line_stays_short():
    """What collects the line keeps eight kilobytes of it.  A record of every workload with numbers of full length."""
    import json
    third = 1.0 / 3.0
    cfg = syn.CONFIGS["cfg3_qwen32b_down_m2048"]
    times = {"us_per_layer": 1e4 * third, "us_per_layer_min": 1e4 * third, "us_per_layer_events": 1e4 * third,
             "us_linear_forward": 1e4 * third, "us_rotate_quant": 1e4 * third}
    roof = bench.roofline_for(cfg, 4, 1e4 * third, 1e3 * third, None, {}, act_bits=6)
    roof.update(peak_measured=1e4 * third, frac_of_measured=third, traffic=10 ** 10)
    side = bench.side_kernel_report(cfg, 1e3 * third)
    extra = [{"workload": "cfg3_qwen32b_down_m2048+row_shift+asym", "M": 4096, "K": 28672, "N": 28672, "r": 64, "kron": "224x128",
              "layer_copies": 99, "launches_per_layer": 4, "stream": times, "graph": times, "roofline": roof,
              "side_kernels": [side], "effective_tops": 1e3 * third} for _ in range(18)]
    quantizer = {"workload": "Gaussian 11008 x 4096 (Kronecker 64 x 64), rank 32", "dtype": "f64", "rounds": 2, "ms_total": 1e2 * third,
                 "svd_iters_per_round": 20, "ms_per_round": 1e2 * third, "loss_history": [third] * 7,
                 "okt_rows": {"ms": third, "bound": "hbm", "bytes_moved": 1, "achieved": 1e3 * third, "peak": 8e3, "unit": "GB/s",
                              "frac": third, "flops": 1},
                 "down_projection": {"workload": "Gaussian 4096 x 11008 (Kronecker 128 x 86), rank 32", "ms_per_round": 1e2 * third,
                                     "loss_history": [third] * 7}}
    line = {"metric": "x" * 80, "value": third, "vs_baseline": None, "dtype_detail": "x" * 130, "data": "synthetic",
            "config": {k: "x" * 20 for k in "abcdefghijkl"}, "timings": {"stream": times, "graph": times}, "roofline": roof,
            "roofline_prefill": roof, "side_kernels": [side], "cpu_baseline": {"sample": "x" * 120, "value": third},
            "other_workloads": extra, "block7b_m1": {k: third for k in ("us_seven_layers", "us_four_merged_layers",
                                                                        "us_gateup_forward", "us_gateup_forward_gated")},
            "quantizer": quantizer, "microbench": {"what": "x" * 220, "a": third, "b": third, "c": third}}
    text = json.dumps(bench.short_line(line), separators=(",", ":"))
    assert len(text) < 7500
    got = json.loads(text)
    assert got["value"] == 0.33333 and len(got["other_workloads"]) == 18
    assert got["other_workloads"][0]["kernel"] == "gemm_sparse_kernel" and got["other_workloads"][0]["us"] == 3333.3
    assert len(json.dumps(line)) > 8192                     # (as it was printed)
