"""Host-side checks of bench.py that need no GPU: the one-GPU rule, the kernel the roofline is quoted on, and the
traffic figure read from profiles/."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert p.returncode != 0
    assert "one GPU" in (p.stdout + p.stderr)
    assert '"metric"' not in p.stdout                       # no result line


def test_roofline_kernel_name_follows_the_dispatch_rule():
    sys.path.insert(0, ROOT)
    import bench
    name = bench.attn_kernel_name
    # cfg2: 37 query blocks x 12 heads fit one round of two-block workgroups; 12 x 37440 slots of K and V = 230 MB
    assert name(37 * 12, 12, 37440, 52, True) == "attn_bf16_d128_pp_kernel<4, true, true, false>"
    assert name(37 * 12, 12, 196608, 52, False) == "attn_bf16_d128_pp_kernel<4, true, false, false>"
    # cfg5: 29 x 40 = 1160 = 2 rounds of 512 + 136 (< 256): one block per workgroup, split with a workspace
    assert name(29 * 40, 40, 230400, 360, False) == "attn_bf16_d128_kernel<4>"
    assert name(29 * 40, 40, 230400, 360, True).startswith("attn_bf16_d128_sk_kernel")
    assert name(29 * 40, 40, 230400, 360, True, fp8=True).startswith("attn_fp8_d128_sk_kernel")
    assert name(1024, 40, 230400, 360, False) == "attn_bf16_d128_pp_kernel<4, true, false, false>"
    assert name(1024 + 256, 8, 1000, 10, False).startswith("attn_bf16_d128_pp_kernel")
    # at most 256 pairs: a block per workgroup; short lists: the one-block kernel
    assert name(13 * 12, 12, 32760, 52, False) == "attn_bf16_d128_pp_kernel<4, true, true, true>"
    assert name(128, 8, 32760, 52, True).startswith("attn_bf16_d128_pp_kernel<4, true, true, true> (+ attn_combine_parts")
    assert name(129, 8, 32760, 52, True) == "attn_bf16_d128_pp_kernel<4, true, true, true>"
    assert name(256, 8, 32760, 5, True) == name(444, 12, 32760, 2, True) == "attn_bf16_d128_kernel<4>"
    assert name(444, 12, 32760, 5, True) == "attn_bf16_d128_pp_kernel<4, true, true, false>"
    # the same rules as the launchers' sources state them, and the instantiations that are named
    src = lambda f: open(os.path.join(ROOT, "paper_2602_01801_amd", "csrc", f)).read()  # noqa: E731
    order = [src("attention.hip").index(rule) for rule in (
        "if (ws && d == 128 && BQ == 128 && full_per > 0)",
        "n_items <= 256 && n_tiles > 5)",
        "n_items <= 512 && n_tiles <= 5 && (n_items <= 256 || n_tiles <= 2))",
        "(n_items <= 512 || n_items % 512 == 0 || n_items % 512 >= 256))")]
    assert order == sorted(order)
    assert "tail_per <= 24 && (float)n_tiles * (1.2f - 0.0375f * (float)tail_per) > 30.0f" in src("common.hpp")
    assert "ws && n_qb * H <= 256 ? attn_parts(" in src("attention_fp8.hip")
    assert "((tail96 <= 24 && n_tiles >= 120) || (tail96 <= 40 && n_tiles >= 150))" in src("attention_fp8.hip")
    assert "tail64 >= 5 && tail64 <= 24 && n_tiles >= 150" in src("attention_fp8.hip")
    # 8-bit, by pairs per XCD: one round of 96 is left alone or filled up from 64, a short second one is shared out
    split = lambda per, tiles: name(8 * per, 40, 230400, tiles, True, fp8=True).startswith("attn_fp8_d128_sk_kernel")  # noqa: E731
    assert [split(66, 360), split(70, 180), split(70, 149), split(93, 360), split(98, 120), split(98, 119)] == [False, True, False, False, True, False]
    assert [split(132, 150), split(132, 149), split(145, 360), split(160, 360)] == [True, False, True, False]
    assert "(size_t)H * (size_t)C * D * 2 * 2 <= ((size_t)256 << 20)" in src("attention_d128_pp.hip")
    assert "template <int NWG, bool CONTIG, bool BIAS_X, bool SPLIT>" in src("attention_d128_pp.hip")


def test_traffic_figure_is_read_from_the_committed_profile():
    sys.path.insert(0, ROOT)
    import bench
    t, src = bench.profiled_traffic("cfg2")
    assert t is not None and 50e6 < t < 400e6               # fetch + write of one self-attention launch at cfg2
    assert src == "profiles/cfg2_chunk_step_hbm_traffic.txt"
    t5, src5 = bench.profiled_traffic("cfg5full")
    assert t5 is not None and 5e9 < t5 < 14e9             # the world-model launch gathers 13.7 GB, most of it from HBM
    assert src5 == "profiles/cfg5full_chunk_step_hbm_traffic.txt"
    t8, src8 = bench.profiled_traffic("cfg5full_fp8")
    assert t8 is not None and 2e9 < t8 < 7e9              # half the bytes per row
    assert src8 == "profiles/cfg5full_fp8_hbm_traffic.txt"
    # a workload without a committed counter summary reports no traffic rather than another workload's
    assert bench.profiled_traffic("cfg5") == bench.profiled_traffic("cfg2_fp8") == (None, None)


def test_gathered_bytes_count_rows_of_the_cache_that_is_attended():
    import types
    import torch
    sys.path.insert(0, ROOT)
    import bench
    cls = next(c for c in vars(bench).values() if isinstance(c, type) and hasattr(c, "gathered_bytes"))
    cache = types.SimpleNamespace(K=torch.zeros(1, dtype=torch.bfloat16), len=torch.tensor([130], dtype=torch.int32))
    sel = (torch.tensor([[[0, 2, -1]]], dtype=torch.int32), torch.tensor([[2]], dtype=torch.int32))
    layer = dict(t=torch, sel=sel, cache=cache, BK=64, n_sel=3, H=1, n_q=100, d=128)
    q_and_o = 2 * 100 * 128 * 2
    for kv8, es in ((None, 2), ((None, None), 1)):
        got = cls.gathered_bytes(types.SimpleNamespace(kv8=kv8, **layer))
        assert got == (64 + 2) * 128 * es * 2 + q_and_o
