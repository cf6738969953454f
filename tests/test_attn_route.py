"""The rule by which a bf16 attention call chooses its kernel, on the host: both sides of each of its lines, what the benchmark
names, and what no call may reach."""
import os
import sys

import pytest

import paper_2602_01801_amd as fa

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def route(n_items, d, BQ, n_sel, ws=False, BK=64):
    return fa.attn_route(n_items, d, BQ, BK, n_sel, ws)


def test_lines_between_the_kernels_of_128_wide_heads():
    for args, want in [
        ((257, 128, 128, 1), ("one", 0)), ((256, 128, 128, 5), ("one", 0)), ((256, 128, 128, 6), ("pair_split", 1)),
        ((512, 128, 128, 2), ("one", 0)), ((512, 128, 128, 3), ("pair", 0)), ((513, 128, 128, 2), ("one", 0)),
        ((767, 128, 128, 60), ("one", 0)), ((768, 128, 128, 60), ("pair", 0)), ((1024, 128, 128, 2), ("pair", 0)),
        # a short last round is shared out with a workspace
        ((1160, 128, 128, 360), ("one", 0)), ((1160, 128, 128, 360, True), ("one_shared", 128)),
        ((1160, 128, 128, 54, True), ("one_shared", 128)), ((1160, 128, 128, 53, True), ("one", 0)),
        ((513, 128, 128, 40, True), ("one_shared", 64)), ((704, 128, 128, 360, True), ("one_shared", 64)),
        ((705, 128, 128, 360, True), ("one", 0))]:
        assert route(*args) == want, args


def test_a_call_without_fragments_takes_the_same_kernel_with_and_without_a_workspace():
    for d in (64, 128):
        for BQ in (64, 128):
            for n_items in (1, 3, 9, 12, 31, 64, 65, 100, 128, 129, 200, 256, 257, 320, 400, 512, 900, 2048, 2049):
                for n_sel in (1, 2, 3, 5, 6, 8, 9, 17, 20, 24, 33, 50, 100, 400):
                    kernel, n = route(n_items, d, BQ, n_sel, True)
                    if kernel == "one_shared" or kernel == "pair_split" and n > 1:
                        assert d == 128 and BQ == 128
                        assert kernel == "one_shared" or n_items <= 128 and n_sel > 8 and n * n_items <= 512   # what the interface says
                    else:
                        assert (kernel, n) == route(n_items, d, BQ, n_sel, False), (d, BQ, n_items, n_sel)


def test_arguments_that_no_call_takes_are_refused():
    for bad in ((0, 128, 128, 64, 1), (1, 96, 128, 64, 1), (1, 128, 32, 64, 1), (1, 128, 128, 48, 1), (1, 128, 128, 64, 0)):
        with pytest.raises(fa.FastarError):
            fa.attn_route(*bad, False)


def test_the_benchmark_names_the_kernel_of_the_rule():
    sys.path.insert(0, ROOT)
    import bench
    of = {"plain": "attn_bf16_kernel", "waves": "attn_bf16_waves_kernel", "one": "attn_bf16_d128_kernel", "one_shared": "attn_bf16_d128_sk_kernel",
          "pair": "attn_bf16_d128_pp_kernel", "pair_split": "attn_bf16_d128_pp_kernel"}
    for n_items in (1, 4, 5, 11, 12, 64, 65, 128, 129, 256, 444, 600, 1160):
        for n_tiles in (1, 2, 5, 8, 9, 24, 52, 360):
            for ws in (False, True):
                name, (kernel, n) = bench.attn_kernel_name(n_items, 12, 37440, n_tiles, ws), route(n_items, 128, 128, n_tiles, ws)
                assert name.startswith(of[kernel])
                assert kernel != "waves" or name == "attn_bf16_waves_kernel<128, %d, true>" % n
                assert ("combine_parts" in name) == (kernel == "pair_split" and n > 1)
