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


def test_lines_of_the_kernel_whose_wavefronts_share_a_group_of_queries():
    waves = lambda *a, **k: (lambda r: r[1] if r[0] == "waves" else 0)(route(*a, **k))  # noqa: E731
    # 64-wide heads, blocks of 64 queries: the shortest list by number of blocks, single keys, the longest beyond 2048 blocks
    for n_items, least in ((320, 1), (321, 3), (1024, 3), (1025, 5), (1300, 5), (1301, 8), (1536, 8), (1537, 3), (2048, 3), (2049, 4), (4096, 4)):
        assert waves(n_items, 64, 64, least) > 0 and (least == 1 or waves(n_items, 64, 64, least - 1) == 0), n_items
    assert waves(320, 64, 64, 1, BK=1) == 2 and waves(321, 64, 64, 128, BK=1) == 0 and waves(321, 64, 64, 129, BK=1) == 2
    assert (waves(2048, 64, 64, 65), waves(2049, 64, 64, 64), waves(2049, 64, 64, 65), waves(4097, 64, 64, 20)) == (4, 4, 0, 0)
    assert [waves(128, 64, 64, n) for n in (1, 2, 11, 12)] == [2, 4, 4, 8] and [waves(129, 64, 64, n) for n in (31, 32)] == [4, 8]
    assert [waves(257, 64, 64, n) for n in (1, 2, 31, 32)] == [2, 2, 2, 4]
    # of 128
    for n_items, least in ((128, 1), (129, 2), (160, 2), (161, 3), (320, 3), (321, 16), (448, 16)):
        assert waves(n_items, 64, 128, least) > 0 and (least == 1 or waves(n_items, 64, 128, least - 1) == 0), n_items
    assert waves(321, 64, 128, 16) == 4 and waves(449, 64, 128, 60) == 0
    # 128-wide heads, blocks of 64 queries: key blocks of 64 only
    for n_items, least in ((1, 2), (128, 2), (129, 8), (256, 8), (257, 3), (384, 3)):
        assert waves(n_items, 128, 64, least) > 0 and waves(n_items, 128, 64, least - 1) == 0, n_items
    assert waves(385, 128, 64, 30) == 0 and waves(10, 128, 64, 200, BK=32) == 0
    assert [waves(128, 128, 64, n) for n in (23, 24)] == [4, 8] and waves(256, 128, 64, 24) == 4 and waves(257, 128, 64, 300) == 2
    # of 128: the longest list without a workspace, and with one where the others leave fragments
    for n_items, least in ((1, 2), (64, 2), (65, 6), (128, 6)):
        assert waves(n_items, 128, 128, least) > 0 and waves(n_items, 128, 128, least - 1) == 0, n_items
    assert waves(64, 128, 128, 1000) == 8 and [waves(n, 128, 128, 32) for n in (65, 128, 129)] == [4, 4, 0] and waves(65, 128, 128, 33) == 0
    for n_items, most in ((4, 9), (12, 20), (28, 28), (36, 32), (64, 32), (65, 20)):
        assert waves(n_items, 128, 128, most, True) > 0 and waves(n_items, 128, 128, most + 1, True) == 0, n_items
        assert route(n_items, 128, 128, most + 1, True)[1] > 1      # fragments


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
