"""GPU parity of the 8-bit floating-point K/V path: fastar_kv_to_fp8 bit for bit, sparse_attn_fwd_fp8 within a
tolerance, both against the CPU oracle on the same seeded inputs, through the C ABI.

Tolerance of the attention (derived, then written here): keys, values and queries are the same E4M3 values on both
sides and the scores are accumulated in fp32 from exact products, so what differs is the rounding of the softmax weights
to E4M3 (3 mantissa bits: relative error up to 2^-4 per weight, also in the row sum the kernel divides by) and of the
output to bf16.  An output is a convex combination of values; perturbing the weights by a relative eps moves it by at
most 2 eps times the spread of the contributing values around it.  With eps = 2^-4 and spreads of about 1 (values
N(0, 1.2)) the bound is about 0.13, the typical error (independent roundings over tens of keys) a few hundredths:
max-abs <= 0.1, and mean-abs <= 0.01 so that a systematic error cannot hide under the bound.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01801_amd as fa
from workloads import CONFIGS, FrameStream, make_codec, to_f32, to_storage

from gpu_util import dev_cache, dev_codec, storage_to_f64, to_dev, to_host

pytestmark = pytest.mark.gpu

ATOL_MAX, ATOL_MEAN = 0.1, 0.01


def rand_cache(rng, H, C, d, lens, dtype):
    c = oracle.Cache.empty(H, C, d, 32, dtype)
    c.K[:] = to_storage((rng.standard_normal((H, C, d)) * 1.2).astype(np.float32), dtype)
    c.V[:] = to_storage((rng.standard_normal((H, C, d)) * 1.2).astype(np.float32), dtype)
    c.cnt[:] = rng.integers(1, 6, size=(H, C))
    c.stamp[:] = rng.integers(0, 5, size=(H, C))
    c.len[:] = lens
    return c


@pytest.mark.parametrize("dtype,C,lens", [("bf16", 640, [640, 333, 1]), ("fp32", 200, [200, 130, 0]),
                                          ("bf16", 64 * 50 + 17, [3217, 3000, 64])])
def test_kv_to_fp8_bit_exact_and_incremental(dtype, C, lens):
    rng = np.random.default_rng(C)
    H, d = 3, 128
    c = rand_cache(rng, H, C, d, lens, dtype)
    # awkward values: beyond the format's range, subnormal, exact ties between neighbouring codes, signed zeros
    special = np.array([500.0, -1e6, 448.0, 2.0 ** -10, 3 * 2.0 ** -10, 1.0625, 1.1875, -0.0, 0.0, 2.0 ** -12, 0.0146], np.float32)
    if lens[0] > 4:
        c.K[0, 0, :special.size] = to_storage(special, dtype)
        c.V[0, 1, :special.size] = to_storage(-special, dtype)
    for h in range(H):                                    # dead slots are never read: poison them
        c.K[h, lens[h]:] = to_storage(np.full((C - lens[h], d), np.nan, np.float32), dtype)
        c.V[h, lens[h]:] = to_storage(np.full((C - lens[h], d), np.nan, np.float32), dtype)
    K8r, V8r = oracle.kv8_empty(H, C, d)
    K8r[:], V8r[:] = 0x11, 0x11
    K8, V8 = to_dev(K8r), to_dev(V8r)
    gpu = dev_cache(c)
    oracle.kv_to_fp8(c, K8r, V8r)
    fa.kv_to_fp8(gpu, K8, V8)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(K8), K8r) and np.array_equal(to_host(V8), V8r)
    # a later frame rewrites a few slots: only their blocks change
    c.stamp[:, : min(lens)] = np.where(rng.random((H, min(lens))) < 0.02, 7, c.stamp[:, : min(lens)])
    c.K[:, : min(lens)] = to_storage((rng.standard_normal((H, min(lens), d))).astype(np.float32), dtype)
    gpu = dev_cache(c)
    oracle.kv_to_fp8(c, K8r, V8r, stamp_lo=7)
    fa.kv_to_fp8(gpu, K8, V8, stamp_lo=7)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(K8), K8r) and np.array_equal(to_host(V8), V8r)


def check_fp8_attention(Q, c, sel, nsel, scale, use_cnt=True):
    H, C, d = c.K.shape
    K8r, V8r = oracle.kv8_empty(H, C, d)
    oracle.kv_to_fp8(c, K8r, V8r)
    K8, V8 = fa.kv8_empty(H, C, d)
    fa.kv_to_fp8(dev_cache(c), K8, V8)
    cnt = c.cnt if use_cnt else None
    O, lse = fa.sparse_attn_fwd_fp8(to_dev(Q), K8, V8, None if cnt is None else to_dev(cnt), to_dev(c.len), C,
                                    to_dev(sel), to_dev(nsel), 128, 64, scale)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(K8), K8r) and np.array_equal(to_host(V8), V8r)
    O_r, lse_r = oracle.sparse_attn_fwd_fp8(Q, K8r, V8r, cnt, c.len, C, sel, nsel, 128, 64, scale)
    got = storage_to_f64(to_host(O))
    assert np.isfinite(got).all()
    err = np.abs(got - O_r)
    assert err.max() <= ATOL_MAX, f"max |O - O_ref| = {err.max()}"
    assert err.mean() <= ATOL_MEAN, f"mean |O - O_ref| = {err.mean()}"
    lg = to_host(lse).astype(np.float64)
    empty = np.isneginf(lse_r)
    assert np.array_equal(np.isneginf(lg), empty)
    assert np.abs(lg[~empty] - lse_r[~empty]).max() <= 0.05
    return err.max(), err.mean()


@pytest.mark.parametrize("n_blk,cut", [(1, 0), (15, 3), (16, 0), (17, 63), (33, 1), (50, 0)])
def test_kv_to_fp8_finds_the_blocks_a_frame_wrote(n_blk, cut):
    # a workgroup per block: a run of written slots, single ones, none
    rng = np.random.default_rng(n_blk)
    H, d, C = 3, 128, 64 * n_blk - cut
    c = rand_cache(rng, H, C, d, [C, max(1, C - 70), C], "bf16")
    c.stamp[:] = 3
    c.stamp[0, C // 3: C // 3 + 200] = 7
    c.stamp[0, C - 1] = c.stamp[1, 0] = 7
    c.stamp[1, C - 1] = 7                      # beyond the head's length: not looked at (C > 70)
    K8r, V8r = oracle.kv8_empty(H, C, d)
    K8r[:], V8r[:] = 0x22, 0x33
    K8, V8 = to_dev(K8r), to_dev(V8r)
    oracle.kv_to_fp8(c, K8r, V8r, stamp_lo=7)
    fa.kv_to_fp8(dev_cache(c), K8, V8, stamp_lo=7)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(K8), K8r) and np.array_equal(to_host(V8), V8r)
    assert (K8r[2] == 0x22).all()              # a head in which nothing was written stays as it is


@pytest.mark.parametrize("H,n_blk,cut", [(3, 10923, 0), (3, 10925, 63), (3, 21847, 5), (4, 32771, 1)])
def test_kv_to_fp8_of_long_caches_finds_the_blocks_a_frame_wrote(H, n_blk, cut):
    # two, four and eight blocks per workgroup, a grid apart, from 32768, 65536 and 131072 blocks on (and one just below),
    # against a rebuild, which takes a workgroup per block at any size
    g = torch.Generator(device="cuda").manual_seed(n_blk)
    d, C = 128, 64 * n_blk - cut
    normal = lambda: torch.randn((H, C, d), generator=g, device="cuda", dtype=torch.bfloat16)
    cache = fa.Cache.empty(H, C, d, 32, torch.bfloat16)
    cache.K[:], cache.V[:] = normal(), normal()
    cache.stamp.fill_(3)
    cache.len.fill_(C)
    cache.len[1] = C - 200
    cache.stamp[0, C // 3: C // 3 + 5000] = 7
    cache.stamp[:, -1] = 7                                    # beyond the second head's length
    cache.stamp.view(-1)[torch.randint(0, H * C, (n_blk // 3,), generator=g, device="cuda")] = 7
    whole = [torch.full_like(t, 0x55) for t in fa.kv8_empty(H, C, d)]
    fa.kv_to_fp8(cache, *whole)
    part = [torch.full_like(t, 0x55) for t in whole]
    fa.kv_to_fp8(cache, *part, stamp_lo=7)
    torch.cuda.synchronize()
    live = torch.arange(C, device="cuda")[None, :] < cache.len[:, None]
    written = torch.zeros((H, 64 * n_blk), dtype=torch.bool, device="cuda")
    written[:, :C] = (cache.stamp >= 7) & live
    dirty = written.view(H, n_blk, 64).any(2)
    assert 0 < int(dirty.sum()) < H * n_blk // 2
    for got, want in zip(part, whole):
        got, want = got.view(H, n_blk, -1), want.view(H, n_blk, -1)
        assert (got[~dirty] == 0x55).all() and torch.equal(got[dirty], want[dirty])


@pytest.mark.parametrize("H,n_q,C,lens,n_sel,seed", [
    (2, 256, 1280, [1280, 546], 5, 0),            # ragged last block, cfg1-like sizes at d = 128
    (3, 300, 64 * 40, [2560, 2000, 0], 9, 1),     # ragged queries, an empty head
    (2, 4680, 64 * 100 + 5, [6405, 6300], 30, 2), # many tiles, capacity that is no multiple of the block
    (1, 130, 640, [640], 10, 3),                  # every block selected
])
def test_fp8_attention_matches_the_oracle(H, n_q, C, lens, n_sel, seed):
    rng = np.random.default_rng(seed)
    d = 128
    c = rand_cache(rng, H, C, d, lens, "bf16")
    for h in range(H):
        c.K[h, lens[h]:] = to_storage(np.full((C - lens[h], d), np.nan, np.float32), "bf16")   # dead slots: poison
        c.V[h, lens[h]:] = to_storage(np.full((C - lens[h], d), np.nan, np.float32), "bf16")
    Q = to_storage((rng.standard_normal((H, n_q, d)) * 1.1).astype(np.float32), "bf16")
    n_qb = (n_q + 127) // 128
    n_kb = (C + 63) // 64
    sel = np.full((H, n_qb, n_sel), -1, np.int32)
    nsel = np.zeros((H, n_qb), np.int32)
    for h in range(H):
        for b in range(n_qb):
            m = int(rng.integers(max(1, n_sel // 2), n_sel + 1))
            row = np.sort(rng.choice(n_kb, size=min(m, n_kb), replace=False)).astype(np.int32)
            if rng.random() < 0.4 and row.size > 2:
                row[rng.integers(0, row.size)] = -1                     # padding inside the list
            sel[h, b, :row.size] = row
            nsel[h, b] = row.size
    check_fp8_attention(Q, c, sel, nsel, d ** -0.5)
    check_fp8_attention(Q, c, sel, nsel, d ** -0.5, use_cnt=False)


@pytest.mark.parametrize("counts", [(1, 2, 3), (4, 5, 7), (255, 256, 257, 258, 259), (511, 512, 515, 600)])
def test_fp8_attention_at_the_edges_of_its_pipeline(counts):
    # lists that end while the first tiles are being asked for, and around the pieces (256 entries) in which a list goes
    # through LDS; entries of -1 at the pieces' edges, the last block short
    rng = np.random.default_rng(counts[0])
    H, d, n_kb = 1, 128, 640
    C = 64 * n_kb - 7
    c = rand_cache(rng, H, C, d, [C], "bf16")
    n_qb, n_sel = len(counts), max(counts)
    Q = to_storage((rng.standard_normal((H, 128 * n_qb - 5, d)) * 1.1).astype(np.float32), "bf16")
    sel = np.full((H, n_qb, n_sel), -1, np.int32)
    for b, m in enumerate(counts):
        sel[0, b, :m] = np.sort(rng.choice(n_kb - 1, size=m, replace=False))
        sel[0, b, m - 1] = n_kb - 1
        for edge in (0, 255, 256, 511, 512):
            if m > 3 and edge < m - 1 and (b + edge) % 2:
                sel[0, b, edge] = -1
    nsel = np.array([counts], np.int32)
    check_fp8_attention(Q, c, sel, nsel, d ** -0.5)
    check_fp8_attention(Q, c, sel, nsel, d ** -0.5, use_cnt=False)


# pairs per XCD range, of which whole rounds of 96 or 64 workgroups are taken whole: sizes at the edges of the rule
@pytest.mark.parametrize("H,n_qb,n_sel,split", [
    (33, 16, 180, False),                          # 66 per range: one round
    (23, 24, 150, True), (23, 24, 149, False),     # 69 (64 whole)
    (26, 30, 120, True), (26, 30, 119, False),     # 98 (96 whole)
    (24, 44, 150, True),                           # 132 (96 whole)
    (31, 35, 150, True)])                          # 136 (96 whole; the last range is short)
def test_fp8_attention_split_by_the_workgroups_a_unit_holds(H, n_qb, n_sel, split):
    d, C, n_q = 128, 64 * 300 - 9, 128 * n_qb - 40
    g = torch.Generator(device="cuda").manual_seed(H + n_sel)
    normal = lambda n: torch.randn((H, n, d), device="cuda", generator=g).bfloat16()  # noqa: E731
    cache = fa.Cache.empty(H, C, d, 32, torch.bfloat16)
    cache.K[:], cache.V[:] = normal(C), normal(C)
    cache.stamp.zero_()
    cache.cnt[:] = torch.randint(1, 6, (H, C), device="cuda", generator=g, dtype=torch.int32)
    cache.len.fill_(C)
    cache.len[2] = C // 2
    K8, V8 = fa.kv8_empty(H, C, d)
    fa.kv_to_fp8(cache, K8, V8)
    sel = torch.rand((H, n_qb, 300), device="cuda", generator=g).topk(n_sel, dim=2).indices.sort(dim=2).values.to(torch.int32).contiguous()
    nsel = torch.full((H, n_qb), n_sel, dtype=torch.int32, device="cuda")
    nsel[1, 3], nsel[H - 1, n_qb - 1] = 7, 0
    ws = torch.full((fa.workspace_bytes(fa.OP_ATTN, H, n_q, C),), 0x5A, dtype=torch.uint8, device="cuda")
    args = (normal(n_q), K8, V8, cache.cnt, cache.len, C, sel, nsel, 128, 64, d ** -0.5)
    O, lse = fa.sparse_attn_fwd_fp8(*args, ws=ws)
    O_plain, lse_plain = fa.sparse_attn_fwd_fp8(*args)
    torch.cuda.synchronize()
    assert bool((ws != 0x5A).any()) == split           # fragments, or untouched
    diff = (O.float() - O_plain.float()).abs()
    # a fragment rounds its weights against its own reference maximum; without fragments it is the same launch
    assert torch.isfinite(O.float()).all() and diff.max() <= (ATOL_MAX if split else 0) and diff.mean() <= (ATOL_MEAN if split else 0)
    fin = torch.isfinite(lse_plain)
    assert torch.equal(fin, torch.isfinite(lse)) and (lse[fin] - lse_plain[fin]).abs().max() <= 0.05


@pytest.mark.parametrize("H,n_q,C,n_sel", [
    (20, 3600, 64 * 300, 150),     # 580 query blocks: 73 per XCD range, 9 of them left over by the whole round
    (33, 2048, 64 * 256, 128),     # 528 blocks: 2 per range left over
])
def test_fp8_attention_with_a_workspace_splits_the_launch_and_matches_the_plain_one_and_the_oracle(H, n_q, C, n_sel):
    # sparse_attn_fwd_fp8_ws: the query blocks that whole rounds of workgroups leave over are cut into equal shares of
    # their tiles and combined from fragments.  Against the plain launch everywhere, against the oracle on sampled
    # (head, query block) pairs: whole ones, cut ones, a short and an empty list, a head that is not full.
    rng = np.random.default_rng(H + n_sel)
    d = 128
    g = torch.Generator(device="cuda").manual_seed(H * 7 + n_sel)
    Q = (torch.randn(H, n_q, d, device="cuda", generator=g) * 1.1).bfloat16()
    K = torch.randn(H, C, d, device="cuda", generator=g).bfloat16()
    V = torch.randn(H, C, d, device="cuda", generator=g).bfloat16()
    cnt = torch.randint(1, 6, (H, C), device="cuda", generator=g, dtype=torch.int32)
    lens = np.full(H, C, np.int32)
    lens[3] = C // 2 + 17
    gpu = fa.Cache.empty(H, C, d, 32, torch.bfloat16)
    gpu.K.copy_(K); gpu.V.copy_(V); gpu.cnt.copy_(cnt); gpu.stamp.zero_(); gpu.len.copy_(to_dev(lens))
    K8, V8 = fa.kv8_empty(H, C, d)
    fa.kv_to_fp8(gpu, K8, V8)
    n_qb, n_kb = -(-n_q // 128), C // 64
    sel = np.stack([np.stack([np.sort(rng.choice(n_kb, n_sel, replace=False)) for _ in range(n_qb)]) for _ in range(H)]).astype(np.int32)
    nsel = np.full((H, n_qb), n_sel, np.int32)
    total = n_qb * H
    per = -(-total // 8)
    tail_per = per % 64
    assert per > 64 and 0 < tail_per <= 24, "the shape is meant to take the split launch"
    to_item = lambda vi: (vi // tail_per) * per + (per - tail_per) + vi % tail_per
    W = 8 * tail_per * n_sel
    cut = sorted({to_item((i * W // 512) // n_sel) for i in range(1, 512) if (i * W // 512) % n_sel} - set(range(total, 8 * per)))
    short_item, empty_item = cut[1], to_item(1) if to_item(1) not in cut[:3] else to_item(2)
    nsel.reshape(-1)[short_item] = n_sel // 3
    sel.reshape(total, n_sel)[short_item, n_sel // 3:] = -1
    nsel.reshape(-1)[empty_item] = 0
    sel.reshape(total, n_sel)[empty_item, :] = -1
    ws = torch.empty(fa.workspace_bytes(fa.OP_ATTN, H, n_q, C), dtype=torch.uint8, device="cuda")
    args = (Q, K8, V8, cnt, to_dev(lens), C, to_dev(sel), to_dev(nsel), 128, 64, d ** -0.5)
    O_ws, lse_ws = fa.sparse_attn_fwd_fp8(*args, ws=ws)
    O_pl, lse_pl = fa.sparse_attn_fwd_fp8(*args)
    torch.cuda.synchronize()
    a, b = storage_to_f64(to_host(O_ws)), storage_to_f64(to_host(O_pl))
    # a fragment rounds its weights to E4M3 against its own reference maximum: the two launches differ like either does from the oracle
    assert np.isfinite(a).all() and np.abs(a - b).max() <= ATOL_MAX and np.abs(a - b).mean() <= ATOL_MEAN
    lw, lp = to_host(lse_ws).astype(np.float64), to_host(lse_pl).astype(np.float64)
    fin = np.isfinite(lp)
    assert np.array_equal(fin, np.isfinite(lw)) and np.abs(lw[fin] - lp[fin]).max() <= 0.05
    Kc, Vc = to_host(K8), to_host(V8)
    sample = sorted(set([0, n_qb - 1, total - 1, short_item, empty_item, 3 * n_qb] + cut[:2] + cut[-1:]))
    for item in sample:
        h, bq = divmod(item, n_qb)
        q0, q1 = bq * 128, min((bq + 1) * 128, n_q)
        O_r, lse_r = oracle.sparse_attn_fwd_fp8(to_host(Q[h:h + 1, q0:q1]), Kc[h:h + 1], Vc[h:h + 1], to_host(cnt[h:h + 1]),
                                                lens[h:h + 1], C, sel[h:h + 1, bq:bq + 1], nsel[h:h + 1, bq:bq + 1], 128, 64,
                                                d ** -0.5)
        err = np.abs(a[h, q0:q1] - O_r[0])
        assert err.max() <= ATOL_MAX and err.mean() <= ATOL_MEAN, f"item {item}: {err.max()} {err.mean()}"
        ok = np.isfinite(lse_r[0])
        assert np.array_equal(ok, np.isfinite(lw[h, q0:q1])) and np.abs(lw[h, q0:q1][ok] - lse_r[0][ok]).max(initial=0.0) <= 0.05


@pytest.mark.parametrize("scale", [1e-45, 1e-39, 1e-38, 5.4e-31, 5.6e-31])
def test_fp8_attention_with_scales_down_to_the_smallest(scale):
    rng = np.random.default_rng(21)
    c = rand_cache(rng, 2, 64 * 20 + 9, 128, [64 * 20 + 9, 700], "bf16")
    Q = to_storage(rng.standard_normal((2, 200, 128)).astype(np.float32), "bf16")
    sel = np.tile(np.arange(0, 20, 2, dtype=np.int32), (2, 2, 1))
    nsel = np.full((2, 2), 10, np.int32)
    for use_cnt in (True, False):
        check_fp8_attention(Q, c, sel, nsel, scale, use_cnt)


def test_fp8_attention_with_steadily_climbing_logits_and_a_dominant_key():
    # the reference maximum is updated lazily: scores that climb along the key list, and one key that dominates a row
    rng = np.random.default_rng(9)
    H, n_q, C, d = 1, 128, 64 * 24, 128
    c = rand_cache(rng, H, C, d, [C], "bf16")
    k = to_f32(c.K)
    ramp = np.linspace(0.2, 3.0, C)[None, :, None].astype(np.float32)
    qdir = rng.standard_normal(d).astype(np.float32)
    qdir /= np.linalg.norm(qdir)
    k = k * 0.3 + ramp * qdir[None, None, :] * 3.0
    c.K[:] = to_storage(k, "bf16")
    Q = to_storage((qdir[None, None, :] * 6.0 + 0.1 * rng.standard_normal((H, n_q, d))).astype(np.float32), "bf16")
    sel = np.arange(24, dtype=np.int32)[None, None, :].repeat(H, 0)
    nsel = np.full((H, 1), 24, np.int32)
    check_fp8_attention(Q, c, sel, nsel, d ** -0.5)


def test_fp8_attention_on_a_tempcache_rollout_cfg2_heads():
    # the Wan-shaped layer on two heads: cache built by the oracle's TempCache, selection by the oracle's AnnSA
    c = dict(CONFIGS["cfg2"])
    H, T, d, r = 2, c["T"], c["d"], c["r"]
    fs = FrameStream(c["seed"], c["cfg_id"], H, d, T, c["n_c"], c["p"], c["sigma_d"], "bf16")
    codec = make_codec(c["seed"], c["cfg_id"], d, r)
    cache = oracle.Cache.empty(H, 6 * T, d, r, "bf16")
    prev = None
    for f in range(6):
        K, V = fs.next_frame()
        prev, _, _ = oracle.tempcache_compress(cache, codec.R, codec.qscale, codec.shift, K, V, cand=prev,
                                               tau2_q16=int(round(0.98 ** 2 * 65536)), frame_id=f)
    Q = fs.queries(1)
    qc = oracle.encode(Q, codec.R, codec.qscale, codec.shift)
    sel, nsel = oracle.ann_select_self(qc, cache.code, cache.len, 128, 4, 64, 12)
    emax, emean = check_fp8_attention(Q, cache, sel, nsel, d ** -0.5)
    # and the 8-bit result stays close to the attention on the bf16 cache itself
    O16, _ = oracle.sparse_attn_fwd(Q, cache.K, cache.V, cache.cnt, cache.len, sel, nsel, 128, 64, d ** -0.5)
    K8r, V8r = oracle.kv8_empty(H, 6 * T, d)
    oracle.kv_to_fp8(cache, K8r, V8r)
    O8, _ = oracle.sparse_attn_fwd_fp8(Q, K8r, V8r, cache.cnt, cache.len, 6 * T, sel, nsel, 128, 64, d ** -0.5)
    assert np.abs(O8 - O16).mean() < 0.05


def test_fp8_entry_points_reject_unsupported_shapes():
    L = fa.lib()
    Q = torch.zeros((1, 128, 128), dtype=torch.bfloat16, device="cuda")
    K8, V8 = fa.kv8_empty(1, 128)
    ln = torch.tensor([128], dtype=torch.int32, device="cuda")
    sel = torch.zeros((1, 1, 2), dtype=torch.int32, device="cuda")
    ns = torch.ones((1, 1), dtype=torch.int32, device="cuda")
    O = torch.empty_like(Q)
    args = lambda d, BQ, BK: (Q.data_ptr(), 128, K8.data_ptr(), V8.data_ptr(), None, ln.data_ptr(), 1, 128, d,
                              sel.data_ptr(), ns.data_ptr(), BQ, BK, 2, 0.1, O.data_ptr(), None, None)
    assert L.sparse_attn_fwd_fp8(*args(64, 128, 64)) == -2
    assert L.sparse_attn_fwd_fp8(*args(128, 64, 64)) == -2
    assert L.sparse_attn_fwd_fp8(*args(128, 128, 32)) == -2
    assert L.sparse_attn_fwd_fp8(*args(128, 128, 64)) == 0
    torch.cuda.synchronize()
