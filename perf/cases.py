"""What a user of the library has it do, as measurable cases.

The unit of work is one *chunk* of a generated video at one attention layer, through the public entry points: merge the
chunk's frames into the bounded cache (tempcache_compress), encode the queries, select key blocks, attend to them, and
attend to the selected prompt tokens.  Cases differ in the layer's size, the data type, the state of the cache and the
options of the calls; two of them are parts that programs also run alone (the start of a rollout, and the attention
over a long prompt).

Inputs follow the structure the method is made for: keys and queries in per-head clusters laid out in raster runs, a
fraction of a frame's tokens repeating the previous frame up to a small drift, the others drawn anew; prompts of which a
few clusters lie next to query clusters.  Everything is drawn on the GPU from the seed.

A rollout goes on for as long as it is asked to: the frames a state holds are visited forwards and backwards in turn,
so that consecutive frames are always neighbours in time and repeat each other in the same proportion.  The cache is
full from the start (the steady state of a long rollout, in which every frame evicts), except at a rollout's start.
"""
import math

import numpy as np
import torch

import paper_2602_01801_amd as fa

SIGMA_W = 0.3       # standard deviation inside a cluster
QRANGE = 4.5        # |x| that the 8-bit quantiser maps to 127
SHIFT = 4           # requantisation shift of the codes
TAU2 = int(round(0.98 ** 2 * 65536))   # merge threshold: cosine 0.98
BK = 64             # keys per key block
N_REP = 4           # summaries per query block
HASH_BITS = 128     # sign codes
N_BUCKETS = 2       # prompt tokens a key or query belongs to
RING = 6            # chunks of different frames and queries a state holds

DEFAULTS = dict(path="step", dtype="bf16", d=128, r=32, BQ=128, kv="cache", ann="int8", rep="last", match="previous",
                keep=0.10, n_p=512, n_sel_p=64, repeat=0.8, drift=0.02, clusters=64)


def _case(**over):
    return dict(DEFAULTS, **over)


def listed():
    return [
        # the smallest layer, fp32: the configuration that results are checked on; launches and host time are all of it
        _case(name="tiny_f32", H=2, d=64, T=256, frames=1, cap=4, dtype="f32", BQ=128, keep=0.25, n_p=64, n_sel_p=16,
              repeat=0.7, clusters=16),
        # a small layer with 64-wide heads, sizes that fit no tile, two frames a chunk
        _case(name="small_d64", H=3, d=64, T=390, frames=2, cap=9, BQ=64, keep=0.2, n_p=77, n_sel_p=20, clusters=30),
        # fp32 at an ordinary size: a user who does without bf16
        _case(name="mid_f32", H=4, T=780, frames=1, cap=12, dtype="f32", n_p=200, n_sel_p=48),
        # the Wan-1.3B-shaped layer in its steady state: the ordinary step
        _case(name="wan", H=12, T=1560, frames=3, cap=24),
        # the first chunk of a rollout at that layer: empty cache, whole-cache match for the first frame
        _case(name="wan_start", path="start", H=12, T=1560, frames=3, cap=24, keep=0.3),
        # that layer matching every live slot of the cache and keeping mean keys
        _case(name="wan_match_all", H=12, T=1560, frames=1, cap=21, match="all", rep="mean"),
        # that layer selecting by sign codes (hashes of the whole cache are computed for the chunk, the cache keeps none)
        _case(name="wan_lsh", H=12, T=1560, frames=3, cap=24, ann="lsh"),
        # that layer selecting by prompt-induced buckets, sink and local blocks forced
        _case(name="wan_buckets", H=12, T=1560, frames=3, cap=24, ann="buckets"),
        # attention over a long prompt alone
        _case(name="prompt_long", path="prompt", H=12, T=1560, frames=3, cap=1, n_p=2048),
        # nothing divides anything: odd heads, frame, capacity and budget, prompt budget beyond the fused launch
        _case(name="ragged", H=7, T=2011, frames=2, cap=17, keep=0.15, n_p=333, n_sel_p=90, clusters=71),
        # the world-model layer on its full cache: the largest step
        _case(name="world", H=40, T=3600, frames=1, cap=64, repeat=0.9, drift=0.01, clusters=128),
        # the same over the 8-bit copy of the cache
        _case(name="world_fp8", H=40, T=3600, frames=1, cap=64, kv="fp8", repeat=0.9, drift=0.01, clusters=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# fp32 and match = "all" are used at small and ordinary layers only; the limits keep every drawn case below the largest listed
_MOST_PAIRS = {"bf16": 40 * 3600 * 23040, "f32": 12 * 3 * 1560 * 3744}


def draw(rng):
    while True:
        kind = rng.choices(["plain", "d64", "f32", "fp8", "lsh", "buckets", "start", "prompt", "all"],
                           [32, 10, 11, 12, 8, 8, 7, 6, 6])[0]
        c = _case(H=_log(rng, 1, 40), T=_log(rng, 96, 3600), frames=rng.choice([1, 1, 2, 3]), cap=_log(rng, 4, 64))
        c["keep"] = round(rng.choice([0.05, 0.1, 0.1, 0.15, 0.25]), 2)
        c["n_p"] = _log(rng, 48, 2048)
        c["n_sel_p"] = max(8, min(c["n_p"] // 4, rng.choice([32, 64, 64, 96])))
        c["repeat"] = rng.choice([0.6, 0.8, 0.9])
        c["clusters"] = max(4, min(128, c["T"] // 24))
        if kind != "start":
            c["rep"] = rng.choices(["last", "mean", "medoid"], [8, 1, 1])[0]
        if kind == "d64":
            c["d"], c["BQ"] = 64, rng.choice([64, 128])
        elif kind == "f32":
            c["dtype"], c["d"] = "f32", rng.choice([64, 128])
        elif kind == "fp8":
            c["kv"] = "fp8"
        elif kind in ("lsh", "buckets"):
            c["ann"] = kind
        elif kind in ("start", "prompt"):
            c["path"] = kind
            if kind == "start":
                c["cap"] = max(c["cap"], c["frames"])
            else:
                c["cap"] = 1
        elif kind == "all":
            c["match"] = "all"
        elif rng.random() < 0.15:
            c["r"] = 64
        n_q, C = c["frames"] * c["T"], c["cap"] * c["T"]
        pairs = c["H"] * n_q * min(C, _n_sel(c) * BK)
        whole = c["H"] * C
        if pairs > _MOST_PAIRS[c["dtype"]] or c["H"] * C > 40 * 230400 or -(-n_q // c["BQ"]) > 200:
            continue
        if c["match"] == "all" and c["H"] * n_q * C > 12 * 3 * 1560 * 24 * 1560:
            continue
        if kind in ("lsh", "buckets") and (whole > 12 * 64 * 1560 or -(-n_q // c["BQ"]) * (-(-c["n_p"] // 32)) * 4 > 48 * 1024):
            continue
        if c["path"] == "step" and whole * c["d"] < 2 * 4 * 256 * 64:
            continue
        return c


def _n_sel(c):
    live = c["frames"] if c["path"] == "start" else c["cap"]
    return max(2, math.ceil(c["keep"] * math.ceil(live * c["T"] / BK)))


class _Stream:
    """Frames and queries of one layer, drawn on the GPU."""

    def __init__(self, c, g):
        self.c, self.g = c, g
        self.dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        self.centreK = self.normal(c["H"], c["clusters"], c["d"])
        self.centreV = self.normal(c["H"], c["clusters"], c["d"])
        self.cluster = (torch.arange(c["T"], device="cuda") * c["clusters"]) // c["T"]
        self.K = self.V = None

    def normal(self, *shape):
        return torch.randn(shape, device="cuda", generator=self.g)

    def fresh(self, centres):
        return centres[:, self.cluster, :] + SIGMA_W * self.normal(self.c["H"], self.c["T"], self.c["d"])

    def frame(self):
        K, V = self.fresh(self.centreK), self.fresh(self.centreV)
        if self.K is not None:
            same = (torch.rand((self.c["T"],), device="cuda", generator=self.g) < self.c["repeat"])[None, :, None]
            K = torch.where(same, self.K + self.c["drift"] * self.normal(*K.shape), K)
            V = torch.where(same, self.V + self.c["drift"] * self.normal(*V.shape), V)
        self.K, self.V = K, V
        return K.to(self.dt), V.to(self.dt)

    def queries(self):
        return torch.cat([self.fresh(self.centreK) for _ in range(self.c["frames"])], dim=1).to(self.dt)

    def prompt(self):
        c = self.c
        n_pc = max(4, min(32, c["n_p"] // 8))
        cK, cV = self.normal(c["H"], n_pc, c["d"]), self.normal(c["H"], n_pc, c["d"])
        near = torch.randperm(c["clusters"], device="cuda", generator=self.g)[:3]
        cK[:, :3] = self.centreK[:, near] + 0.1 * self.normal(c["H"], 3, c["d"])
        of = torch.randint(0, n_pc, (c["n_p"],), device="cuda", generator=self.g)
        noise = lambda: SIGMA_W * self.normal(c["H"], c["n_p"], c["d"])  # noqa: E731
        return (cK[:, of] + noise()).to(self.dt), (cV[:, of] + noise()).to(self.dt)


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    H, d, r, T, F, BQ = c["H"], c["d"], c["r"], c["T"], c["frames"], c["BQ"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)
    s = dict(c=c, i32=dict(dtype=torch.int32, device="cuda"))
    stream = _Stream(c, g)
    n_q, C = F * T, c["cap"] * T
    n_qb = -(-n_q // BQ)
    sign = lambda w: (torch.randint(0, 2, (d, w), device="cuda", generator=g) * 2 - 1).to(torch.int8)  # noqa: E731
    s["codec"] = codec = fa.Codec(sign(r), float(np.float32(127.0 / QRANGE)), SHIFT)
    new = lambda shape, dt: torch.empty(shape, dtype=dt, device="cuda")  # noqa: E731
    scratch = lambda op, n, k, rr: new((max(256, fa.workspace_bytes(op, H, n, k, rr, BQ, BK, N_REP)),), torch.uint8)  # noqa: E731

    # the prompt and its codes are fixed for a rollout
    s["pK"], s["pV"] = stream.prompt()
    s["pcode"] = fa.encode(s["pK"], codec)
    s["plen"] = torch.full((H,), c["n_p"], **s["i32"])
    s["fused"] = c["dtype"] == "bf16" and d == 128 and BQ == 128 and c["n_sel_p"] <= 64
    s["csel"] = (new((H, n_qb, c["n_sel_p"]), torch.int32), new((H, n_qb), torch.int32))
    s["Ox"] = new((H, n_q, d), stream.dt)
    if not s["fused"]:
        s["ws_x"] = scratch(fa.OP_SELECT_CROSS, n_q, c["n_p"], r)
    s["qcode"] = new((H, n_q, r), torch.int8)
    s["chunk"] = 0
    if c["path"] == "prompt":
        s["Q"] = [stream.queries() for _ in range(RING)]
        return s

    # the cache: full, with the frames as they came (multiplicity 1), or empty at a rollout's start
    s["cache"] = cache = fa.Cache.empty(H, C, d, r, stream.dt)
    s["frame_id"], s["prev"] = 0, None
    if c["path"] == "step":
        for f in range(c["cap"]):
            cache.K[:, f * T:(f + 1) * T], cache.V[:, f * T:(f + 1) * T] = stream.frame()
            cache.stamp[:, f * T:(f + 1) * T] = f
        cache.cnt.fill_(1)
        cache.len.fill_(C)
        fa.encode(cache.K, codec, out=cache.code)
        s["frame_id"] = c["cap"]
        s["prev"] = torch.arange(C - T, C, **s["i32"]).repeat(H, 1).contiguous()
    s["new"] = [stream.frame() for _ in range(RING * F)]
    s["Q"] = [stream.queries() for _ in range(RING)]
    s["at"] = 0
    # merge maps of the previous chunk and of this one
    s["maps"] = [(new((H, T), torch.int32), new((H, T), torch.uint8), new((H, 8), torch.int32)) for _ in range(2 * F)]
    s["ws_c"] = torch.zeros(fa.workspace_bytes(fa.OP_COMPRESS, H, T, C, r), dtype=torch.uint8, device="cuda")
    s["n_sel"] = n_sel = _n_sel(c)
    s["sel"] = (new((H, n_qb, n_sel), torch.int32), new((H, n_qb), torch.int32))
    s["O"] = (new((H, n_q, d), stream.dt), new((H, n_q), torch.float32))
    s["ws_a"] = scratch(fa.OP_ATTN, n_q, C, r) if stream.dt == torch.bfloat16 and d == 128 else None
    if c["kv"] == "fp8":
        s["kv8"] = fa.kv8_empty(H, C, d)
        fa.kv_to_fp8(cache, *s["kv8"])
    if c["ann"] == "int8":
        s["ws_s"] = scratch(fa.OP_SELECT_SELF, n_q, C, r)
    elif c["ann"] == "lsh":
        s["Rb"] = sign(HASH_BITS)
        s["qbits"] = new((H, n_q, HASH_BITS // 32), torch.int32)
        s["kbits"] = new((H, C, HASH_BITS // 32), torch.int32)
        s["ws_s"] = scratch(fa.OP_SELECT_LSH, n_q, C, HASH_BITS)
    else:   # buckets of the cache's slots, kept up to date slot by slot
        s["kbucket"] = fa.prompt_buckets(cache.code, s["pcode"], N_BUCKETS)
        s["qbucket"] = torch.full((H, n_q, N_BUCKETS), -1, **s["i32"])
        s["ws_s"] = scratch(fa.OP_SELECT_BUCKETS, n_q, C, c["n_p"])
    return s


def run(s):
    c = s["c"]
    BQ, scale = c["BQ"], c["d"] ** -0.5
    Q = s["Q"][s["chunk"] % RING]
    out = {}
    if c["path"] != "prompt":
        out.update(_cache_and_self(s, c, Q, BQ, scale))
    else:
        fa.encode(Q, s["codec"], out=s["qcode"])
    if s["fused"]:
        fa.ann_cross_attn_fwd(Q, s["qcode"], s["pK"], s["pV"], s["pcode"], BQ, c["n_sel_p"], scale, out=(*s["csel"], s["Ox"]))
    else:
        fa.ann_select_cross(s["qcode"], s["pcode"], BQ, c["n_sel_p"], ws=s["ws_x"], out=s["csel"])
        fa.sparse_attn_fwd(Q, s["pK"], s["pV"], None, s["plen"], *s["csel"], BQ, 1, scale, out=(s["Ox"], None), want_lse=False)
    s["chunk"] += 1
    out.update(qcode=s["qcode"], csel=s["csel"], Ox=s["Ox"])
    return out


def _cache_and_self(s, c, Q, BQ, scale):
    cache, F = s["cache"], c["frames"]
    if c["path"] == "start":
        cache.len.zero_()
        s["prev"], s["frame_id"] = None, 0
    first = s["frame_id"]
    maps = s["maps"][(s["chunk"] & 1) * F:][:F]
    n = len(s["new"])
    for f in range(F):
        at = s["at"] % (2 * n - 2)          # 0 .. n-1 and back
        K, V = s["new"][min(at, 2 * n - 2 - at)]
        s["at"] += 1
        fa.tempcache_compress(cache, s["codec"], K, V, cand=None if c["match"] == "all" else s["prev"], tau2_q16=TAU2,
                              frame_id=s["frame_id"], rep_mode={"last": fa.REP_LAST, "mean": fa.REP_MEAN, "medoid": fa.REP_MEDOID}[c["rep"]],
                              ws=s["ws_c"], out=maps[f], ws_persistent=True)
        s["prev"] = maps[f][0]
        s["frame_id"] += 1
        if c["ann"] == "buckets":
            fa.prompt_buckets(cache.code, s["pcode"], N_BUCKETS, idx=s["prev"], out=s["kbucket"])
    if c["kv"] == "fp8":
        fa.kv_to_fp8(cache, *s["kv8"], stamp_lo=first)
    fa.encode(Q, s["codec"], out=s["qcode"])
    if c["ann"] == "int8":
        fa.ann_select_self(s["qcode"], cache.code, cache.len, BQ, N_REP, BK, s["n_sel"], ws=s["ws_s"], out=s["sel"])
    elif c["ann"] == "lsh":
        fa.encode_sign(Q, s["Rb"], s["codec"].qscale, out=s["qbits"])
        fa.encode_sign(cache.K, s["Rb"], s["codec"].qscale, out=s["kbits"])
        fa.ann_select_lsh(s["qbits"], s["kbits"], cache.len, BQ, N_REP, BK, s["n_sel"], ws=s["ws_s"], out=s["sel"])
    else:
        fa.prompt_buckets(s["qcode"], s["pcode"], N_BUCKETS, out=s["qbucket"])
        fa.ann_select_buckets(s["qbucket"], s["kbucket"], cache.len, c["n_p"], BQ, BK, s["n_sel"], n_sink=1, n_local=1,
                              ws=s["ws_s"], out=s["sel"])
    if c["kv"] == "fp8":
        fa.sparse_attn_fwd_fp8(Q, *s["kv8"], cache.cnt, cache.len, cache.K.shape[1], *s["sel"], BQ, BK, scale, out=s["O"], ws=s["ws_a"])
    else:
        fa.sparse_attn_fwd(Q, cache.K, cache.V, cache.cnt, cache.len, *s["sel"], BQ, BK, scale, out=s["O"], ws=s["ws_a"])
    return dict(maps=maps, sel=s["sel"], O=s["O"], cache=[cache.K, cache.V, cache.code, cache.cnt, cache.stamp, cache.len],
                kv8=s.get("kv8"))


def work(case):
    c = dict(DEFAULTS, **case)
    H, d, r, T, F = c["H"], c["d"], c["r"], c["T"], c["frames"]
    es = 2 if c["dtype"] == "bf16" else 4
    n_q = F * T
    n_qb = -(-n_q // c["BQ"])
    row = d * es
    # queries in, codes of the queries out, prompt in, prompt attention out
    b = H * (n_q * (2 * row + r) + c["n_p"] * (2 * row + r))
    f = H * n_q * (4.0 * d * min(c["n_sel_p"], c["n_p"]) + 2.0 * c["n_p"] * r + 2.0 * d * r)
    if c["path"] != "prompt":
        live = (F if c["path"] == "start" else c["cap"]) * T
        n_sel = _n_sel(c)
        kept = min(1.0, n_sel * BK / live)
        kv_row = 2 * d if c["kv"] == "fp8" else 2 * row
        # a frame: its rows in, the matched key, the value read and written, the key written, codes and the rest
        b += H * F * T * (6 * row + 2 * r + 40)
        f += H * F * T * (2.0 * d * r + 2.0 * r * (live if c["match"] == "all" else T))
        if c["kv"] == "fp8":
            b += H * F * T * (2 * row + 2 * d)
        # selection: what the cache keeps for it, once
        if c["ann"] == "lsh":
            b += H * (live * (row + HASH_BITS // 8) + n_q * HASH_BITS // 8)
            f += H * (2.0 * HASH_BITS * d * (live + n_q) + 2.0 * HASH_BITS * live * n_qb * N_REP)
        elif c["ann"] == "buckets":
            b += H * (live + n_q) * 4 * N_BUCKETS
            f += H * 2.0 * r * c["n_p"] * (n_q + F * T)
        else:
            b += H * live * r
            f += H * 2.0 * r * live * n_qb * N_REP
        b += H * n_qb * n_sel * 4
        # attention: every key block that some query block wants, once; outputs
        b += H * (live * (1.0 - (1.0 - kept) ** n_qb) * kv_row + n_q * (row + 4))
        f += H * 4.0 * d * n_q * min(live, n_sel * BK)
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """About four times what the attention outputs of the listed and drawn shapes differ by from the same sums in 64 bits
    (bf16: 1.7e-3 and 5.7e-3 at most, the rounding of the stored output; fp32: up to 6e-6 and 4e-5 over long key lists; the
    8-bit copy: 2.3e-3 and 1.4e-2 with the weights unrounded).  Whole numbers (codes, maps, selections, multiplicities) and
    the cache's keys are the same everywhere."""
    c = dict(DEFAULTS, **case)
    if c["kv"] == "fp8":
        return {"rel": 1e-2, "max": 0.06}
    if c["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 0.025}
    return {"rel": 1.5e-5, "max": 1.5e-4}
