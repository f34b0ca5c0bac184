"""The work a program has this library do, case by case, for measurement.

A case is one pass of one of six paths over one synthetic batch:

  step       a worker's whole training step: np_dedup, np_route, np_lookup_fwd by key, np_lookup_bwd into send order,
             np_sparse_adagrad (the _t calls on 16-bit tables)
  local      a worker that owns every row it touches: np_dedup without the inverse map, np_lookup_fwd_t by key,
             np_lookup_bwd_adagrad_t
  retrieve   forward only (evaluation, prefetch): np_lookup_fwd_t by key
  requester  a worker's share of a sharded step on global ids: np_dedup, np_route with the composed map, pooling straight
             from the buffer of received rows, np_lookup_bwd into send order
  owner      the shard's share of it: np_dedup of the sources' key lists laid end to end, one gather of the distinct rows,
             the rows handed back per source, the sources' gradients merged, np_sparse_adagrad
  sync       dual-buffer synchronisation between two consecutive batches: np_intersect, np_sync_rows

The shapes are the five configurations of ``paper_2604_06956_amd.workloads`` (tables cut to at most 100 M rows, so that
several states fit one GPU) and plain variations of them.  Keys follow a bounded Zipf law per table, popular ranks
scattered over the rows; lengths follow the configurations' laws; gradients are N(0, 1); the Adagrad state is that of a run
under way.  Everything is made on the GPU from the seed.
"""
import functools
import math

import numpy as np
import torch

from paper_2604_06956_amd import binding as B
from paper_2604_06956_amd import workloads as wl

LR, EPS = 0.01, 1e-8
MODES = {"sum": B.POOL_SUM, "mean": B.POOL_MEAN, "seq": B.SEQ}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
DEV = "cuda"

# rows: the fused table's rows; tables > 1 splits them into tables of log-uniform sizes, 100:1 from largest to smallest.
# len / max_len: "uniform" 1..max_len, "poisson" mean len, "clip" the same clipped to 1..max_len, "fixed" len,
# "seq" one length per sample, uniform in len..max_len, shared by its features.
DEFAULTS = dict(path="step", samples=256, features=8, law="poisson", len=8, max_len=64, rows=100_000, tables=1, alpha=1.05, dim=64,
                mode="sum", table="f32", out="f32", shards=64, hash=True)


def _case(name, **kw):
    c = dict(DEFAULTS, **kw)
    c["name"] = name
    return c


def listed():
    return [
        # one small evaluation batch: the latency of a single call
        _case("retrieve tiny", path="retrieve", samples=256, features=8, law="uniform", max_len=20, dim=16),
        # the smallest training step (configuration "tiny"): launches and host work
        _case("step tiny", samples=256, features=8, law="uniform", max_len=20, dim=16, shards=8, hash=False),
        # a small job on odd sizes: samples, bag lengths and row width fit no tile, 16-bit table
        _case("step ragged f16", samples=1013, features=7, law="uniform", max_len=64, rows=3_000_017, dim=36, alpha=1.2, mode="mean",
              table="f16", shards=37),
        # a micro-batch of a local trainer: one of the pieces a frozen window is cut into
        _case("local micro-batch", path="local", samples=2048, features=26, law="clip", len=4, rows=30_000_000, tables=26, alpha=1.1,
              dim=128),
        # click-through model, one bag per table (configuration "dlrm")
        _case("step dlrm", samples=16_384, features=26, law="clip", len=4, rows=60_000_000, tables=26, alpha=1.1, mode="mean"),
        # a few keys carry most of the traffic (configuration "skew")
        _case("step skew", samples=65_536, features=1, law="fixed", len=32, rows=50_000_000, alpha=1.5, shards=1536),
        # behaviour sequences without pooling, bf16 in and out (configuration "seq")
        _case("step seq", samples=4096, features=4, law="seq", len=200, max_len=1000, rows=40_000_000, tables=4, alpha=1.2, dim=128,
              mode="seq", out="bf16", shards=1536),
        # the largest single-GPU batch (configuration "large")
        _case("step large", samples=131_072, features=40, rows=100_000_000, shards=1536),
        # a local trainer on a 16-bit table
        _case("local bf16", path="local", samples=32_768, features=40, rows=200_000_000, table="bf16"),
        # one worker of a 1,536-shard job: 40-bit global ids, wide rows, bf16 activations
        _case("requester wide ids", path="requester", samples=16_384, features=26, law="clip", len=4, rows=1 << 40, alpha=1.1,
              dim=128, out="bf16", shards=1536),
        # the shard that answers 16 such workers
        _case("owner merge", path="owner", samples=16_384, features=8, len=8, rows=50_000_000, shards=16),
        # two consecutive batches' key sets, the common rows copied
        _case("sync", path="sync", samples=65_536, features=40, rows=100_000_000),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    path = rng.choice(["step", "step", "step", "local", "local", "retrieve", "requester", "owner", "sync"])
    mode = rng.choice(["sum", "mean", "seq"] if path in ("step", "local", "retrieve") else ["sum", "mean"])
    dim = rng.choice([8, 16, 20, 32, 36, 64, 64, 72, 96, 128, 128, 136, 256])
    table = rng.choice(["f32", "f32", "bf16", "f16"]) if path in ("step", "local", "retrieve") else "f32"
    most = min(16e6, 1.2e9 / dim)
    n = _log_uniform(rng, 2e3, most)
    features = rng.randint(1, 40) if mode != "seq" else rng.randint(1, 4)
    if mode == "seq":
        lo = rng.randint(20, 200)
        hi = lo + rng.randint(50, 800)
        law, length, max_len, mean_len = "seq", lo, hi, (lo + hi) / 2
    else:
        law = rng.choice(["uniform", "poisson", "clip", "fixed"])
        length = rng.randint(2, 32)
        max_len = rng.randint(2 * length, 4 * length)
        mean_len = (1 + max_len) / 2 if law == "uniform" else length
    samples = max(1, int(n / (features * mean_len)))
    if path == "requester":
        rows = 1 << rng.randint(33, 41)
    else:
        rows = int(_log_uniform(rng, 1e4, min(1e8, 26e9 / (dim * (4 if table == "f32" else 2)))))
    tables = 1 if path == "requester" or rows < 1e5 else rng.randint(1, features)
    return dict(path=path, samples=samples, features=features, law=law, len=length, max_len=max_len, rows=rows, tables=tables,
                alpha=round(rng.uniform(1.05, 1.5), 3), dim=dim, mode=mode, table=table,
                out="bf16" if mode == "seq" or rng.random() < 0.2 else "f32",
                shards=rng.randint(2, 16) if path == "owner" else rng.choice([1, 8, 37, 64, 500, 1536]), hash=rng.random() < 0.7)


# ---- inputs ----------------------------------------------------------------------------------------------


def _table_rows(c):
    """Rows of every table of the fused one; they add up to c["rows"]."""
    T = c["tables"]
    if T == 1:
        return [c["rows"]]
    w = [10.0 ** (-2.0 * ((7 * t) % T) / (T - 1)) for t in range(T)]
    rows = [max(1, int(c["rows"] * x / sum(w))) for x in w]
    rows[0] += c["rows"] - sum(rows)
    return rows


def _key_bits(c):
    return max(1, (c["rows"] - 1).bit_length())


def _lengths(c, g):
    bags = c["samples"] * c["features"]
    if c["law"] == "seq":
        return torch.randint(c["len"], c["max_len"] + 1, (c["samples"],), generator=g, device=DEV).repeat(c["features"])
    if c["law"] == "fixed":
        return torch.full((bags,), c["len"], dtype=torch.int64, device=DEV)
    if c["law"] == "uniform":
        return torch.randint(1, c["max_len"] + 1, (bags,), generator=g, device=DEV)
    lengths = torch.poisson(torch.full((bags,), float(c["len"]), device=DEV), generator=g).long()
    return lengths.clamp(1, c["max_len"]) if c["law"] == "clip" else lengths


def _zipf_ranks(R, alpha, u):
    """Ranks 0..R-1, p(r) ~ (r+1)^-alpha: an exact cumulative sum for the head, its integral inverted for the tail."""
    M = min(R, 1 << 20)
    cdf = torch.cumsum(torch.arange(1, M + 1, dtype=torch.float64, device=DEV).pow_(-alpha), 0)
    head = float(cdf[-1])
    lo, hi = M + 0.5, R + 0.5
    tail = (lo ** (1 - alpha) - hi ** (1 - alpha)) / (alpha - 1) if R > M else 0.0
    u = u * (head + tail)
    ranks = torch.searchsorted(cdf, u, right=True).clamp_(max=M - 1)
    if R > M:
        x = (lo ** (1 - alpha) - (u - head).clamp_(min=0) * (alpha - 1)).clamp_(min=hi ** (1 - alpha)).pow_(1 / (1 - alpha))
        ranks = torch.where(u < head, ranks, x.round_().long().clamp_(M + 1, R) - 1)
    return ranks


def _rank_to_id(ranks, R, offset):
    """Popular ranks scattered over 0..R-1 (a bijection)."""
    if R <= 1 << 30:
        return (ranks * wl.RANK_STRIDE + offset) % R
    bits = R.bit_length() - 1  # global ids: R is a power of two
    x = (ranks * -7046029254386353131) & (R - 1)  # an odd factor, wrapping
    return (x ^ (x >> (bits // 2 + 1))) & (R - 1)


def _keys(c, offsets, g):
    """int64 row ids of the whole batch; bags lie feature by feature, feature f reads table f % tables."""
    S, F, T = c["samples"], c["features"], c["tables"]
    rows = _table_rows(c)
    at = offsets[::S].tolist()
    keys = torch.empty(at[-1], dtype=torch.int64, device=DEV)
    base = np.concatenate([[0], np.cumsum(rows)])
    for t in range(T):
        mine = [(at[f], at[f + 1]) for f in range(t, F, T)] if T > 1 else [(0, at[-1])]
        n = sum(b - a for a, b in mine)
        if not n:
            continue
        u = torch.rand(n, dtype=torch.float64, generator=g, device=DEV)
        ids = _rank_to_id(_zipf_ranks(rows[t], c["alpha"], u), rows[t], 12345 + 7919 * t) + int(base[t])
        done = 0
        for a, b in mine:
            keys[a:b] = ids[done:done + b - a]
            done += b - a
    return keys


def _batch(c, g):
    lengths = _lengths(c, g)
    offsets = torch.zeros(lengths.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lengths, 0, out=offsets[1:])
    return _keys(c, offsets, g), offsets.int()


def _zeros(*shape, dtype=torch.int32):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def _ws(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device=DEV)


def _dedup_buffers(n, inverse=True):
    return dict(unique=_zeros(n, dtype=torch.int64), inverse=_zeros(n) if inverse else None, counts=_zeros(n), occ_offsets=_zeros(n + 1),
                occ=_zeros(n), num_unique=_zeros(1))


def _route_buffers(n, S, compose=False):
    r = dict(send_keys=_zeros(n, dtype=torch.int64), splits=_zeros(S), send_offsets=_zeros(S + 1), send_from_unique=_zeros(n),
             unique_to_send=_zeros(n))
    if compose:
        r["lookup_to_send"] = _zeros(n)
    return r


def _randn(shape, g, dtype=torch.float32):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype)


def _table(c, seed, g):
    table = torch.empty((c["rows"], c["dim"]), dtype=DTYPES[c["table"]], device=DEV)
    B.np_util_table_init_t(table, seed & 0x7FFFFFFF)
    return table, torch.rand(c["rows"], generator=g, device=DEV)


def _distinct(keys, bits):
    d = B.np_dedup(keys, bits)
    return d["unique"][:int(d["num_unique"])]


def _room(expected):
    """Entries a program sets aside for a batch of about this many: its buffers keep their size from batch to batch."""
    return int(1.03 * expected + 8 * math.sqrt(expected * 64)) + 64


def prepare(case, seed):
    c = case
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    s = dict(case=c, mode=MODES[c["mode"]], bits=_key_bits(c), fn=B.SHARD_HASH if c["hash"] else B.SHARD_MOD)
    D, S, path = c["dim"], c["shards"], c["path"]

    if path == "sync":
        for who in "ab":
            s["keys_" + who] = _distinct(_batch(c, g)[0], s["bits"])
            s["cap_" + who] = s["keys_" + who].numel()
            s["num_" + who] = torch.tensor([s["cap_" + who]], dtype=torch.int32, device=DEV)
        s["cap"], room = min(s["cap_a"], s["cap_b"]), _room(_sizes(c, c["samples"])[2])
        s["active"], s["prefetch"] = _randn((room, D), g), _randn((room, D), g)
        s["isec"] = dict(idx_a=_zeros(room), idx_b=_zeros(room), num_common=_zeros(1))
        s["ws"] = _ws(int(B.lib.np_intersect_workspace_bytes(s["cap_b"])))
        return s

    if path == "owner":
        part = dict(c, samples=max(1, c["samples"] // S))
        lists = [_distinct(_batch(part, g)[0], s["bits"]) for _ in range(S)]
        s["keys"] = torch.cat(lists)
        n, room = s["keys"].numel(), _room(S * _sizes(part, part["samples"])[2])
        s["dY"], s["reply"], s["rows"] = _randn((n, D), g), _zeros(room, D, dtype=torch.float32), _zeros(room, D, dtype=torch.float32)
        s["iota"], s["count"] = torch.arange(n, dtype=torch.int32, device=DEV), torch.tensor([n], dtype=torch.int32, device=DEV)
        s["off"], s["no_bags"], s["no_out"] = torch.arange(n + 1, dtype=torch.int32, device=DEV), _zeros(1), _zeros(0, D, dtype=torch.float32)
        s["mode"], s["max_len"], bags = B.POOL_SUM, 1, n
    else:
        s["keys"], s["off"] = _batch(c, g)
        n, bags = s["keys"].numel(), s["off"].numel() - 1
        room, s["max_len"] = _room(_sizes(c, c["samples"])[1]), c["max_len"]
        seq = c["mode"] == "seq"
        shape = (bags, s["max_len"], D) if seq else (bags, D)
        s["out"], s["out_dtype"] = _zeros(*shape, dtype=DTYPES[c["out"]]), B.BF16 if c["out"] == "bf16" else B.F32
        if path != "retrieve":
            s["dY"] = _randn(shape, g, DTYPES[c["out"]])
    if n > room:
        raise ValueError("a batch larger than its buffers")
    s["n"] = s["cap"] = n
    if path == "requester":
        s["received"] = _randn((n, D), g) * 0.01
    else:
        s["table"], s["state"] = _table(c, seed, g)
    if path == "retrieve":
        return s
    s["dd"], s["ws_d"] = _dedup_buffers(room, path != "local"), _ws(B.np_dedup_workspace_bytes(n, s["bits"]))
    s["ws_b"] = _ws(B.np_lookup_bwd_workspace_bytes(bags, n, D, s["mode"]))
    if path != "local":
        s["grads"] = _zeros(room, D, dtype=torch.float32)
    if path in ("step", "requester"):
        s["rr"], s["ws_r"] = _route_buffers(room, S, path == "requester"), _ws(B.np_route_workspace_bytes(n, S))
    return s


# ---- one pass --------------------------------------------------------------------------------------------


def run(s):
    c, D, n, cap, mode = s["case"], s["case"]["dim"], s.get("n"), s["cap"], s["mode"]
    path = c["path"]

    if path == "sync":
        i = s["isec"]
        B.np_intersect(s["keys_a"], s["num_a"], s["cap_a"], s["keys_b"], s["num_b"], s["cap_b"], out=i, ws=s["ws"])
        B.np_sync_rows(s["active"], i["idx_a"], s["prefetch"], i["idx_b"], i["num_common"], cap)
        return [i, s["prefetch"]]

    if path == "retrieve":
        out, _ = B.np_lookup_fwd_t(s["table"], s["keys"], None, s["off"], n, mode, s["max_len"], s["out_dtype"], out=s["out"])
        return out

    d = s["dd"]
    if path == "local":
        B.np_dedup(s["keys"], s["bits"], out=d, ws=s["ws_d"], want_inverse=False)
        B.np_lookup_fwd_t(s["table"], s["keys"], None, s["off"], n, mode, s["max_len"], s["out_dtype"], out=s["out"])
        B.np_lookup_bwd_adagrad_t(s["dY"], mode, s["max_len"], s["off"], n, d["occ_offsets"], d["occ"], d["unique"], d["num_unique"], cap,
                                  s["table"], s["state"], LR, EPS, ws=s["ws_b"])
        return [d, s["out"], s["table"], s["state"]]

    B.np_dedup(s["keys"], s["bits"], out=d, ws=s["ws_d"])
    if path == "owner":
        B.np_lookup_fwd(s["table"], d["unique"], None, s["no_bags"], 0, mode, num_list=d["num_unique"], cap=cap, want_rows=True,
                        out=s["no_out"], rows_out=s["rows"])
        B.np_sync_rows(s["rows"], d["inverse"], s["reply"], s["iota"], s["count"], n)
        B.np_lookup_bwd(s["dY"], D, mode, 1, s["off"], n, d["occ_offsets"], d["occ"], d["num_unique"], cap, grads=s["grads"], ws=s["ws_b"])
        B.np_sparse_adagrad(s["table"], s["state"], d["unique"], s["grads"], d["num_unique"], cap, LR, EPS)
        return [d, s["rows"], s["reply"], s["grads"], s["table"], s["state"]]

    r = s["rr"]
    if path == "requester":
        B.np_route(d["unique"], d["num_unique"], cap, c["shards"], s["fn"], inverse=d["inverse"], n=n, out=r, ws=s["ws_r"])
        B.np_lookup_fwd(s["received"], None, r["lookup_to_send"], s["off"], n, mode, s["max_len"], s["out_dtype"], out=s["out"])
    else:
        fwd = B.np_lookup_fwd if c["table"] == "f32" else B.np_lookup_fwd_t
        B.np_route(d["unique"], d["num_unique"], cap, c["shards"], s["fn"], out=r, ws=s["ws_r"])
        fwd(s["table"], s["keys"], None, s["off"], n, mode, s["max_len"], s["out_dtype"], out=s["out"])
    B.np_lookup_bwd(s["dY"], D, mode, s["max_len"], s["off"], n, d["occ_offsets"], d["occ"], d["num_unique"], cap,
                    unique_to_send=r["unique_to_send"], grads=s["grads"], ws=s["ws_b"])
    if path == "requester":
        return [d, r, s["out"], s["grads"]]
    update = B.np_sparse_adagrad if c["table"] == "f32" else B.np_sparse_adagrad_t
    update(s["table"], s["state"], r["send_keys"], s["grads"], d["num_unique"], cap, LR, EPS)
    return [d, r, s["out"], s["grads"], s["table"], s["state"]]


# ---- what a pass cannot do without -----------------------------------------------------------------------


@functools.lru_cache(maxsize=None)
def _expected_unique(rows, alpha, n):
    return wl.expected_unique(rows, alpha, n)


def _sizes(c, samples):
    """Expected lookups, distinct keys and longest bag of a batch of this many samples."""
    bags = samples * c["features"]
    mean = {"uniform": (1 + c["max_len"]) / 2, "seq": (c["len"] + c["max_len"]) / 2}.get(c["law"], c["len"])
    n, rows, T = bags * mean, _table_rows(c), c["tables"]
    U = 0.0
    for t in range(T):
        feats = len(range(t, c["features"], T)) if T > 1 else c["features"]
        if feats:
            U += _expected_unique(rows[t], c["alpha"], round(samples * feats * mean))
    return bags, n, U


def work(case):
    c = case
    D, path = c["dim"], c["path"]
    bags, n, U = _sizes(c, c["samples"])
    row, trow = 4 * D, D * (4 if c["table"] == "f32" else 2)
    elem = 2 if c["out"] == "bf16" else 4
    if path == "sync":
        common = 0.4 * U  # about what two batches of one popularity law share
        return {"bytes": 16 * U + 8 * common + 2 * common * row, "flops": 0}
    if path == "owner":
        per = _sizes(c, max(1, c["samples"] // c["shards"]))[2]
        m = per * c["shards"]
        dedup = 8 * m + 8 * m + 16 * U
        return {"bytes": dedup + U * row + m * row + m * row + 2 * U * row + U * row + 8 * U, "flops": (m + 5 * U) * D}
    out = bags * elem * D * (c["max_len"] if c["mode"] == "seq" else 1)
    grad_in = n * elem * D if c["mode"] == "seq" else out
    forward = 8 * n + 4 * bags + U * trow + out
    if path == "retrieve":
        return {"bytes": forward, "flops": n * D}
    dedup = 4 * n + 16 * U + (0 if path == "local" else 4 * n)  # the keys are counted with the forward
    if path == "local":
        return {"bytes": dedup + forward + grad_in + U * trow + 8 * U, "flops": (2 * n + 5 * U) * D}
    route = 16 * U + 8 * c["shards"]
    if path == "requester":
        return {"bytes": dedup + route + 8 * n + 4 * bags + 4 * n + U * row + out + grad_in + U * row, "flops": 2 * n * D}
    return {"bytes": dedup + route + forward + grad_in + U * row + U * trow + 8 * U, "flops": (2 * n + 5 * U) * D}


def tolerance(case):
    c = case
    if c["path"] == "sync":
        return "exact"  # whole numbers and copied rows
    if c["path"] == "retrieve" and c["out"] == "f32":
        return {"rel": 1e-5}  # 16-bit rows are widened exactly, the sums are fp32
    if c["table"] == "bf16" or c["out"] == "bf16":
        return {"rel": 2e-3, "max": 1e-2}  # a value on a rounding boundary may fall to either neighbour, 2^-8 apart
    if c["table"] == "f16":
        return {"rel": 3e-4, "max": 2e-3}  # the same with neighbours 2^-10 apart
    return {"rel": 1e-5}  # fp32 sums in another order
