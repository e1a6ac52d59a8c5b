"""Cases by which the speed of the distance stage is measured.

Each case is a dict of plain values; `listed()` gives the fixed ones, `draw()`
another one of the same ranges.  `prepare()` makes what a program holds before
the call (keys, a resident database, encrypted queries), `run()` is one pass
through the public entry points, `work()` the bytes and operations that one
pass cannot do without.

Kinds of work:

  scan      the server's distance stage for Q queries against every chunk of a
            resident database (linear scan, or one batch of the serving loop);
            `digits`: the database also holds its int8 digit form,
            `private`: the circuit-private form, `mode`: fused launches or a
            replayed graph
  worklist  phase 2 of the clustered form on a resident cluster-packed
            database: every query scans the chunks of its own clusters and the
            stash
  gathered  phase 2 of the clustered form on chunks packed and encoded per
            call from the selected clusters' points, with the stash as tail
  encode    a server's points into their resident form
  encrypt   a client's queries into ciphertexts
  decrypt   a client's answer (one query's ciphertexts) into shares
  kmeans    rounds of the balanced clustering's k-means

Every output is an integer (residues, shares, assignments).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1904_02033_amd import balance, clustered, native as nat, stage

_MODES = {"fused": nat.SANNS_MODE_FUSED, "batched": nat.SANNS_MODE_BATCHED}


def _scan(n, d, dtype, Q, **kw):
    c = {"kind": "scan", "N": 8192, "n": n, "d": d, "dtype": dtype, "Q": Q, "mode": "batched",
         "digits": False, "private": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one query against 10,000 points, where launches
        # and the depth of each kernel count
        _scan(10_000, 128, "u8", 1, N=4096, mode="fused", name="scan-10Kx128-q1"),
        # one query against a million points: the database is streamed once
        _scan(1_000_000, 128, "u8", 1, mode="fused", name="scan-1Mx128-q1"),
        # the benchmark's batch: 64 queries on the matrix-core schedule
        _scan(1_000_000, 128, "u8", 64, digits=True, name="batch-1Mx128-q64"),
        # one launch of the serving loop with a few waiting requests
        _scan(1_000_000, 96, "i8", 9, digits=True, mode="fused", name="serve-1Mx96-q9"),
        # a batch on a context with no flags set (64-bit residues alone)
        _scan(100_000, 128, "u8", 32, name="batch-100Kx128-q32"),
        # a batch whose answers are re-randomised and flooded
        _scan(100_000, 96, "i8", 16, digits=True, private=True, name="private-100Kx96-q16"),
        # phase 2 of the clustered form, resident and gathered
        {"kind": "worklist", "name": "clusters-2Mx96-q8", "N": 8192, "n": 2_000_000, "d": 96,
         "dtype": "i8", "Q": 8, "u": 32, "cluster": 600, "stash": 20_000},
        {"kind": "gathered", "name": "gathered-2Mx96-q32", "N": 8192, "n": 2_000_000, "d": 96,
         "dtype": "i8", "Q": 32, "u": 64, "cluster": 600, "stash": 100_000},
        # a server's set-up: 200,000 points with the digit form
        {"kind": "encode", "name": "encode-200Kx128", "N": 8192, "n": 200_000, "d": 128,
         "dtype": "u8", "digits": True},
        # the client's two halves: four queries out, one million-point answer in
        {"kind": "encrypt", "name": "encrypt-q4x128", "N": 8192, "d": 128, "dtype": "u8", "Q": 4},
        {"kind": "decrypt", "name": "decrypt-123", "N": 8192, "M": 123},
        # rounds of the clustering that prepares an index
        {"kind": "kmeans", "name": "kmeans-200Kx96-k2000", "n": 200_000, "d": 96, "k": 2000,
         "iters": 6},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan"] * 5 + ["private", "worklist", "gathered", "encode", "encrypt",
                                      "decrypt", "kmeans"])
    N = rng.choice([4096, 8192, 8192])
    dtype = rng.choice(["u8", "i8"])
    d = rng.choice([64, 96, 100, 128, rng.randint(16, 200)])
    if kind in ("scan", "private"):
        n = _log(rng, 5_000, 1_000_000)
        Q = rng.choice([1, 2, rng.randint(2, 16), rng.randint(1, 64)])
        digits = rng.random() < 0.5
        most = 20e6 * 128 if not digits or d > 128 or kind == "private" else 60e6 * 128
        n = max(5_000, min(n, int(most / (Q * d))))
        return _scan(n, d, dtype, Q, N=N, digits=digits, private=kind == "private",
                     mode=rng.choice(["fused", "batched"]))
    if kind in ("worklist", "gathered"):
        return {"kind": kind, "N": 8192, "n": _log(rng, 100_000, 1_500_000), "d": min(d, 128),
                "dtype": dtype, "Q": rng.randint(1, 16), "u": rng.randint(4, 48),
                "cluster": rng.randint(100, 800), "stash": _log(rng, 2_000, 60_000)}
    if kind == "encode":
        return {"kind": kind, "N": N, "n": _log(rng, 5_000, 300_000), "d": d, "dtype": dtype,
                "digits": rng.random() < 0.5}
    if kind == "encrypt":
        return {"kind": kind, "N": N, "d": d, "dtype": dtype, "Q": rng.randint(1, 8)}
    if kind == "decrypt":
        return {"kind": kind, "N": N, "M": _log(rng, 1, 500)}
    return {"kind": kind, "n": _log(rng, 5_000, 200_000), "d": min(d, 128), "k": _log(rng, 30, 2500),
            "iters": rng.randint(2, 6)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _limbs(N):
    return 2 if N == 4096 else 3


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _points(n, d, dtype, g, centres=None):
    """uint8: a mixture of 1,000 Gaussians, clipped to bytes; int8: directions
    on the sphere of radius 127."""
    if dtype == "u8":
        comp = torch.randint(0, len(centres), (n,), device="cuda", generator=g)
        x = torch.randn((n, d), device="cuda", generator=g)
        return (centres[comp] + 20.0 * x).round_().clamp_(0, 255).to(torch.uint8)
    x = torch.randn((n, d), device="cuda", generator=g)
    x *= 127.0 / x.norm(dim=1, keepdim=True)
    return x.round_().clamp_(-127, 127).to(torch.int8)


def _points_and_queries(c, n, Q, g):
    cen = torch.rand((1000, c["d"]), device="cuda", generator=g) * 255.0
    return (_points(n, c["d"], c["dtype"], g, cen),
            _points(Q, c["d"], c["dtype"], g, cen).to(torch.int32))


def _context(c):
    N = c["N"]
    p = nat.sanns_params_derive(N, _limbs(N), 26 if c.get("dtype") == "i8" else 25)
    if c.get("digits"):
        p.flags |= nat.SANNS_FLAG_DIGIT_DB
    return stage.Context(params=p)


def _key(seed):
    return np.random.default_rng(seed).integers(0, 256, 32, dtype=np.uint8).tobytes()


def _ids(Q, seed):
    return (torch.arange(Q, dtype=torch.int64, device="cuda") + 1000 * seed).view(torch.uint64)


def _clusters(c):
    """Sizes of clusters bounded as the balanced clustering bounds them, and
    the clusters that each query selects.  They come from the case alone, so
    that every seed gives the same number of output rows."""
    r = np.random.default_rng(c["n"] + c["u"])
    inside = c["n"] - c["stash"]
    k = max(c["u"], inside // c["cluster"])
    size = r.integers(max(1, c["cluster"] // 8), 2 * c["cluster"], k)
    size = np.maximum(1, size * inside // size.sum())
    size[-1] += inside - size.sum()
    return size, [np.sort(r.choice(k, c["u"], replace=False)) for _ in range(c["Q"])]


def prepare(case, seed):
    c, kind = case, case["kind"]
    g = _gen(seed)
    s = {"case": c}
    if kind == "kmeans":
        s["km"] = balance.KMeans(_points(c["n"], c["d"], "i8", g))
        s["init"] = np.random.default_rng(seed).permutation(c["n"])[:c["k"]].astype(np.int64)
        return s
    s["ctx"] = ctx = _context(c)
    if kind == "encode":
        s["points"] = _points_and_queries(c, c["n"], 1, g)[0]
        s["slots"] = stage.linear_slot_map(c["n"], c["N"],
                                           np.random.default_rng(seed).permutation(c["n"]))
        return s
    s["sk"] = sk = stage.keygen(ctx, seed)
    if kind == "encrypt":
        s["msgs"] = _points_and_queries(c, 1, c["Q"], g)[1].contiguous()
        s["seed"] = seed + 7
        return s
    if kind == "decrypt":
        # an answer: encryptions of uniform values below t at coefficient 0
        # under uniform masks, which is what the server's outputs look like
        t = ctx.t
        msgs = torch.randint(0, t, (c["M"], 1), device="cuda", generator=g, dtype=torch.int32)
        s["ct"] = stage.encrypt_query_seeded(ctx, sk, msgs, seed + 7)[:, 0].contiguous()
        s["qnorm2"] = torch.randint(0, t, (1,), device="cuda", generator=g,
                                    dtype=torch.int32).repeat(c["M"]).view(torch.uint32)
        return s
    Q = c["Q"]
    points, queries = _points_and_queries(c, c["n"], Q, g)
    s["ct"] = stage.encrypt_query_seeded(ctx, sk, queries.contiguous(), seed + 7)
    s["ids"], s["key"] = _ids(Q, seed), _key(seed)
    if kind == "scan":
        slots = stage.linear_slot_map(c["n"], c["N"],
                                      np.random.default_rng(seed).permutation(c["n"]))
        s["db"] = stage.encode_db(ctx, points, slots)
        s["dist"] = stage.Distances(ctx, s["db"], Q, mode=_MODES[c["mode"]],
                                    private=c["private"])
        s["pk"] = None
        if c["private"]:
            s["pk"] = torch.stack([stage.public_key(ctx, sk, seed + 100 + q).view(torch.int64)
                                   for q in range(Q)]).view(torch.uint64)
        return s
    size, s["selected"] = _clusters(c)
    r = np.random.default_rng(seed)
    centres = r.integers(-127, 128, (len(size), c["d"])).astype(np.int8)
    if c["dtype"] == "u8":
        centres = (centres.astype(np.int16) + 128).astype(np.uint8)
    s["server"] = clustered.ClusteredServer(
        ctx, points.cpu().numpy(), size, centres, c["stash"], r.permutation(len(size)),
        r.permutation(c["stash"]), s["key"], _key(seed + 1), gathered=kind == "gathered")
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def _i64(x):
    return x.view(torch.int64)


def _i32(x):
    return x.view(torch.int32)


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "scan":
        ct, share = s["dist"].run(s["ct"], s["key"], s["ids"], pk=s["pk"])
        return [_i64(ct), _i32(share)]
    if kind == "worklist":
        ct, share, work = s["server"].point_distances(s["ct"], s["ids"], s["selected"],
                                                      mode=nat.SANNS_MODE_FUSED)
        return [_i64(ct), _i32(share), work.astype(np.int64)]
    if kind == "gathered":
        (ct, share, slot, rows), (ct2, share2) = s["server"].point_distances_gathered(
            s["ct"], s["ids"], s["selected"])
        return [_i64(ct), _i32(share), slot, rows.astype(np.int64), _i64(ct2), _i32(share2)]
    if kind == "encode":
        ctx, c = s["ctx"], s["case"]
        db = stage.encode_db(ctx, s["points"], s["slots"])
        C, d, N, L = db.n_chunks, db.d, ctx.N, ctx.L
        a, b = L * C * d * N * 8, C * N * 4
        out = [db.mem[:a].view(torch.int64), db.mem[a:a + b].view(torch.int32)]
        if c["digits"] and d <= 128:
            out.append(db.mem[a + b:a + b + L * N * C * (7 * ((d + 31) // 32 * 32) + 16)])
        return out
    if kind == "encrypt":
        return _i64(stage.encrypt_query_seeded(s["ctx"], s["sk"], s["msgs"], s["seed"]))
    if kind == "decrypt":
        return _i32(stage.decrypt_shares(s["ctx"], s["sk"], s["ct"], s["qnorm2"]))
    C, assign, rounds = s["km"].run(s["init"], s["case"]["iters"])
    return [C, assign, rounds]


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def work(case):
    """Bytes: every input read once and every output written once.  Flops: two
    per multiply-add of residues (or of int8 coordinates in k-means) and two
    per butterfly of the transforms."""
    c, kind = case, case["kind"]
    if kind == "kmeans":
        n, d, k, it = c["n"], c["d"], c["k"], c["iters"]
        return {"bytes": it * (n * d + 4 * n + 4 * k * d), "flops": it * 2.0 * n * k * d}
    N, L = c["N"], _limbs(c["N"])
    poly, ntt = 8 * N, N * math.log2(N)  # bytes of a residue polynomial, flops of its transform
    d = c.get("d", 1)
    if kind == "encode":
        C = -(-c["n"] // N)
        out = L * C * d * poly + 4 * C * N
        if c["digits"] and d <= 128:
            out += L * N * C * 7 * d
        return {"bytes": c["n"] * d + 8 * C * N + out, "flops": L * C * d * ntt}
    if kind == "encrypt":
        polys = c["Q"] * d * L
        return {"bytes": 4 * c["Q"] * d + 2 * polys * poly, "flops": polys * (2 * ntt + 2 * N)}
    if kind == "decrypt":
        polys = c["M"] * L
        return {"bytes": 2 * polys * poly + 4 * c["M"] * N, "flops": polys * (2 * ntt + 2 * N)}
    Q = c["Q"]
    if kind == "scan":
        C = -(-c["n"] // N)
        rows, read, enc = Q * C, L * C * d * poly + 4 * C * N, 0
    elif kind == "worklist":
        stash = -(-c["stash"] // N)
        mine = min(-(-(c["n"] - c["stash"]) // N), c["u"])
        rows, enc = Q * (mine + stash), 0
        read = (min(Q * mine, -(-(c["n"] - c["stash"]) // N)) + stash) * L * d * poly
    else:
        stash = -(-c["stash"] // N)
        mine = Q * -(-c["u"] * c["cluster"] // N)
        rows, enc = mine + Q * stash, mine * d * L
        read = stash * L * d * poly + Q * c["u"] * c["cluster"] * d
    polys = 2 * L * (Q * d + rows) + enc
    out = rows * (2 * L * poly + 4 * N)
    return {"bytes": Q * d * 2 * L * poly + read + out,
            "flops": polys * ntt + rows * 2.0 * 2 * L * N * d}


def exact(case, seed):
    """k-means rounds in 64-bit arithmetic (every value is a whole number that
    a double holds); the other kinds return ciphertexts, residues and masks,
    whole numbers that have no plain 64-bit counterpart."""
    if case["kind"] != "kmeans":
        return None
    s = prepare(case, seed)
    X = s["km"].X.double()
    n, k = X.shape[0], case["k"]
    C = 256.0 * X[torch.as_tensor(s["init"], device="cuda")]
    prev, rounds = None, case["iters"]
    for it in range(case["iters"]):
        cn, cur = C.square().sum(1), []
        j = torch.arange(k, device="cuda", dtype=torch.float64)
        for i in range(0, n, 16384):
            # the smaller index wins a tie
            key = (cn - 512.0 * (X[i:i + 16384] @ C.T)) * k + j
            cur.append(key.argmin(1))
        cur = torch.cat(cur)
        if prev is not None and bool((cur == prev).all()):
            rounds = it + 1
            break
        cnt = torch.bincount(cur, minlength=k).double()
        sums = torch.zeros_like(C).index_add_(0, cur, X)
        num, den = 512 * sums.long() + cnt.long()[:, None], 2 * cnt.long().clamp(min=1)[:, None]
        C = torch.where(cnt[:, None] > 0, num.div(den, rounding_mode="floor").double(), C)
        prev = cur
    return [C, prev, rounds]
