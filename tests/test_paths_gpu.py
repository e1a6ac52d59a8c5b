"""The launch rules' branches at the sizes where they change: many transforms of
each ring degree against the persistent launch, one query against few chunks
with the coordinates split over a workgroup's waves, the matrix-core schedule's
row tiles of 16, 32 and 64, point rows gathered 16, 4 or 1 bytes at a time,
decryption in batches, seeded encryption under primes away from 2^54, and the
k-means kernels at the edges of their tiles.  Every value is an integer:
equality throughout."""
import numpy as np
import pytest

import oracle
from oracle import balance as obal

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_02033_amd import native as nat, stage
    return nat, stage


def _dev(x, dtype=None):
    t = torch.as_tensor(np.ascontiguousarray(x))
    return (t.to(dtype) if dtype is not None else t).cuda()


def _ctx(nat, stage, N, qs, t, flags=0):
    p = nat.sanns_params()
    p.N, p.L, p.t = N, len(qs), t
    for l, q in enumerate(qs):
        p.q[l] = q
    p.flags = nat.SANNS_FLAG_INSECURE_TEST | flags
    return stage.Context(params=p)


def _seeded(nat, stage, N, L, n, d, Q, seed, flags=0):
    """A context, an encoded database and seeded queries, all on the device."""
    qs, t = oracle.rns_primes(N, L), oracle.plain_modulus(N, 27)
    ctx = _ctx(nat, stage, N, qs, t, flags)
    g = np.random.default_rng(seed)
    pts = g.integers(0, 256, (n, d)).astype(np.uint8)
    que = g.integers(0, 256, (Q, d)).astype(np.uint8)
    slot = stage.linear_slot_map(n, N, g.permutation(n))
    db = stage.encode_db(ctx, pts, slot)
    sk = stage.keygen(ctx, seed)
    ct = stage.encrypt_query_seeded(ctx, sk, _dev(que.astype(np.int32)), seed + 1)
    ids = _dev(np.arange(Q, dtype=np.uint64) + np.uint64(seed))
    return ctx, db, sk, ct, ids, pts, que, slot


def _run(stage, ctx, db, ct, ids, mode, schedule=(0, 0)):
    ctx.set_schedule(*schedule)
    out, share = stage.Distances(ctx, db, ct.shape[0], mode=mode).run(ct, b"k" * 32, ids)
    torch.cuda.synchronize()
    ctx.device_status()
    ctx.set_schedule()
    return out, share


def _check_distances(stage, ctx, sk, out, share, pts, que, slot, C):
    qn = (que.astype(np.int64) ** 2).sum(1) % ctx.t
    client = stage.decrypt_shares(ctx, sk, out, _dev(np.repeat(qn, C).astype(np.uint32)))
    tot = (client.cpu().numpy().astype(np.int64) + share.cpu().numpy()) % ctx.t
    for m in range(len(tot)):
        ids = slot[m % C * ctx.N:(m % C + 1) * ctx.N]
        real = ids >= 0
        assert (tot[m][real] == oracle.sqdist(que[m // C], pts[ids[real]])).all(), m


# about a thousand polynomials and more in each direction; the persistent form
# takes them from its own work queue
@pytest.mark.parametrize("N,L,Q,d,C", [(4096, 2, 8, 33, 33), (8192, 3, 8, 23, 22),
                                       (16384, 4, 7, 19, 19), (4096, 2, 8, 31, 31)])
def test_many_transforms(mods, N, L, Q, d, C):
    nat, stage = mods
    ctx, db, sk, ct, ids, pts, que, slot = _seeded(nat, stage, N, L, C * N - 5, d, Q, 10 + d)
    out, share = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED)
    po, psh = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_PERSISTENT)
    assert torch.equal(out.view(torch.int64), po.view(torch.int64))
    assert torch.equal(share.view(torch.int32), psh.view(torch.int32))
    _check_distances(stage, ctx, sk, out, share, pts, que, slot, C)


@pytest.mark.parametrize("N,L", [(64, 1), (256, 2), (4096, 2), (8192, 3)])
@pytest.mark.parametrize("d", [1, 3, 4, 5, 130, 1013])
def test_split_coordinates_one_query(mods, N, L, d):
    nat, stage = mods
    for C in (1, 3, 9) if d < 1000 else (2,):
        ctx, db, sk, ct, ids, pts, que, slot = _seeded(nat, stage, N, L, C * N - 3, d, 1, d + C)
        out, share = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED)
        go, gs = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED, (1, 1))
        assert torch.equal(out.view(torch.int64), go.view(torch.int64)), (d, C)
        assert torch.equal(share.view(torch.int32), gs.view(torch.int32))
        if L > 1:  # (one 54-bit prime does not hold the noise)
            _check_distances(stage, ctx, sk, out, share, pts, que, slot, C)
        ctx.close()


# queries at both sides of each row tile, chunks at both sides of a column tile,
# contractions of 32, 64, 96 and 128 coordinates (ragged ones too)
@pytest.mark.parametrize("Q", [2, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("d", [5, 32, 50, 96, 128])
def test_row_tiles(mods, Q, d):
    nat, stage = mods
    N, L = 256, 2
    for C in (3, 65):
        ctx, db, sk, ct, ids, pts, que, slot = _seeded(nat, stage, N, L, C * N - 9, d, Q, Q + d,
                                                       nat.SANNS_FLAG_DIGIT_DB)
        want = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED, (0, 0, 22))
        for mode in (nat.SANNS_MODE_FUSED, nat.SANNS_MODE_BATCHED):
            for lds in (nat.SANNS_SCHEDULE_MFMA, 0):  # forced, and as the model chooses
                got = _run(stage, ctx, db, ct, ids, mode, (0, 0, lds))
                assert torch.equal(got[0].view(torch.int64), want[0].view(torch.int64)), (C, lds)
                assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
        _check_distances(stage, ctx, sk, *got, pts, que, slot, C)
        ctx.close()


@pytest.mark.parametrize("dtype", [np.uint8, np.int8])
@pytest.mark.parametrize("d", [7, 20, 32])
def test_gather_widths(mods, d, dtype):
    """Rows at every alignment give the same database, padding slots too."""
    nat, stage = mods
    N, n = 256, 700
    ctx = _ctx(nat, stage, N, oracle.rns_primes(N, 2), oracle.plain_modulus(N, 27))
    g = np.random.default_rng(d)
    pts = g.integers(np.iinfo(dtype).min, np.iinfo(dtype).max + 1, (n, d)).astype(dtype)
    slot = np.full(3 * N, -1, dtype=np.int64)
    slot[g.permutation(3 * N)[:n]] = np.arange(n)
    used = 2 * 3 * d * N * 8 + 3 * N * 4
    want = None
    for off in (0, 4, 1):
        buf = torch.zeros(n * d + 16, dtype=torch.uint8, device="cuda")
        view = buf[off:off + n * d]
        view.copy_(torch.as_tensor(pts.view(np.uint8).reshape(-1)))
        db = stage.encode_db(ctx, view.view(torch.int8 if dtype == np.int8 else torch.uint8)
                             .view(n, d), slot)
        mem = db.mem[:used].cpu()
        assert want is None or torch.equal(mem, want), off
        want = mem
    norms = want[-3 * N * 4:].numpy().view(np.uint32)
    ref = np.where(slot >= 0, (pts.astype(np.int64) ** 2).sum(1)[np.maximum(slot, 0)], 0)
    assert (norms == ref).all()


def test_decrypt_batches(mods):
    """1,025 ciphertexts of 64 KiB residues: one more than a batch holds."""
    nat, stage = mods
    N, L, M = 4096, 2, 1025
    qs = oracle.rns_primes(N, L)
    ctx = _ctx(nat, stage, N, qs, oracle.plain_modulus(N, 25))
    sk = stage.keygen(ctx, 3)
    ct = torch.randint(0, min(qs), (M, 2, L, N), device="cuda").view(torch.uint64)
    qn = torch.arange(M, dtype=torch.int32, device="cuda").view(torch.uint32)
    got = stage.decrypt_shares(ctx, sk, ct, qn).cpu().numpy()
    for m in (0, 511, 1023, 1024):
        one = ct.view(torch.int64)[m:m + 1].contiguous().view(torch.uint64)
        alone = stage.decrypt_shares(ctx, sk, one, qn.view(torch.int32)[m:m + 1].view(torch.uint32))
        assert (alone.cpu().numpy()[0] == got[m]).all(), m


def test_seeded_encryption_general_primes(mods):
    nat, stage = mods
    N, Q, d = 4096, 2, 3
    qs = oracle.rns_primes(N, 1, bits=50) + oracle.rns_primes(N, 1)
    P = oracle.Params(N, qs, oracle.plain_modulus(N, 25))
    ctx = _ctx(nat, stage, N, qs, P.t)
    sk = stage.keygen(ctx, 5)
    msgs = np.arange(Q * d, dtype=np.int32).reshape(Q, d) - 2
    ct = stage.encrypt_query_seeded(ctx, sk, _dev(msgs), 77).cpu().numpy()
    s = oracle.sample_secret(5, N)
    a, e = oracle.sample_encryption(P, 77, Q, d)
    for q in range(Q):
        want = oracle.encrypt_constants(P, s, a[q], e[q], [int(x) for x in msgs[q]])
        assert (ct[q] == want).all()


@pytest.mark.parametrize("d", [1, 31, 33, 64, 65, 96, 97, 128, 160, 255, 256])
@pytest.mark.parametrize("n,k", [(1, 1), (255, 15), (257, 16), (300, 65), (513, 129)])
def test_kmeans_tile_edges(mods, n, d, k):
    """Extreme coordinates and centres (the largest norms and products),
    duplicate centres (ties), odd d (bytes and word rows)."""
    nat, _ = mods
    g = np.random.default_rng(n + d + k)
    X = g.integers(-128, 128, (n, d)).astype(np.int8)
    X[0], X[-1] = -128, 127
    C = g.integers(-128 * 256, 127 * 256 + 1, (k, d)).astype(np.int32)
    C[0] = -128 * 256
    if k > 2:
        C[k - 1], C[k // 2] = 127 * 256, C[0]
    Xd, Cd = _dev(X), _dev(C)
    ws = torch.empty(nat.sanns_kmeans_workspace(k, d), dtype=torch.uint8, device="cuda")
    a = torch.empty(n, dtype=torch.int32, device="cuda")
    nat.sanns_kmeans_assign(Xd.data_ptr(), n, d, Cd.data_ptr(), k, 0, a.data_ptr(), 0,
                            ws.data_ptr(), ws.numel(), 0)
    want = obal.assign(X, C)
    assert (a.cpu().numpy() == want).all()
    nat.sanns_kmeans_update(Xd.data_ptr(), n, d, a.data_ptr(), k, Cd.data_ptr(), 0,
                            ws.data_ptr(), ws.numel(), 0)
    assert (Cd.cpu().numpy() == obal.update(X, want, C)).all()


# sums gathered in LDS tables of 8, 4 and 2 coordinate pairs, at both sides of
# each table's largest k and of n = 64 k; d odd and one slice short
@pytest.mark.parametrize("k", [1, 40, 2258, 2260, 4265, 4267, 7679, 7682])
@pytest.mark.parametrize("extra", [-1, 0, 777])
def test_kmeans_update_tables(mods, k, extra):
    nat, _ = mods
    n, d = max(64 * k, 20000) + extra, 33
    g = torch.Generator(device="cuda").manual_seed(k + extra)
    X = torch.randint(-128, 128, (n, d), dtype=torch.int8, device="cuda", generator=g)
    a = torch.randint(-1, k + 1, (n,), dtype=torch.int32, device="cuda", generator=g)
    C = torch.full((k, d), 7, dtype=torch.int32, device="cuda")
    cnt = torch.empty(k, dtype=torch.int64, device="cuda")
    ws = torch.empty(nat.sanns_kmeans_workspace(k, d), dtype=torch.uint8, device="cuda")
    nat.sanns_kmeans_update(X.data_ptr(), n, d, a.data_ptr(), k, C.data_ptr(), cnt.data_ptr(),
                            ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    x, lab = X.cpu().numpy().astype(np.int64), a.cpu().numpy()
    real = (lab >= 0) & (lab < k)
    c = np.bincount(lab[real], minlength=k)
    s = np.stack([np.bincount(lab[real], weights=x[real, i], minlength=k) for i in range(d)], 1)
    want = np.where(c[:, None] > 0, (512 * s.astype(np.int64) + c[:, None]) //
                    np.maximum(2 * c[:, None], 1), 7)
    assert (cnt.cpu().numpy() == c).all() and (C.cpu().numpy() == want).all()


@pytest.mark.parametrize("n", [(1 << 32) // 255 - 1, (1 << 32) // 255 + 1])
def test_kmeans_update_many_points(mods, n):
    """Both forms of the sums: two coordinates per add, and one where their
    halves could carry; every point of one cluster at the largest coordinate."""
    nat, _ = mods
    d, k = 3, 2
    X = torch.full((n, d), 127, dtype=torch.int8, device="cuda")
    X[0] = -128
    a = torch.zeros(n, dtype=torch.int32, device="cuda")
    C = torch.full((k, d), 7, dtype=torch.int32, device="cuda")
    cnt = torch.empty(k, dtype=torch.int64, device="cuda")
    ws = torch.empty(nat.sanns_kmeans_workspace(k, d), dtype=torch.uint8, device="cuda")
    nat.sanns_kmeans_update(X.data_ptr(), n, d, a.data_ptr(), k, C.data_ptr(), cnt.data_ptr(),
                            ws.data_ptr(), ws.numel(), 0)
    s = 127 * (n - 1) - 128
    assert C[0].tolist() == [(512 * s + n) // (2 * n)] * d and C[1].tolist() == [7] * d
    assert cnt.tolist() == [n, 0]


# the widest rows of each contraction form, those whose sums hold products of two
# shapes (d = 193 .. 224, as 65 .. 96 and 129 .. 160 above) among them
@pytest.mark.parametrize("d", [80, 130, 161, 192, 193, 200, 224, 225])
def test_kmeans_wide_rows(mods, d):
    test_kmeans_tile_edges(mods, 513, d, 129)


# launches on both sides of the largest that take the transforms' form for few
# polynomials (768 of N = 8192, 256 of N = 16384): forward 2 L d, inverse 2 L C,
# encoding L d C
@pytest.mark.parametrize("N,L,d,C", [(8192, 3, 128, 2), (8192, 3, 129, 2), (8192, 3, 2, 128),
                                     (8192, 3, 2, 129), (16384, 2, 64, 2), (16384, 2, 65, 2),
                                     (16384, 2, 2, 64), (16384, 2, 2, 65)])
def test_few_transforms(mods, N, L, d, C):
    nat, stage = mods
    ctx, db, sk, ct, ids, pts, que, slot = _seeded(nat, stage, N, L, C * N - 5, d, 1, d + C)
    out, share = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED)
    po, psh = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_PERSISTENT)
    assert torch.equal(out.view(torch.int64), po.view(torch.int64))
    assert torch.equal(share.view(torch.int32), psh.view(torch.int32))
    _check_distances(stage, ctx, sk, out, share, pts, que, slot, C)
    pk = stage.public_key(ctx, sk, 9).view(torch.int64)[None].contiguous().view(torch.uint64)
    D = stage.Distances(ctx, db, 1, private=True)
    out, share = D.run(ct, b"k" * 32, ids, pk=pk, flood_bits=20)
    torch.cuda.synchronize()
    _check_distances(stage, ctx, sk, out, share, pts, que, slot, C)


# both sides of the lines where one query goes from split coordinates to whole ones
@pytest.mark.parametrize("N,L,d,C", [(8192, 3, 128, 12), (8192, 3, 128, 13), (8192, 3, 16, 8),
                                     (8192, 3, 16, 9), (256, 1, 33, 2560), (256, 1, 33, 2561),
                                     (8192, 3, 40, 24), (8192, 3, 40, 25),
                                     (4096, 2, 128, 56), (4096, 2, 128, 57)])
def test_split_coordinates_line(mods, N, L, d, C):
    nat, stage = mods
    ctx, db, sk, ct, ids, pts, que, slot = _seeded(nat, stage, N, L, C * N - 3, d, 1, d + C)
    out, share = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED)
    go, gs = _run(stage, ctx, db, ct, ids, nat.SANNS_MODE_FUSED, (1, 8))
    assert torch.equal(out.view(torch.int64), go.view(torch.int64))
    assert torch.equal(share.view(torch.int32), gs.view(torch.int32))
    if L > 1:
        _check_distances(stage, ctx, sk, out, share, pts, que, slot, C)


def test_kmeans_centre_blocks(mods):
    """More centres than a packed index holds (2^22): two blocks, whose winners are
    compared in 64 bits; nearest centres in either, and equal ones in both, where the
    lower index wins."""
    nat, _ = mods
    n, d, B = 70, 4, 1 << 22
    k = B + 70
    g = np.random.default_rng(22)
    X = g.integers(-128, 128, (n, d)).astype(np.int8)
    C = g.integers(-128 * 256, 127 * 256 + 1, (k, d)).astype(np.int32)
    for i, js in enumerate([(100, B + 5), (B + 69,), (B - 1, B), (B + 64,), (0, B), (B - 1 - 64,),
                            (B + 3, B + 66)]):
        C[list(js)] = 256 * X[i].astype(np.int32)
    C[B - 1] = 256 * X[2].astype(np.int32)
    C[B] = C[B - 1]
    Xd, Cd = _dev(X), _dev(C)
    ws = torch.empty(nat.sanns_kmeans_workspace(k, d), dtype=torch.uint8, device="cuda")
    a = torch.empty(n, dtype=torch.int32, device="cuda")
    nat.sanns_kmeans_assign(Xd.data_ptr(), n, d, Cd.data_ptr(), k, 0, a.data_ptr(), 0,
                            ws.data_ptr(), ws.numel(), 0)
    c64 = C.astype(np.int64)
    nrm = (c64 * c64).sum(1)
    want = [int(np.argmin(nrm - 512 * (c64 @ x))) for x in X.astype(np.int64)]
    got = a.cpu().numpy().tolist()
    assert got == want
    assert want[:4] == [100, B + 69, B - 1, B + 64] and want[6] == B + 3


@pytest.mark.parametrize("d", [1, 24, 96, 200])
@pytest.mark.parametrize("far", [32640, -32769, 40000, 1 << 20, (1 << 31) - 1, -(1 << 31)])
def test_kmeans_far_centres(mods, d, far):
    """Centres beyond the points' grid (unused slots set far away, say): every int32
    is a coordinate, alone, beside near centres, twice, and in all centres."""
    nat, _ = mods
    n, k = 300, 131
    g = np.random.default_rng(d)
    X = g.integers(-128, 128, (n, d)).astype(np.int8)
    X[0], X[1] = -128, 127
    C = g.integers(-128 * 256, 127 * 256 + 1, (k, d)).astype(np.int64)
    some = C.copy()
    some[[3, 70, 130]] = far
    some[90, d // 2] = far
    every = np.clip(C + far, -(1 << 31), (1 << 31) - 1)
    every[60] = every[5]
    one = np.clip(C[:1] + far, -(1 << 31), (1 << 31) - 1)
    for cen in (some, every, one):
        kk = len(cen)
        Xd, Cd = _dev(X), _dev(cen.astype(np.int32))
        ws = torch.empty(nat.sanns_kmeans_workspace(kk, d), dtype=torch.uint8, device="cuda")
        a = torch.empty(n, dtype=torch.int32, device="cuda")
        prev = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        changed = torch.zeros(1, dtype=torch.int32, device="cuda")
        nat.sanns_kmeans_assign(Xd.data_ptr(), n, d, Cd.data_ptr(), kk, prev.data_ptr(),
                                a.data_ptr(), changed.data_ptr(), ws.data_ptr(), ws.numel(), 0)
        co = cen.astype(object)
        nrm = (co * co).sum(1)
        key = nrm[None, :] - 512 * (X.astype(object) @ co.T)
        want = [int(np.argmin(r)) for r in key]
        assert a.cpu().numpy().tolist() == want
        assert int(changed) == n


# one slot per thread for rows read by bytes, two otherwise
@pytest.mark.parametrize("dtype", [np.uint8, np.int8])
@pytest.mark.parametrize("d", [1, 4, 9, 16, 36, 147])
def test_gather_slots(mods, d, dtype):
    test_gather_widths(mods, d, dtype)


# one and two coordinates apart, three in pairs, each with LDS tables where clusters
# are large
@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("n,k", [(3000, 400), (20000, 3)])
def test_kmeans_update_narrow(mods, n, k, d):
    nat, _ = mods
    g = np.random.default_rng(n + d)
    X = g.integers(-128, 128, (n, d)).astype(np.int8)
    a = g.integers(0, k, n).astype(np.int32)
    C = np.full((k, d), 7, dtype=np.int32)
    Xd, Ad, Cd = _dev(X), _dev(a), _dev(C)
    ws = torch.empty(nat.sanns_kmeans_workspace(k, d), dtype=torch.uint8, device="cuda")
    nat.sanns_kmeans_update(Xd.data_ptr(), n, d, Ad.data_ptr(), k, Cd.data_ptr(), 0,
                            ws.data_ptr(), ws.numel(), 0)
    assert (Cd.cpu().numpy() == obal.update(X, a, C)).all()
