"""Primes that are not 2^54 - delta with a small delta: every kernel has a general
form for them, and the primes that sanns_params_derive gives never take it.  Each
ring degree through encryption, encoding, every mode and schedule, decryption,
gathered calls and the circuit-private form, against the oracle."""
import numpy as np
import pytest

import oracle
from problem import make_problem, oracle_outputs, oracle_query_ct
from test_gathered_gpu import _run as run_gathered
from test_private_gpu import _check_shares, _oracle_rows, _public_keys, _setup

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_02033_amd import clustered, native as nat, stage
    return nat, stage, clustered


def _primes(N, kind):
    if kind == "mixed":  # one of each: the context takes the general forms
        return oracle.rns_primes(N, 1, bits=50) + oracle.rns_primes(N, 1)
    return oracle.rns_primes(N, 2, bits=50)


@pytest.mark.parametrize("kind", ["50-bit", "mixed"])
@pytest.mark.parametrize("N", [1 << k for k in range(4, 15)])
def test_every_degree(mods, N, kind):
    nat, stage, _ = mods
    Q, d, C = 2, 7, 3
    pb = make_problem(N, 2, 25, C * N - 3, d, Q, seed=N, qs=_primes(N, kind))
    work = [(q, k) for q in range(Q) for k in range(C)]
    want, r = oracle_outputs(pb, work, {})
    ctx, db, sk, ct, qids = _setup(nat, stage, pb, digits=True)
    enc = ct.cpu().numpy()
    for q in range(Q):
        assert (enc[q] == oracle_query_ct(pb, q)).all()
    modes = [(nat.SANNS_MODE_PLAIN, 0), (nat.SANNS_MODE_FUSED, 0), (nat.SANNS_MODE_BATCHED, 0)]
    if N >= 64:
        modes += [(nat.SANNS_MODE_FUSED, nat.SANNS_SCHEDULE_MFMA), (nat.SANNS_MODE_FUSED, 22)]
    if N >= 2048:
        modes.append((nat.SANNS_MODE_PERSISTENT, 0))
    for mode, lds in modes:
        ctx.set_schedule(0, 0, lds)
        out, share = stage.Distances(ctx, db, Q, mode=mode).run(ct, pb.key, qids)
        torch.cuda.synchronize()
        ctx.device_status()
        assert (out.cpu().numpy() == want).all(), (mode, lds)
        assert (share.cpu().numpy() == r).all(), (mode, lds)
        ctx.set_schedule()
    one = stage.Distances(ctx, db, 1)  # one query: the split coordinates
    out1, _ = one.run(ct[:1], pb.key, qids[:1])
    assert (out1.cpu().numpy() == want[:C]).all()
    _check_shares(stage, ctx, pb, sk, out, share, work)
    ctx.close()


@pytest.mark.parametrize("N", [256, 2048, 8192, 16384])
@pytest.mark.parametrize("share", [False, True], ids=["points", "shares"])
def test_gathered(mods, N, share):
    nat, stage, _ = mods
    pb = make_problem(N, 2, 25, 2 * N, 5, 2, seed=N + 1, qs=_primes(N, "50-bit"))
    lists = [np.arange(N + 9), np.arange(N, 2 * N - 1)]
    assert run_gathered(nat, stage, pb, share, lists, 5, 0 if share else N + 1) == 3


@pytest.mark.parametrize("N", [64, 2048, 8192, 16384])
def test_private_form(mods, N):
    nat, stage, _ = mods
    pb = make_problem(N, 2, 22, N + 5, 4, 2, seed=N + 2, qs=_primes(N, "50-bit"))
    ctx, db, sk, ct, qids = _setup(nat, stage, pb)
    pks, pkd = _public_keys(stage, ctx, pb, sk, 700)
    b = nat.sanns_flood_bits(ctx.handle)
    out, share = stage.Distances(ctx, db, 2, private=True).run(ct, pb.key, qids, pk=pkd)
    torch.cuda.synchronize()
    ctx.device_status()
    pairs = [divmod(m, db.n_chunks) for m in range(2 * db.n_chunks)]
    want = _oracle_rows(pb, pks, list(enumerate(pairs)), b, {})
    for m, (w_ct, w_r) in want.items():
        assert (out.cpu().numpy()[m] == w_ct).all(), m
        assert (share.cpu().numpy()[m] == w_r).all(), m
    _check_shares(stage, ctx, pb, sk, out, share, pairs)
    ctx.close()
