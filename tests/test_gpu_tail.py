"""Last steps of a retrieve with a query's candidates shared by one to eight workgroups, at the border between the two
orderings (256 and 257), and with a crowded band that the last workgroup to arrive refines, against the oracle."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import DT, _make_bank, _unit

pytestmark = pytest.mark.gpu


# candidates of 96 KB and less stay with one workgroup; 8 x 96 KB and more go to eight of them (few queries)
@pytest.mark.parametrize("near", [0, 3000])
@pytest.mark.parametrize("dtype,d,nq,k1", [
    ("bf16", 64, 2, 16), ("bf16", 512, 3, 128), ("f32", 520, 2, 128), ("f16", 1544, 5, 256), ("bf16", 1536, 2, 257), ("f32", 1024, 64, 64)])
def test_shared_candidates(orc, dtype, d, nq, k1, near):
    rng = np.random.default_rng([71, d, nq, k1])
    v = _unit(rng, 1, d)
    rows = _unit(rng, 6000, d)
    if near:
        x = v + np.float32(0.001) * rng.standard_normal((near, d)).astype(np.float32) * rng.uniform(0, 1, (near, 1)).astype(np.float32)
        rows = np.concatenate([x, rows[near:]])[rng.permutation(6000)]
        rows = (rows / np.linalg.norm(rows, axis=1, keepdims=True)).astype(np.float32)
    q = np.concatenate([v, _unit(rng, nq - 1, d)])
    qtab = rng.uniform(-1, 1, (2, 6000)).astype(np.float32)
    print(f"tail {dtype} d={d} B={nq} k1={k1} near={near}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    stored, qr = orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype])
    first = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
    o_ids, o_sims = orc.recall(stored, qr, k1, threads=8)
    stats = parity.check_retrieve(orc, stored, qr, qtab[1], k1, 8, 0.5, first, ora_recall=(o_ids, o_sims))
    if near:                                                        # every candidate ties by the bound above: here the bound is an fp32 similarity's resolution
        band = (orc.sims_of(stored, qr[0], np.arange(6000, dtype=np.int32)) > o_sims[0, k1 - 1] - 2e-5).sum()
        assert band > (512 if k1 <= 256 else k1 + 256)               # the case is what it claims to be
        for b in range(nq):
            only = sorted(set(first["cand_ids"][b].tolist()) - set(o_ids[b].tolist()))
            assert not only or np.all(orc.sims_of(stored, qr[b], np.array(only, np.int32)) > o_sims[b, k1 - 1] - 3e-7), b
    else:
        assert stats["boundary_swaps"] == 0 and stats["final_swaps"] == 0, stats
    again = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
    assert all(np.array_equal(first[k], again[k]) for k in ("ids", "scores", "cand_ids", "cand_sims"))
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()


# The crowded band with one to eight workgroups per query, by rows that differ by a fraction of the scan's margin.  Shared
# through the survivor lists that a call leaves unused, or, with the built-in scratch's 64 lists and more than 32 queries, by the
# last workgroup alone; bands of one and of several pieces of ids; the crowded query first, in the middle and last.
CROWDED = [
    ("f32", 136, 2, 200, 2200, 1), ("bf16", 512, 3, 128, 3000, 0), ("f16", 2040, 33, 250, 5000, 32), ("f32", 1024, 64, 64, 900, 20),
    ("f32", 520, 1, 256, 7900, 0), ("bf16", 64, 130, 16, 4100, 77), ("f32", 520, 3, 257, 7900, 2), ("bf16", 1536, 2, 960, 6000, 1)]


@pytest.mark.parametrize("dtype,d,nq,k1,near,at,static", [c + (False,) for c in CROWDED] + [c + (True,) for c in CROWDED if c[2] <= 64 and c[3] <= 256])
def test_crowded_band_is_refined(orc, dtype, d, nq, k1, near, at, static):
    rng = np.random.default_rng([72, d, nq, k1])
    N = 9000
    v = _unit(rng, 1, d)
    rows = _unit(rng, N, d)
    step = np.float32({"f32": 2e-4, "f16": 5e-4, "bf16": 1e-3}[dtype] * (512 / d) ** 0.5)
    x = v + step * rng.standard_normal((near, d)).astype(np.float32) * rng.uniform(0.2, 1, (near, 1)).astype(np.float32)
    where = np.sort(rng.permutation(N)[:near])
    rows[where] = x / np.linalg.norm(x, axis=1, keepdims=True)
    q = _unit(rng, nq, d)
    q[at] = v[0] + (np.float32(0.02) * _unit(rng, 1, d)[0] if dtype == "f32" else 0)     # fp32: similarities that spread over the band
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    stored, qr = orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype])
    ids, sims = orc.recall(stored, qr, k1, threads=8)
    kth = sims[at, k1 - 1]
    band = (orc.sims_of(stored, qr[at], np.arange(N, dtype=np.int32)) > kth - 2e-5).sum()
    print(f"crowded tail {dtype} d={d} B={nq} k1={k1} near={near}: {band} in the band, pool over {sims[at, 0] - kth:.1e}", flush=True)
    assert band > (512 if k1 <= 256 else k1 + 256)                   # the case is what it claims to be
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    for _ in range(2):
        if static:
            out = (torch.empty((nq, 8), dtype=torch.int32, device="cuda:0"), torch.empty((nq, 8), device="cuda:0"),
                   torch.empty((nq, k1), dtype=torch.int32, device="cuda:0"), torch.empty((nq, k1), device="cuda:0"))
            bank.retrieve_static(torch.from_numpy(q).to("cuda:0"), 1, k1, 8, 0.5, out)
            torch.cuda.synchronize()
            got = dict(zip(("ids", "scores", "cand_ids", "cand_sims"), (t.cpu().numpy() for t in out)))
        else:
            got = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
        for b in range(nq):
            only = sorted(set(got["cand_ids"][b].tolist()) - set(ids[b].tolist()))
            if only:        # the selection ranks by similarities rounded to fp32 when the band stays crowded: two roundings of 6e-8
                assert np.all(orc.sims_of(stored, qr[b], np.array(only, np.int32)) > sims[b, k1 - 1] - 3e-7), b
        stats = parity.check_retrieve(orc, stored, qr, qtab[1], k1, 8, 0.5, got, ora_recall=(ids, sims))
        if (orc.sims_of(stored, qr[at], np.arange(N, dtype=np.int32)) > kth - 4e-7).sum() <= (512 if k1 <= 256 else k1 + 256):
            assert stats["boundary_swaps"] == 0, stats                # what ties in fp32 was ordered in fp64
        assert stats["order_swaps"] == 0 and stats["final_swaps"] == 0, stats
    assert not bank.retrieve_flags(nq).cpu().numpy().any()
    bank.close()


# Edges of what a workgroup's rows and lanes are: pools of 16, 32 and 64 rows and one more (64, 32 and 16 lanes to a row, then two
# rows to a lane group), rows shorter than a lane group's reach and of every remainder, the longest rows with the largest pool,
# and lists whose lengths lie around multiples of the 1024 keys a selection takes at a time.
@pytest.mark.parametrize("dtype,N,d,nq,k1", [
    ("f32", 1023, 8, 1, 1), ("f32", 1025, 72, 2, 16), ("bf16", 2048, 8, 3, 17), ("f16", 2049, 136, 1, 32), ("bf16", 3073, 200, 2, 33),
    ("f32", 4096, 328, 1, 64), ("f16", 5121, 520, 130, 65), ("bf16", 6143, 1032, 2, 129), ("f16", 8191, 2056, 1, 256), ("f32", 7169, 520, 1, 257),
    ("bf16", 2500, 16384, 1, 2048), ("f32", 1100, 16384, 2, 40), ("f16", 900, 72, 300, 100), ("f32", 40, 64, 3, 64)])
def test_rows_and_lanes_of_the_scoring(orc, dtype, N, d, nq, k1):
    rng = np.random.default_rng([73, N, d])
    rows = _unit(rng, N, d) * rng.uniform(0.5, 2.0, (N, 1)).astype(np.float32)
    q = _unit(rng, nq, d)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"scoring {dtype} N={N} d={d} B={nq} k1={k1}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    k2 = min(k1, 8)
    got = parity.gpu_retrieve(bank, torch, q, 1, k1, k2, 0.5)
    parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[1], k1, k2, 0.5, got)
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()


# Copies of a row have the same similarity bit for bit, whichever workgroup scored them and however many rows it had: fp32 rows,
# whose products round in fp64.  66 and 130 candidates over four workgroups are 17 and 16, 33 and 32 rows to one, so that they share out
# their lanes differently; the cut lies between two copies.
@pytest.mark.parametrize("d,nq,k1", [(1024, 64, 65), (1032, 64, 129), (2056, 30, 65)])
def test_copies_tie_across_workgroups(orc, d, nq, k1):
    rng = np.random.default_rng([74, d, k1])
    N, distinct = 6000, (k1 + 1) // 2
    v = _unit(rng, 1, d)
    rows = _unit(rng, N, d)
    where = rng.permutation(N)[:2 * distinct].reshape(distinct, 2)
    x = v + _unit(rng, distinct, d) * np.linspace(0.1, 0.9, distinct, dtype=np.float32)[:, None]
    rows[where[:, 0]] = rows[where[:, 1]] = x * rng.uniform(0.5, 2.0, (distinct, 1)).astype(np.float32)
    q = (v + 0.05 * _unit(rng, nq, d)).astype(np.float32)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"copies d={d} B={nq} k1={k1}", flush=True)
    bank = _make_bank("f32", rows, qtab, max_B=2 * nq, max_k1=k1)
    got = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
    stats = parity.check_retrieve(orc, rows, q, qtab[1], k1, 8, 0.5, got)
    assert stats["boundary_swaps"] == 0 and stats["order_swaps"] == 0 and stats["final_swaps"] == 0, stats
    for b in (0, nq // 2, nq - 1):                                   # a query's pool does not depend on the queries it comes with
        alone = parity.gpu_retrieve(bank, torch, q[b:b + 1], 1, k1, 8, 0.5)
        assert np.array_equal(alone["ids"][0], got["ids"][b]) and np.array_equal(alone["cand_ids"][0], got["cand_ids"][b]), b
    bank.close()


# A crowded band of copies that ends in a short piece of ids (2304 to a piece).
@pytest.mark.parametrize("nq,k1,near", [(64, 256, 2310), (6, 960, 2324), (130, 100, 2318)])
def test_copies_tie_across_pieces_of_a_crowded_band(orc, nq, k1, near):
    rng = np.random.default_rng([75, nq, k1])
    N, d = 9000, 1024
    v = _unit(rng, 1, d)
    rows = _unit(rng, N, d)
    x = v + np.float32(1.4e-4) * rng.standard_normal((near // 2, d)).astype(np.float32) * rng.uniform(0.2, 1, (near // 2, 1)).astype(np.float32)
    where = rng.permutation(N)[:near].reshape(near // 2, 2)
    rows[where[:, 0]] = rows[where[:, 1]] = x / np.linalg.norm(x, axis=1, keepdims=True)
    q = (v + np.float32(0.01) * _unit(rng, nq, d)).astype(np.float32)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    ids, sims = orc.recall(rows, q, k1, threads=8)
    spread = max(sims[b, k1 - 1] - orc.sims_of(rows, q[b], where.reshape(-1).astype(np.int32)).min() for b in range(nq))
    print(f"crowded copies B={nq} k1={k1} near={near}: down to {spread:.1e} below the pool", flush=True)
    assert spread < 1.2e-4                                           # every one of them lies within the scan's margin: the case is what it claims to be
    bank = _make_bank("f32", rows, qtab, max_B=2 * nq, max_k1=k1)
    got = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
    parity.check_retrieve(orc, rows, q, qtab[1], k1, 8, 0.5, got, ora_recall=(ids, sims))
    twin = dict(zip(where[:, 0].tolist(), where[:, 1].tolist())) | dict(zip(where[:, 1].tolist(), where[:, 0].tolist()))
    for b in range(nq):                                              # the pool is cut at equal fp32 roundings by id, so a copy's lower id is in it if the other is
        at = {int(i): j for j, i in enumerate(got["cand_ids"][b])}
        for i, j in at.items():
            assert i < twin[i] or at.get(twin[i], k1) < j, (b, i, twin[i])
    bank.close()
