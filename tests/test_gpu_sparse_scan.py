"""The scans of sparse passes: edges of the query tiles (16, 32, 64; up to 4 queries on fp32 rows), of the bank's tiles, of
the k dimension's split over eight wavefronts, masks, one pass and several, against the oracle."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import _check_masked, _make_bank, _unit

pytestmark = pytest.mark.gpu
DT = {"f32": 0, "bf16": 1, "f16": 2}


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype,N,d,nq", [
    ("bf16", 1, 8, 1), ("f16", 255, 64, 16), ("f32", 257, 72, 17), ("bf16", 8192, 320, 32), ("f16", 8193, 200, 33),
    ("f32", 9001, 520, 64), ("bf16", 16641, 1032, 65), ("f16", 16385, 2056, 7), ("f32", 30011, 136, 9), ("bf16", 30000, 192, 129),
    ("f32", 257, 72, 1), ("f32", 9001, 328, 2), ("f32", 20003, 136, 4)])
def test_sparse_passes_match_oracle(orc, dtype, N, d, nq, masked):
    rng = np.random.default_rng([41, N, nq])
    rows = _unit(rng, N, d) * rng.uniform(0.5, 2.0, (N, 1)).astype(np.float32)
    rows[N - 1] = rows[0]                                            # an exact tie, one copy in the last row
    q = _unit(rng, nq, d)
    q[nq - 1] = rows[0]
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    k1, k2 = 64, 8
    print(f"sparse {dtype} N={N} d={d} B={nq} masked={masked}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    if masked:
        tags = rng.choice(4, N, p=[0.55, 0.3, 0.13, 0.02]).astype(np.uint32) | (rng.integers(0, 40, N).astype(np.uint32) << 8)
        bank.set_tags(0, torch.from_numpy(tags.astype(np.int64)))
        allow = rng.choice([0b0001, 0b0011, 0b0100, 0b1111, 0b1000, 0], nq).astype(np.uint32)
        exclude = np.where(rng.random(nq) < 0.5, rng.integers(0, 40, nq), 0xffffffff).astype(np.uint32)
        _check_masked(orc, bank, dtype, rows, q, tags, allow, exclude, qtab, 1, k1, k2, 0.5)
    else:
        got = parity.gpu_retrieve(bank, torch, q, 1, k1, k2, 0.5)
        stats = parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[1], k1, k2, 0.5, got)
        assert stats["boundary_swaps"] == 0 and stats["final_swaps"] == 0
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()


@pytest.mark.parametrize("dtype,N,d,nq", [
    ("f32", 300, 8, 1), ("f32", 9001, 328, 3), ("f32", 8191, 136, 4), ("f32", 5000, 72, 5), ("bf16", 257, 8, 1), ("bf16", 12000, 200, 16),
    ("f16", 8193, 136, 7), ("f16", 70, 1032, 15), ("bf16", 9000, 64, 17)])
def test_queries_at_any_address(orc, dtype, N, d, nq):
    """Few queries at a multiple of 16 bytes are read as given by the first pass, which prepares them for the others on the
    way; at another address a launch of its own does.  Both give the oracle's result."""
    rng = np.random.default_rng([47, N, nq])
    rows = _unit(rng, N, d)
    q = _unit(rng, nq, d) * rng.uniform(0.1, 9.0, (nq, 1)).astype(np.float32)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    k1 = min(N, 64)
    print(f"addresses {dtype} N={N} d={d} B={nq}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    room = torch.zeros(nq * d + 1, device="cuda:0")
    room[1:] = torch.from_numpy(q).to("cuda:0").view(-1)
    odd = room[1:].view(nq, d)
    assert odd.data_ptr() % 16 == 4
    results = []
    for queries in (torch.from_numpy(q).to("cuda:0"), odd):
        ids, scores, cand, sims = bank.retrieve(queries, 1, k1, 8, 0.5, want_candidates=True)
        got = {"ids": ids.cpu().numpy(), "scores": scores.cpu().numpy(), "cand_ids": cand.cpu().numpy(), "cand_sims": sims.cpu().numpy()}
        parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[1], k1, 8, 0.5, got)
        results.append(got)
    assert all(np.array_equal(results[0][k], results[1][k]) for k in results[0])
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()


@pytest.mark.parametrize("scale", [1e-24, 1e-20, 1e22])
@pytest.mark.parametrize("dtype,N,d,nq", [("f32", 20000, 72, 1), ("f32", 60000, 328, 4), ("f32", 20000, 136, 7), ("bf16", 20000, 64, 1), ("bf16", 60000, 200, 16)])
def test_queries_of_any_norm(orc, dtype, N, d, nq, scale):
    """Queries whose squares a float does not hold, over banks of several passes: a similarity does not depend on the query's norm."""
    rng = np.random.default_rng([48, N, nq])
    rows = _unit(rng, N, d)
    q = (_unit(rng, nq, d) * rng.uniform(0.5, 2.0, (nq, 1)) * scale).astype(np.float32)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"norms {dtype} N={N} d={d} B={nq} scale={scale}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=64)
    stored, qr = orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype])
    room = torch.zeros(nq * d + 1, device="cuda:0")
    room[1:] = torch.from_numpy(q).to("cuda:0").view(-1)
    for queries in (torch.from_numpy(q).to("cuda:0"), room[1:].view(nq, d)):
        ids, scores, cand, sims = bank.retrieve(queries, 1, 64, 8, 0.5, want_candidates=True)
        got = {"ids": ids.cpu().numpy(), "scores": scores.cpu().numpy(), "cand_ids": cand.cpu().numpy(), "cand_sims": sims.cpu().numpy()}
        stats = parity.check_retrieve(orc, stored, qr, qtab[1], 64, 8, 0.5, got)
        assert stats["boundary_swaps"] == 0 and stats["final_swaps"] == 0
        assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()
