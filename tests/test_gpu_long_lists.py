"""Pools of more than 256 with two survivor lists to a query (while three quarters of the lists would lie idle) and with one, masked
and plain, lists of many lengths, against the oracle; and a list of either size that overflows."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import _check_masked, _make_bank, _unit

pytestmark = pytest.mark.gpu
DT = {"f32": 0, "bf16": 1, "f16": 2}


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype,N,d,nq,k1", [
    ("f32", 20011, 72, 1, 257), ("f32", 60001, 64, 64, 960), ("bf16", 60017, 64, 64, 300), ("bf16", 60017, 64, 65, 300), ("f16", 16385, 136, 3, 2048),
    ("f16", 100003, 64, 33, 1024), ("bf16", 500, 64, 2, 2048)])
def test_large_pools_match_oracle(orc, dtype, N, d, nq, k1, masked):
    rng = np.random.default_rng([53, N, nq])
    rows = _unit(rng, N, d)
    q = _unit(rng, nq, d)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"long lists {dtype} N={N} d={d} B={nq} k1={k1} masked={masked}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    if masked:
        tags = rng.choice(4, N, p=[0.55, 0.3, 0.13, 0.02]).astype(np.uint32) | (rng.integers(0, 40, N).astype(np.uint32) << 8)
        bank.set_tags(0, torch.from_numpy(tags.astype(np.int64)))
        allow = rng.choice([0b0001, 0b0011, 0b0100, 0b1111], nq).astype(np.uint32)
        exclude = np.where(rng.random(nq) < 0.5, rng.integers(0, 40, nq), 0xffffffff).astype(np.uint32)
        _check_masked(orc, bank, dtype, rows, q, tags, allow, exclude, qtab, 1, k1, 8, 0.5)
    else:
        got = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
        parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[1], k1, 8, 0.5, got)
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()


@pytest.mark.parametrize("nq", [2, 65])
def test_an_overflowing_list_is_flagged_and_answered_exactly(orc, nq):
    rng = np.random.default_rng([54, nq])
    v = _unit(rng, 1, 128)
    rows = np.concatenate([np.repeat(v, 40000, axis=0), _unit(rng, 4000, 128)])[rng.permutation(44000)]
    q = np.concatenate([v, _unit(rng, nq - 1, 128)])
    qtab = rng.uniform(-1, 1, (2, 44000)).astype(np.float32)
    print(f"long lists overflow B={nq}", flush=True)
    bank = _make_bank("bf16", rows, qtab, max_B=nq, max_k1=300)
    parity.gpu_retrieve(bank, torch, q, 1, 300, 8, 0.5)
    flags = bank.retrieve_flags(nq).cpu().numpy()
    assert flags[0] == 1
    ids, scores, cand, sims = bank.retrieve_exact(torch.from_numpy(q).to("cuda:0"), 1, 300, 8, 0.5, want_candidates=True)
    copies = np.sort(np.nonzero((rows == v).all(axis=1))[0])[:300]
    assert np.array_equal(cand[0].cpu().numpy(), copies)
    bank.close()
