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
    parity.check_retrieve(orc, stored, qr, qtab[1], k1, 8, 0.5, first)
    again = parity.gpu_retrieve(bank, torch, q, 1, k1, 8, 0.5)
    assert all(np.array_equal(first[k], again[k]) for k in ("ids", "scores", "cand_ids", "cand_sims"))
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()
