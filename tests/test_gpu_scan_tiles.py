"""Matrix-core scan, every query tile (32, 64, 128, 256, several of 256) and store type: odd and even numbers of k-blocks, a
bank that ends inside a block of rows, enough tiles for the filtering passes, masked and plain, against the oracle."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import _check_masked, _make_bank, _unit

pytestmark = pytest.mark.gpu
DT = {"f32": 0, "bf16": 1, "f16": 2}


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype,N,d,nq", [
    ("f32", 60017, 136, 9), ("f32", 60001, 64, 40), ("f32", 50031, 72, 100), ("f32", 40007, 136, 150), ("f32", 30011, 64, 300),
    ("bf16", 90113, 64, 20), ("bf16", 70001, 136, 50), ("bf16", 60015, 192, 70), ("bf16", 40009, 320, 129), ("bf16", 30029, 64, 513),
    ("f16", 90117, 72, 31), ("f16", 70000, 64, 64), ("f16", 50016, 264, 128), ("f16", 40013, 64, 256), ("f16", 30033, 136, 257)])
def test_every_query_tile_matches_oracle(orc, dtype, N, d, nq, masked):
    rng = np.random.default_rng([43, N, nq])
    rows = _unit(rng, N, d) * rng.uniform(0.5, 2.0, (N, 1)).astype(np.float32)
    rows[N - 1] = rows[300]                                          # an exact tie, one copy in the last row
    q = _unit(rng, nq, d)
    q[nq - 1] = rows[300]
    q[:4] = _unit(rng, 1, d) + 0.05 * _unit(rng, 4, d)               # queries that keep the same rows: several in one lane
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    k1, k2 = 100, 8
    print(f"tiles {dtype} N={N} d={d} B={nq} masked={masked}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    if masked:
        tags = rng.choice(4, N, p=[0.55, 0.3, 0.13, 0.02]).astype(np.uint32) | (rng.integers(0, 40, N).astype(np.uint32) << 8)
        bank.set_tags(0, torch.from_numpy(tags.astype(np.int64)))
        allow = rng.choice([0b0001, 0b0011, 0b0100, 0b1111], nq).astype(np.uint32)
        exclude = np.where(rng.random(nq) < 0.5, rng.integers(0, 40, nq), 0xffffffff).astype(np.uint32)
        _check_masked(orc, bank, dtype, rows, q, tags, allow, exclude, qtab, 1, k1, k2, 0.5)
    else:
        got = parity.gpu_retrieve(bank, torch, q, 1, k1, k2, 0.5)
        parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[1], k1, k2, 0.5, got)
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()
