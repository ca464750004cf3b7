"""Matrix-core scan of 16-bit stores with 128 or 256 queries to a tile, whose operands pass through rings in LDS: one to seven k-blocks (a ring
has three places), one and several tiles to a workgroup, one and several query tiles, lists that run full, against the oracle."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import _make_bank, _unit

pytestmark = pytest.mark.gpu
DT = {"bf16": 1, "f16": 2}


@pytest.mark.parametrize("dtype,N,d,nq,k1", [
    ("bf16", 200003, 64, 130, 64),                  # a k-block to a tile; three tiles to a workgroup
    ("f16", 190001, 128, 256, 100), ("bf16", 150017, 192, 200, 64), ("f16", 100003, 256, 129, 33), ("bf16", 90001, 320, 256, 64),
    ("f16", 70001, 384, 250, 16), ("bf16", 60013, 448, 131, 128),
    ("bf16", 140009, 72, 700, 64), ("f16", 80021, 200, 1024, 32),    # three and four query tiles on shared bank tiles
    ("bf16", 30011, 64, 256, 256),                  # many survivors to a tile: a list has room for a part
    ("f16", 8193, 64, 300, 8),                     # the filtering pass is one row
    ("bf16", 120011, 64, 65, 64), ("f16", 90001, 192, 128, 256), ("bf16", 50021, 328, 100, 17), ("f16", 60001, 448, 97, 64)])   # 128 queries to a tile
def test_operand_rings_match_oracle(orc, dtype, N, d, nq, k1):
    rng = np.random.default_rng([47, N, nq])
    rows = _unit(rng, N, d) * rng.uniform(0.5, 2.0, (N, 1)).astype(np.float32)
    q = _unit(rng, nq, d)
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"ring {dtype} N={N} d={d} B={nq} k1={k1}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    got = parity.gpu_retrieve(bank, torch, q, 0, k1, 8, 0.5)
    parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[0], k1, 8, 0.5, got)
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()
