"""Ordering of a pool of more than 256 whose similarities fp32 hardly tells apart (near-duplicates of the query): the order is that of fp64, and it
takes no longer than that of a pool which spreads."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import _dev, _make_bank, _unit

pytestmark = pytest.mark.gpu


def _near(rng, v, n, N, amp):
    d = v.shape[1]
    rows = _unit(rng, N, d)
    x = v + np.float32(amp / d ** 0.5) * rng.standard_normal((n, d)).astype(np.float32) * rng.uniform(0.1, 1, (n, 1)).astype(np.float32)
    rows[rng.permutation(N)[:n]] = x / np.linalg.norm(x, axis=1, keepdims=True)
    return rows


# the pool's similarities spread over one step of fp32, some ten, some thousand and very many (distinct in fp64: ties of sums in another order would be no fault)
@pytest.mark.parametrize("amp", [3e-4, 1e-3, 1e-2, 1e-1])
@pytest.mark.parametrize("near,k1", [(300, 257), (1100, 1000), (2100, 2048)])
def test_order_of_near_duplicates(orc, near, k1, amp):
    rng = np.random.default_rng([91, near])
    N, d, nq = 9000, 256, 3
    v = _unit(rng, 1, d)
    rows, q = _near(rng, v, near, N, amp), np.concatenate([v, _unit(rng, 2, d)])
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"near-duplicates near={near} k1={k1} amp={amp}", flush=True)
    bank = _make_bank("f32", rows, qtab, max_B=nq, max_k1=k1)
    got = parity.gpu_retrieve(bank, torch, q, 0, k1, 8, 0.5)
    parity.check_retrieve(orc, rows, q, qtab[0], k1, 8, 0.5, got)
    # what the pool holds is ordered by the fp64 similarities of its members (2e-16 x 256 terms of the sum: 1e-14)
    sims = orc.sims_of(rows, q[0], got["cand_ids"][0])
    assert np.all(np.diff(sims) <= 1e-14)
    assert not bank.retrieve_flags(nq).cpu().numpy().any()
    bank.close()


def test_near_duplicates_cost_no_more():
    """Banks alike but for how far their near-duplicates spread, in turn: 93 and 43 us while the buckets' range was that of the values rounded to
    fp32, 48 and 43 as it is."""
    rng = np.random.default_rng(93)
    N, d, k1 = 9000, 256, 2048
    v = _unit(rng, 1, d)
    q = _dev(np.repeat(v, 4, 0))
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    banks = [_make_bank("f32", _near(rng, v, 2100, N, amp), qtab, max_B=4, max_k1=k1) for amp in (1e-4, 1e-1)]
    best = [float("inf")] * 2
    for _ in range(12):
        for i, bank in enumerate(banks):
            bank.retrieve(q, 0, k1, 8, 0.5)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                bank.retrieve(q, 0, k1, 8, 0.5)
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b))
    print(f"near-duplicates {best[0] * 50:.1f} us, spread {best[1] * 50:.1f} us", flush=True)
    assert best[0] < 1.4 * best[1], best
    for bank in banks:
        bank.close()
