"""Epsilon-greedy filling of the slots: pools at the edges of the 64 members that a lane holds, slots at the edges of the 64 that are drawn
together, runs of greedy slots over several lanes' members, from none that explore to all, against the oracle."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import DT, _dev, _make_bank, _unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k1,k2", [(1, 1), (63, 63), (64, 64), (65, 65), (256, 1), (256, 200), (256, 256), (300, 65), (1000, 32), (1025, 129), (2048, 2048)])
@pytest.mark.parametrize("eps", [0.0, 0.02, 0.5, 1.0])
def test_slots_match_oracle(orc, k1, k2, eps):
    rng = np.random.default_rng([71, k1, k2, int(100 * eps)])
    N, d, nq = 3000, 64, 5
    rows, q = _unit(rng, N, d), _unit(rng, nq, d)
    qtab = np.tile((rng.permutation(N) / N).astype(np.float32), (2, 1))      # distinct: with lambda 1 the greedy order has no near-ties
    print(f"slots k1={k1} k2={k2} eps={eps}", flush=True)
    bank = _make_bank("bf16", rows, qtab, max_B=nq, max_k1=k1)
    ids, sc, cid, _, ex = (t.cpu().numpy() for t in bank.retrieve_eps(_dev(q), 0, k1, k2, 1.0, eps, 99, 7, want_candidates=True))
    st, qr = orc.round_to_store(rows, DT["bf16"]), orc.round_to_store(q, DT["bf16"])
    for b in range(nq):
        want, w_sc, _, w_ex = orc.rerank_eps(cid[b], orc.sims_of(st, qr[b], cid[b]), qtab[0], 1.0, k2, eps, 99, 7, b)
        assert np.array_equal(ids[b], want) and np.array_equal(ex[b], w_ex), f"query {b}"
        assert np.all(np.abs(sc[b] - w_sc) <= 1e-5 * np.maximum(1.0, np.abs(w_sc)))
    assert bank.counters() == (0, 0)
    bank.close()
