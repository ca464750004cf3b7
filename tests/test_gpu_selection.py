"""Selection over lists of every spread that its equal-width first round meets: one outlier far above a narrow band, a few
distinct similarities with many copies each, all equal, evenly spread, against the oracle."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity import DT, _dev, _make_bank, _unit

pytestmark = pytest.mark.gpu


def _rows(kind, rng, N, d, v):
    if kind == "outlier":                   # the query itself, everything else in a band of about 0.01
        x = np.repeat(rng.standard_normal((1, d)), N, axis=0) + 0.02 * rng.standard_normal((N, d))
        x[N // 3] = v[0]
    elif kind == "steps":                   # five distinct rows
        x = rng.standard_normal((5, d))[rng.integers(0, 5, N)]
    elif kind == "equal":
        x = np.repeat(rng.standard_normal((1, d)), N, axis=0)
    else:                                   # similarities evenly spread over [-1, 1]
        w = rng.standard_normal((N, d))
        w -= (w @ v[0])[:, None] * v
        s = np.linspace(-1, 1, N)[rng.permutation(N)][:, None]
        x = s * v + np.sqrt(1 - s * s) * w / np.linalg.norm(w, axis=1, keepdims=True)
    return (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("kind", ["outlier", "steps", "equal", "even"])
@pytest.mark.parametrize("dtype,N,nq,k1", [("f32", 129, 1, 128), ("bf16", 8192, 3, 1), ("f16", 8000, 70, 256), ("f32", 20000, 2, 64)])
def test_lists_of_any_spread(orc, dtype, N, nq, k1, kind):
    rng = np.random.default_rng([61, N, k1])
    d = 64
    v = _unit(rng, 1, d)
    if kind in ("steps", "equal") and N > 8192:
        N = 8100                            # copies past a survivor list's length are lost to a scan by design
    rows = _rows(kind, rng, N, d, v)
    q = np.concatenate([v, _unit(rng, nq, d)])[:nq]
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"selection {kind} {dtype} N={N} B={nq} k1={k1}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    got = parity.gpu_retrieve(bank, torch, q, 0, k1, min(8, k1), 0.5)
    stats = parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[0], k1, min(8, k1), 0.5, got)
    if kind in ("equal", "steps"):
        assert stats["boundary_swaps"] == 0
    assert not bank.retrieve_flags(nq).cpu().numpy().any() and bank.counters() == (0, 0)
    bank.close()


@pytest.mark.parametrize("kind", ["outlier", "steps", "equal"])
@pytest.mark.parametrize("dtype,N,nq,k1", [("bf16", 20000, 3, 200), ("f32", 9000, 2, 1), ("f16", 17000, 9, 64)])
def test_exhaustive_lists_of_any_spread(orc, dtype, N, nq, k1, kind):
    """The same in the exhaustive call, whose selections cut a crowded list back to the pool before any of its places are given out."""
    rng = np.random.default_rng([67, N, k1])
    v = _unit(rng, 1, 64)
    rows = _rows(kind, rng, N, 64, v)
    q = np.concatenate([v, _unit(rng, nq, 64)])[:nq]
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"exhaustive selection {kind} {dtype} N={N} B={nq} k1={k1}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    ids, scores, cid, csim = bank.retrieve_exact(_dev(q), 0, k1, min(8, k1), 0.5, want_candidates=True)
    got = {"ids": ids.cpu().numpy(), "scores": scores.cpu().numpy(), "cand_ids": cid.cpu().numpy(), "cand_sims": csim.cpu().numpy()}
    stats = parity.check_retrieve(orc, orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype]), qtab[0], k1, min(8, k1), 0.5, got)
    if kind in ("equal", "steps"):
        assert stats["boundary_swaps"] == 0
    bank.close()
