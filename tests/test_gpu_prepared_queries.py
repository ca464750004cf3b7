"""Query preparation, a query to a workgroup and by whole fragments: batches at the edges of a fragment's 16 queries and of a round of groups on the
XCDs, rows at the edges of a slice, values that bf16 and fp16 round to infinity, to zero and to a neighbour, NaN, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_10846_amd import binding as B
from tests import parity
from tests.test_gpu_parity import DT, _dev, _make_bank, _unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,nq,d", [
    ("f32", 17, 64), ("f32", 33, 136), ("f32", 129, 72), ("f32", 300, 200), ("f32", 1024, 128),       # by fragments; one slice, one and a part
    ("bf16", 17, 136), ("bf16", 65, 64), ("bf16", 256, 200), ("f16", 130, 72),                        # a query to a workgroup
    ("bf16", 1024, 3016), ("f16", 769, 4096), ("f16", 1000, 3072)])                                   # 16 bits by fragments
def test_prepared_queries_match_oracle(orc, dtype, nq, d):
    rng = np.random.default_rng([97, nq, d])
    N, k1 = 1500, 32
    rows = _unit(rng, N, d)
    q = _unit(rng, nq, d) * np.exp2(rng.integers(-6, 7, (nq, 1))).astype(np.float32)
    q[nq // 2, :3] = np.float32(1 + 2.0 ** -9), np.float32(1 + 2.0 ** -8 + 2.0 ** -9), np.float32(2.0 ** -30)   # halves of a step: to the even neighbour
    qtab = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    print(f"prepared queries {dtype} B={nq} d={d}", flush=True)
    bank = _make_bank(dtype, rows, qtab, max_B=nq, max_k1=k1)
    got = parity.gpu_retrieve(bank, torch, q, 0, k1, 8, 0.5)
    st, qr = orc.round_to_store(rows, DT[dtype]), orc.round_to_store(q, DT[dtype])
    check = np.unique(np.concatenate([np.arange(nq)[-20:], np.arange(0, nq, 16), [nq // 2]]))[:100]
    parity.check_retrieve(orc, st, qr[check], qtab[0], k1, 8, 0.5, {k: v[check] for k, v in got.items()})
    # all of them: the pool's similarities in fp64 (rounded to fp32: 6e-8)
    x, y = _dev(st.astype(np.float64)), _dev(qr.astype(np.float64))
    want = ((y / y.norm(dim=1, keepdim=True)) @ (x / x.norm(dim=1, keepdim=True)).T).topk(k1, dim=1).values.cpu().numpy()
    assert np.abs(want - got["cand_sims"]).max() < 1e-7
    bank.close()


@pytest.mark.parametrize("dtype,nq,d", [("f32", 64, 64), ("bf16", 40, 72), ("f16", 1024, 3072)])
def test_queries_without_a_norm_change_no_other(dtype, nq, d):
    """NaN, infinite and zero queries, and ones that 16 bits round to these: the others' answers are bit for bit those of a batch without."""
    rng = np.random.default_rng([101, nq, d])
    rows, q = _unit(rng, 3000, d), _unit(rng, nq, d)
    bank = _make_bank(dtype, rows, rng.uniform(-1, 1, (2, 3000)).astype(np.float32), max_B=nq, max_k1=16)
    odd = np.arange(5, nq, 13)
    want = parity.gpu_retrieve(bank, torch, q, 0, 16, 4, 0.5)
    for i, b in enumerate(odd):
        q[b] = (np.nan, np.inf, 0.0, 3.4e38, 1e-42, -np.inf)[i % 6]
    got = parity.gpu_retrieve(bank, torch, q, 0, 16, 4, 0.5)
    rest = np.setdiff1d(np.arange(nq), odd)
    for k in ("ids", "scores", "cand_ids", "cand_sims"):
        assert np.array_equal(got[k][rest].view(np.uint32), want[k][rest].view(np.uint32)), k
    bank.close()


def test_fp32_operands_cost_little_more():
    """1024 queries of 4096 on empty banks (their preparation, and an end of the call that finds nothing): fp32 writes twice the operand bytes that 16
    bits do, 48 MB in all where these take 40.  With 16-byte pieces of different queries side by side it took 36.8 us against 30.4, as whole fragments 28 and
    27."""
    q = torch.randn((1024, 4096), device="cuda:0")
    banks = [B.MemoryBank(4096, dtype, 256, max_B=1024, max_k1=1) for dtype in ("f32", "bf16")]
    best = [float("inf")] * 2
    for _ in range(15):
        for i, bank in enumerate(banks):
            bank.retrieve(q, 0, 1, 1, 0.5)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                bank.retrieve(q, 0, 1, 1, 0.5)
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 50)
    print(f"empty bank, fp32 {best[0]:.1f} us, bf16 {best[1]:.1f} us", flush=True)
    for bank in banks:
        bank.close()
    assert best[0] < 1.12 * best[1], best
