"""Batch sizes of the reward shaping at the edges of its one-launch and two-launch forms, the statistics
carried from call to call, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_10846_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stage", [0, 1])
def test_batch_sizes(orc, stage):
    rng = np.random.default_rng(41 + stage)
    bank = B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    state = None
    for M in (1, 1023, 1024, 1025, 1, 1280, 1281, 70001, 3):        # one block, block edges, more blocks than a block adds up at once
        print(f"rewards stage={stage} M={M}", flush=True)
        feasible = (rng.random(M) < 0.7).astype(np.uint8)
        latency, best = rng.uniform(0.1, 5.0, M).astype(np.float32), rng.uniform(0.1, 5.0, M).astype(np.float32)
        want, state = orc.shape_rewards(stage, feasible, latency, best, True, np.float32(0.1), np.float32(2.5), state)
        got = bank.shape_rewards(stage, dev(feasible), dev(latency), dev(best), True, 0.1, 2.5).cpu().numpy()
        # fp64 sums in another order, then one rounding to fp32: 1e-6 as the reward test of the parity suite has it
        assert np.all(np.abs(got - want) <= 1e-6 * np.maximum(1.0, np.abs(want))), M
        plain = bank.shape_rewards(stage, dev(feasible), dev(latency), dev(best), False).cpu().numpy()
        raw, _ = orc.shape_rewards(stage, feasible, latency, best, False, 0.1, 0.0, None)
        assert np.all(np.abs(plain - raw) <= 1e-6)
    n, mu, sd = bank.reward_stats(stage)
    assert n == state[0] and abs(mu - state[1] / state[0]) < 1e-9
    bank.close()


@pytest.mark.parametrize("stage", [0, 1])
def test_long_batches_are_split(orc, stage):
    """Batches that take several pairs of launches (2,097,152 samples each): the statistics are carried from one to the next."""
    rng = np.random.default_rng(43 + stage)
    bank = B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    state, piece = None, 8192 * 256
    for M in (piece, piece + 1, 2 * piece + 777):
        print(f"rewards stage={stage} M={M}", flush=True)
        feasible = (rng.random(M) < 0.7).astype(np.uint8)
        latency, best = rng.uniform(0.1, 5.0, M).astype(np.float32), rng.uniform(0.1, 5.0, M).astype(np.float32)
        want, state = orc.shape_rewards(stage, feasible, latency, best, True, np.float32(0.1), np.float32(2.5), state)
        got = bank.shape_rewards(stage, dev(feasible), dev(latency), dev(best), True, 0.1, 2.5).cpu().numpy()
        # the oracle adds up to 8.4 M fp64 terms one after another (8.4e6 x 1.1e-16 of a mean of magnitude 1), then one rounding to fp32
        assert np.all(np.abs(got - want) <= 1e-6 * np.maximum(1.0, np.abs(want))), M
        n, mu, sd = bank.reward_stats(stage)
        assert n == state[0] and abs(mu - state[1] / state[0]) < 1e-9
    bank.close()


@pytest.mark.parametrize("stage", [0, 1])
def test_pieces_of_one_launch(orc, stage):
    """One to three pieces of 1024 in one launch, the last one full, nearly empty or nearly full, and the first batch beyond."""
    rng = np.random.default_rng(45 + stage)
    bank = B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    state = None
    for M in (1024, 1025, 1087, 1535, 1536, 1537, 2047, 2048, 2049, 3072, 3073):
        print(f"rewards stage={stage} M={M}", flush=True)
        feasible = (rng.random(M) < 0.7).astype(np.uint8)
        latency, best = rng.uniform(0.1, 5.0, M).astype(np.float32), rng.uniform(0.1, 5.0, M).astype(np.float32)
        for normalise in (True, False):
            want, after = orc.shape_rewards(stage, feasible, latency, best, normalise, np.float32(0.1), np.float32(2.5), state)
            got = bank.shape_rewards(stage, dev(feasible), dev(latency), dev(best), normalise, 0.1, 2.5).cpu().numpy()
            # fp64 sums in another order, then one rounding to fp32
            assert np.all(np.abs(got - want) <= 1e-6 * np.maximum(1.0, np.abs(want))), (M, normalise)
            if normalise:
                state = after
        n, mu, sd = bank.reward_stats(stage)
        assert n == state[0] and abs(mu - state[1] / state[0]) < 1e-9
    bank.close()
