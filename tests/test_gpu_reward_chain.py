"""Normalised rewards of 1025 to 16,384 samples: one launch of up to 64 blocks that wait for each other's sums.  Sizes at the edges, many calls
in a row (the words that the blocks meet at are left as they were found), two banks on two streams at a time, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_10846_amd import binding as B

pytestmark = pytest.mark.gpu


def _batch(rng, M):
    return (rng.random(M) < 0.7).astype(np.uint8), rng.uniform(0.1, 5.0, M).astype(np.float32), rng.uniform(0.1, 5.0, M).astype(np.float32)


def _dev(a):
    return torch.from_numpy(a).to("cuda:0")


# fp64 sums in another order, then one rounding to fp32: 1e-6 as the reward test of the parity suite has it
def _close(got, want):
    return np.all(np.abs(got - want) <= 1e-6 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("stage", [0, 1])
def test_sizes_at_the_edges(orc, stage):
    rng = np.random.default_rng(81 + stage)
    bank, state = B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1), None
    for M in (1025, 1279, 1280, 1281, 8192, 16127, 16128, 16129, 16383, 16384, 16385, 1025):
        print(f"chain stage={stage} M={M}", flush=True)
        f, l, b = _batch(rng, M)
        want, state = orc.shape_rewards(stage, f, l, b, True, np.float32(0.1), np.float32(2.5), state)
        assert _close(bank.shape_rewards(stage, _dev(f), _dev(l), _dev(b), True, 0.1, 2.5).cpu().numpy(), want), M
    n, mu, _ = bank.reward_stats(stage)
    assert n == state[0] and abs(mu - state[1] / state[0]) < 1e-9
    bank.close()


def test_two_banks_on_two_streams(orc):
    rng = np.random.default_rng(83)
    banks = [B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    batches = [[_batch(rng, int(rng.integers(1025, 16385))) for _ in range(30)] for _ in range(2)]
    on_gpu = [[tuple(map(_dev, x)) for x in row] for row in batches]
    torch.cuda.synchronize()
    got = [[], []]
    for i in range(30):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                got[k].append(banks[k].shape_rewards(1, *on_gpu[k][i], True, 0.1, 2.5))
    torch.cuda.synchronize()
    for k in range(2):
        state = None
        for (f, l, b), r in zip(batches[k], got[k]):
            want, state = orc.shape_rewards(1, f, l, b, True, np.float32(0.1), np.float32(2.5), state)
            assert _close(r.cpu().numpy(), want)
        banks[k].close()
