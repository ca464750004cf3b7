"""Normalised rewards of 1025 to 16,384 samples: one launch of up to 64 blocks that wait for each other's sums.  Sizes at the edges, many calls
in a row, two banks on two streams at a time, against the oracle; calls on one bank that overlap (which is not supported) end and leave nothing behind
that a later call trips over; calls recorded into a graph."""
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


def test_bits_of_other_calls_are_dropped(orc):
    """Whatever bits overlapping calls have left in the words that the blocks meet at: a later call waits for its own blocks."""
    rng = np.random.default_rng(85)
    bank, state = B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1), None
    for M in (8192, 8000, 16384, 12000, 1025):
        print(f"chain with bits left M={M}", flush=True)
        f, l, b = _batch(rng, M)
        want, state = orc.shape_rewards(1, f, l, b, True, np.float32(0.1), np.float32(2.5), state)
        assert _close(bank.shape_rewards(1, _dev(f), _dev(l), _dev(b), True, 0.1, 2.5).cpu().numpy(), want), M
        bank.workspace[128:144].view(torch.int64).bitwise_or_(0xffffffff)       # (the two words lie there; numbers of calls above, bits below)
    n, mu, _ = bank.reward_stats(1)
    assert n == state[0] and abs(mu - state[1] / state[0]) < 1e-9
    bank.close()


def test_overlapping_calls_end(orc):
    """Two streams on one bank: what comes out means nothing, but every call ends and later calls in order are right."""
    rng = np.random.default_rng(87)
    bank = B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1)
    streams = [torch.cuda.Stream() for _ in range(2)]
    on_gpu = [[tuple(map(_dev, _batch(rng, int(rng.integers(1025, 16385))))) for _ in range(20)] for _ in range(2)]
    torch.cuda.synchronize()
    for i in range(20):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                bank.shape_rewards(1, *on_gpu[k][i], True, 0.1, 2.5)
    torch.cuda.synchronize()
    print("overlapping calls ended", flush=True)
    bank.reward_stats_reset(1)
    state = None
    for M in (16384, 1025, 8192):
        f, l, b = _batch(rng, M)
        want, state = orc.shape_rewards(1, f, l, b, True, np.float32(0.1), np.float32(2.5), state)
        assert _close(bank.shape_rewards(1, _dev(f), _dev(l), _dev(b), True, 0.1, 2.5).cpu().numpy(), want), M
    bank.close()


def test_recorded_calls(orc):
    """A batch recorded into a graph, replayed with calls of its own kind in between: bit for bit what the same calls give eagerly."""
    rng = np.random.default_rng(89)
    one, two = (B.MemoryBank(64, "f32", 256, max_B=1, max_k1=1) for _ in range(2))
    batch, other = (tuple(map(_dev, _batch(rng, M))) for M in (9000, 5000))
    one.shape_rewards(1, *other, True, 0.1, 2.5)
    two.shape_rewards(1, *other, True, 0.1, 2.5)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = one.shape_rewards(1, *batch, True, 0.1, 2.5)
    for i in range(4):
        graph.replay()
        want = two.shape_rewards(1, *batch, True, 0.1, 2.5)
        torch.cuda.synchronize()
        assert torch.equal(out, want), i
        assert torch.equal(one.shape_rewards(1, *other, True, 0.1, 2.5), two.shape_rewards(1, *other, True, 0.1, 2.5)), i
    assert one.reward_stats(1) == two.reward_stats(1)
    one.close()
    two.close()
