"""Value update: batches at the edges of the lists that are ordered by counting, all pairs in one list or spread, few and many
repetitions of an id, ids outside the bank, bit for bit against the sequential fp32 recurrence."""
import numpy as np
import pytest

from tests.test_gpu_parity import _check_update, _make_bank, _unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("distinct", [1, 3, 40, 100000])
@pytest.mark.parametrize("M", [1, 2, 32, 33, 255, 256, 257, 300, 8192, 16384, 16385])
def test_lists_up_to_and_past_the_counted_length(orc, M, distinct):
    rng = np.random.default_rng([51, M, distinct])
    N = 3000
    table = rng.uniform(-1, 1, (2, N)).astype(np.float32)
    bank = _make_bank("f32", _unit(rng, N, 8), table, max_B=1, max_k1=8)
    ids = rng.choice(rng.permutation(N)[:distinct], M).astype(np.int32)
    if distinct > 40 and M > 32:
        ids[rng.permutation(M)[:5]] = [-1, N, N + 7, -2147483648, 2147483647]
    _check_update(orc, bank, 1, table[1], ids, rng.uniform(-1, 1, M).astype(np.float32), 0.1)
    bank.close()
