"""GPU parity of the batched lookup's scan where its ring of steps, its two buffers of queries and its tiles end: from one to seven
64-float steps in a slice with whole and cut last steps, rows that end inside a wave's 16, a workgroup's 64 or 128 and a half of it."""
import numpy as np
import pytest

import synth
from test_gpu_lookup_region import _check_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,Q", [
    (1, 4, 1), (15, 60, 16), (16, 64, 17), (17, 68, 32),           # one step
    (63, 128, 2), (65, 132, 33), (127, 192, 16), (129, 196, 20),   # two to four
    (66000, 64, 17), (66001, 196, 3), (66100, 448, 32),            # one slice of one, four and seven steps
    (4100, 3980, 18), (8000, 2052, 5),                             # eight waves a workgroup
])
def test_lookup_batch_stream(N, d, Q):
    print(f"[case] lookup_batch stream N={N} d={d} Q={Q}", flush=True)
    cache = synth.cache_embeddings(N, d, seed=1)
    if N > 3:
        cache[N - 1] = cache[N // 2]  # the last row, alone in its wave or not, scores like any other
    queries = np.stack([synth.cache_query(cache, seed=1, near=(N - 1 - 37 * t) % N if t % 4 else None, trial=t) for t in range(Q)])
    _check_topk(cache, queries, 0.75, min(N, 64))
    if N > 3:
        idx, sc, _ = _check_topk(cache, queries, 0.75, 2)
        both = [t for t in range(Q) if t % 4 and (N - 1 - 37 * t) % N in (N - 1, N // 2)]
        assert all(list(idx[t]) == [N // 2, N - 1] and sc[t, 0] == sc[t, 1] for t in both)
