"""The lookup whose last workgroup collects what the others leave in the workspace: any content of the workspace beforehand,
calls of different sizes on one workspace, captured launches replayed on changing caches, and the path on which the last
workgroup waits too short a time (forced by the caller) and makes the whole result itself. Every path gives the same bits."""
import pytest
import torch

from paper_2604_04451_amd import binding as B

pytestmark = pytest.mark.gpu
D = 64
ROUNDS = (8192, 0, -1)  # the plain call's wait, one look, none


def _cache(N, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(N, D, generator=g, device="cuda"), torch.randn(D, generator=g, device="cuda")


def _best(cache, q):
    s = (cache.double() @ q.double()) / cache.double().norm(dim=1) / q.double().norm()
    return int(s.argmax()), float(s.max())


def _lookup(cache, q, rounds, ws):
    out = torch.full((3,), -7, dtype=torch.int32, device="cuda")
    return B.chorus_cache_lookup_wait(cache, q, 0.3, rounds, out, ws)


def _ws(N):
    return torch.empty(B.load().chorus_cache_lookup_workspace_bytes(N), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("N", [1, 7, 8, 9, 4097, 16385, 40003])  # one workgroup, several, several rows a wave
def test_any_workspace_and_any_wait(N):
    print(f"[case] lookup in one launch N={N}", flush=True)
    cache, q = _cache(N, N)
    idx, score = _best(cache, q)
    ws, bits = _ws(N), set()
    for fill in (0, 255, 1):
        ws.fill_(fill)
        for rounds in ROUNDS:
            out = _lookup(cache, q, rounds, ws)
            got = B.lookup_result(out)
            assert got[0] == idx and abs(got[1] - score) < 1e-6 and got[2] == (got[1] >= 0.3)
            bits.add(tuple(out.tolist()))
    assert len(bits) == 1


def test_calls_that_share_a_workspace():
    ws = _ws(20000)
    print("[case] lookups on one workspace", flush=True)
    for seed, N in enumerate((20000, 5, 3000, 20000, 12000, 8)):
        cache, q = _cache(N, seed)
        assert B.lookup_result(_lookup(cache, q, 8192, ws))[0] == _best(cache, q)[0]


@pytest.mark.parametrize("rounds", ROUNDS)
def test_replays_on_changing_caches(rounds):
    """A captured launch has the same number at every replay: nothing of an earlier replay may count."""
    print(f"[case] lookup replays rounds={rounds}", flush=True)
    N = 5000
    cache, q = _cache(N, 1)
    ws, out = _ws(N), torch.zeros(3, dtype=torch.int32, device="cuda")
    B.chorus_cache_lookup_wait(cache, q, 0.3, rounds, out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.chorus_cache_lookup_wait(cache, q, 0.3, rounds, out, ws)
    for seed in range(2, 8):
        c, qq = _cache(N, seed)
        cache.copy_(c)
        q.copy_(qq)
        out.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert B.lookup_result(out)[0] == _best(cache, q)[0], seed
