"""The lookup whose last workgroup collects what the others leave in the workspace: any content of the workspace beforehand,
calls of different sizes on one workspace, and the path on which the last workgroup waits too short a time (forced by the caller)
and makes the whole result itself; the two launches of a captured call, replayed on changing caches and workspaces, and of a
cache of over 16 GB. Every path gives the same bits."""
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


def _captured(cache, q, rounds, out, ws):
    B.chorus_cache_lookup_wait(cache, q, 0.3, rounds, out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.chorus_cache_lookup_wait(cache, q, 0.3, rounds, out, ws)
    return graph


@pytest.mark.parametrize("rounds", ROUNDS)
def test_replays_after_other_uses_of_the_workspace(rounds):
    """Between replays the workspace is the caller's: nothing that an earlier replay left in any part of it may count, whatever
    became of the other parts."""
    print(f"[case] lookup replays, workspace used between them, rounds={rounds}", flush=True)
    N = 16384
    cache, q = _cache(N, 1)
    ws, out = _ws(N), torch.zeros(3, dtype=torch.int32, device="cuda")
    graph = _captured(cache, q, rounds, out, ws)
    left = [ws.clone()]
    for seed in range(2, 10):
        c, qq = _cache(N, seed)
        cache.copy_(c)
        q.copy_(qq)
        if seed % 3 == 0:
            ws.copy_(left[seed // 2 % len(left)])  # what an earlier replay left
        elif seed % 3 == 1:
            ws[:4096].fill_(seed)
        else:
            ws[:256].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert B.lookup_result(out)[0] == _best(cache, q)[0], seed
        left.append(ws.clone())


def test_two_graphs_on_one_workspace():
    print("[case] two captured lookups on one workspace", flush=True)
    ws = _ws(16384)
    caches = [_cache(N, N) for N in (16384, 3000)]
    outs = [torch.zeros(3, dtype=torch.int32, device="cuda") for _ in caches]
    graphs = [_captured(c, q, 0, o, ws) for (c, q), o in zip(caches, outs)]
    for seed in range(8):
        for (c, q), o, g in zip(caches, outs, graphs):
            c2, q2 = _cache(len(c), 100 + seed)
            c.copy_(c2)
            q.copy_(q2)
            g.replay()
            torch.cuda.synchronize()
            assert B.lookup_result(o)[0] == _best(c, q)[0], seed


def test_cache_of_more_than_2_32_values():
    """Two launches; row offsets beyond 32 bits in both entry points."""
    N, d = (1 << 20) + 3, 4096
    print(f"[case] lookup N={N} d={d}", flush=True)
    cache, q = torch.zeros(N, d, device="cuda"), torch.ones(d, device="cuda")
    for rows, want in (((5, N - 1), N - 1), ((N - 3, N - 2, 70), 70)):
        for i, r in enumerate(rows):
            cache[r, : d // (2 if i == 0 and want == N - 1 else 1)] = 1.0
        ws, out = _ws(N), torch.full((3,), -7, dtype=torch.int32, device="cuda")
        B.chorus_cache_lookup(cache, q, 0.9, out, ws)
        assert B.lookup_result(out) == (want, 1.0, 1)
        B.chorus_cache_lookup_static(cache, q, 0.9, out.fill_(-7))
        assert B.lookup_result(out) == (want, 1.0, 1)


def test_replay_is_no_slower_after_others():
    """A replay costs what the first one cost, whatever the captured call's wait was: no replay scans alone (1.8 ms here)."""
    print("[case] time of lookup replays", flush=True)
    cache = torch.randn(4096, 4096, device="cuda")
    q, ws, out = torch.randn(4096, device="cuda"), _ws(4096), torch.zeros(3, dtype=torch.int32, device="cuda")
    graph = _captured(cache, q, 0, out, ws)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(3):
        e0.record()
        for _ in range(20):
            graph.replay()
        e1.record()
        e1.synchronize()
        assert e0.elapsed_time(e1) / 20 < 0.2


def test_beside_another_stream():
    """While another stream's products fill the chip a lookup's workgroups start far apart."""
    print("[case] lookups beside products on another stream", flush=True)
    cache, q = _cache(20000, 3)
    idx, _ = _best(cache, q)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    ws, outs = _ws(20000), [torch.full((3,), -7, dtype=torch.int32, device="cuda") for _ in range(40)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(12):
            b = a @ a
    for out in outs:
        B.chorus_cache_lookup(cache, q, 0.3, out, ws)
    torch.cuda.synchronize()
    del b
    assert all(B.lookup_result(o)[0] == idx for o in outs) and len({tuple(o.tolist()) for o in outs}) == 1
