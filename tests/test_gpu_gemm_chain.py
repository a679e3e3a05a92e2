"""GPU parity of the gated residual in chained slices of K (each slice adds to the residual behind the one in front of it) and of the
block's products that take it."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import check, dev_bf16, dev_f32, errs
from oracle import chorus_oracle as O
from paper_2604_04451_amd import binding as B

pytestmark = pytest.mark.gpu
TILES = {1: (64, 64), 2: (128, 256), 3: (256, 256), 5: (128, 128)}


def _ints(shape, seed, lo=-2, hi=3):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(lo, hi, shape, generator=g, device="cuda").to(torch.float32)


@pytest.mark.parametrize("kernel", list(TILES))
@pytest.mark.parametrize("steps,slices", [(1, 1), (2, 2), (7, 3), (9, 4), (30, 2), (61, 3), (80, 4)])
def test_chain(kernel, steps, slices):
    """Small integers: every order of summation gives the same bits. Rows and columns that end inside a tile, on its edge and behind it;
    slices of one step, of unequal length and (from 30 steps on) each longer than the one in front of it; a count that starts anywhere."""
    rows, cols = TILES[kernel]
    for M, N in ((1, 8), (rows - 1, cols), (rows, cols - 8), (2 * rows + 3, 2 * cols + 24)):
        K = 64 * steps
        print(f"[case] gemm chain kernel={kernel} M={M} N={N} K={K} slices={slices}", flush=True)
        A, W, b, g0, g1 = _ints((M, K), 1), _ints((N, K), 2), _ints((N,), 3), _ints((N,), 5), _ints((N,), 6)
        out = _ints((M, N), 4)
        counts = torch.full((-(-M // rows) * -(-N // cols),), 77, dtype=torch.int32, device="cuda")
        for gates, scale, want in (((g0, g1), 2.0, out + 2 * (g0 + g1) * (A @ W.T + b)), ((None, None), 0.5, out + 0.5 * (A @ W.T + b))):
            buf = torch.cat((out, torch.full((2, N), 7.0, device="cuda")))
            B.chorus_gemm_bf16_chain(A.bfloat16(), W.bfloat16(), buf[:M], kernel, slices, b, *gates, scale, counts)
            assert torch.equal(buf[:M], want) and bool((buf[M:] == 7.0).all())


@pytest.mark.parametrize("tm,tn", [(12, 7), (27, 3), (5, 17), (17, 5)])
def test_chain_in_one_group(tm, tn):
    """81, 84 and 85 tiles in three slices: more workgroups than units on an XCD if each took its tiles' slices, so one counter for two XCDs
    and for all."""
    M, N, K = 64 * tm - 1, 64 * tn, 64 * 48
    A, W, out = _ints((M, K), 1), _ints((N, K), 2), _ints((M, N), 4)
    got = out.clone()
    B.chorus_gemm_bf16_chain(A.bfloat16(), W.bfloat16(), got, 1, 3, scale=0.5)
    assert torch.equal(got, out + 0.5 * (A @ W.T))


@pytest.mark.parametrize("M,slices", [(3271, 3), (3500, 3), (1500, 4)])
def test_chains_on_several_streams(M, slices):
    """Six chains at a time, three in a row on each of six streams: waits that depend on what else runs would show here."""
    N, K = 1536, 64 * 32
    A, W, out = _ints((M, K), 1), _ints((N, K), 2), _ints((M, N), 4)
    print(f"[case] gemm chains on streams M={M} slices={slices}", flush=True)
    want = out + 3 * (A @ W.T)
    A, W = A.bfloat16(), W.bfloat16()
    streams = [torch.cuda.Stream() for _ in range(6)]
    got = [out.clone() for _ in streams]
    counts = [torch.full((256,), 77, dtype=torch.int32, device="cuda") for _ in streams]
    torch.cuda.synchronize()
    for _ in range(3):
        for st, o, c in zip(streams, got, counts):
            with torch.cuda.stream(st):
                B.chorus_gemm_bf16_chain(A, W, o, 3, slices, counts=c)
    torch.cuda.synchronize()
    assert all(torch.equal(o, want) for o in got)


def test_chain_refuses():
    A, W = torch.zeros(8, 128, dtype=torch.bfloat16, device="cuda"), torch.zeros(64, 128, dtype=torch.bfloat16, device="cuda")
    out, counts = torch.zeros(8, 64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    for kernel, slices, n in ((4, 2, 1), (0, 2, 1), (6, 2, 1), (1, 0, 1), (1, 5, 1), (1, 3, 1), (1, 2, 0)):
        with pytest.raises(B.ChorusError):
            B.chorus_gemm_bf16_chain(A, W, out, kernel, slices, counts=counts[:n])


# (D, H, F, Ls): blocks whose O, cross-O and second FFN products are chained (True), by chorus_gemm_bf16_chain_plan
BLOCKS = {(1536, 12, 4096, 300): (False, True), (2048, 16, 4096, 1000): (True, True), (2560, 20, 4096, 150): (True, True),
          (1024, 8, 8192, 1000): (False, True)}


def _weights(rnd, D, F):
    t = {}
    for n, o, i in (("qkv", 3 * D, D), ("o", D, D), ("cq", D, D), ("ckv", 2 * D, D), ("co", D, D), ("1", F, D), ("2", D, F)):
        t["w_" + n], t["b_" + n] = (rnd(o, i) * 0.02).bfloat16(), rnd(o) * 0.05
    t.update(mod_table=rnd(6, D) * 0.3, g_q=rnd(D), g_k=rnd(D), g_cq=rnd(D), g_ck=rnd(D), ln3_w=rnd(D), ln3_b=rnd(D))
    return t, B.DeviceBlock(t, B.BlockWeights(**{n: t[n].data_ptr() for n in B._W_FIELDS}))


def test_blocks_on_three_streams():
    """Blocks whose three residual products are all chained, in three streams with a workspace each, against the same calls one by one."""
    D, H, F, Ls = 2048, 16, 4096, 1000
    assert BLOCKS[D, H, F, Ls] == (True, True)
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    _, w = _weights(rnd, D, F)
    shape = B.make_block_shape(D, H, D // H, F, 40, (1, 32, 32))
    ctx, t_mod, x = rnd(40, D).bfloat16(), rnd(6, D) * 0.3, [rnd(Ls, D) for _ in range(3)]
    ws = [torch.full((B.chorus_dit_block_workspace_bytes(shape, Ls),), 255, dtype=torch.uint8, device="cuda") for _ in x]
    step = lambda y, s: B.chorus_dit_block_step(shape, w, y, Ls, None, ctx, t_mod, None, 1.0, s)  # noqa: E731
    want = [v.clone() for v in x]
    for y in want:
        for _ in range(2):
            step(y, ws[0])
    streams = [torch.cuda.Stream() for _ in x]
    torch.cuda.synchronize()
    for _ in range(2):
        for st, y, s in zip(streams, x, ws):
            with torch.cuda.stream(st):
                step(y, s)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(x, want))


@pytest.mark.parametrize("D,H,F,Ls", list(BLOCKS))
def test_block_with_chained_products(D, H, F, Ls):
    """Three replays of a captured block with other work in between, on a workspace that starts anywhere, against the call outside, and
    that against float64 of the FFN branch (its hidden rows rounded to bf16, as are its inputs: 5 roundings of 2^-9 / sqrt(3) at most)."""
    chained = lambda K: B.chorus_gemm_bf16_chain_plan(Ls, D, K, 4 * Ls * D)[3]  # noqa: E731
    assert (chained(D), chained(F)) == BLOCKS[D, H, F, Ls]
    print(f"[case] block chained D={D} F={F} Ls={Ls}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(D + F)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    t, w = _weights(rnd, D, F)
    shape = B.make_block_shape(D, H, D // H, F, 40, (1, 32, 32))
    x, ctx, t_mod = rnd(Ls, D), rnd(40, D).bfloat16(), rnd(6, D) * 0.3
    ws = torch.full((B.chorus_dit_block_workspace_bytes(shape, Ls),), 255, dtype=torch.uint8, device="cuda")
    want = x.clone()
    B.chorus_dit_block_step(shape, w, want, Ls, None, ctx, t_mod, None, 1.0, ws)
    got = x.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.chorus_dit_block_step(shape, w, got, Ls, None, ctx, t_mod, None, 1.0, ws)
    for _ in range(3):
        got.copy_(x)
        ws.fill_(85)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    for n in ("o", "co"):  # the FFN alone
        t["w_" + n].zero_()
        t["b_" + n].zero_()
    y = x.clone()
    B.chorus_dit_block_step(shape, w, y, Ls, None, ctx, t_mod, None, 1.0, ws)
    xd, m = x.double(), (t["mod_table"] + t_mod).double()
    h = (xd - xd.mean(1, keepdim=True)) * (xd.var(1, unbiased=False, keepdim=True) + 1e-6).rsqrt() * (1 + m[4]) + m[3]
    f = torch.nn.functional.gelu(h @ t["w_1"].double().T + t["b_1"].double(), approximate="tanh") @ t["w_2"].double().T + t["b_2"].double()
    delta = m[5] * f
    assert float(((y.double() - xd) - delta).norm() / delta.norm()) < 5 * 2.0 ** -9 / 3 ** 0.5


# (D, H, F, Ls): what the O and cross-O products and self-attention do, by the plan functions: (rows in front, kernel, slices, chained) and
# (whole tiles, slices of the others)
BOTH = {(2048, 16, 2048, 1000): ((0, 5, 2, True), (0, 0)), (5120, 40, 2048, 3266): ((3072, 5, 3, True), (512, 4)),
        (256, 4, 512, 17000): ((0, 0, 0, False), (256, 4))}


@pytest.mark.parametrize("D,H,F,Ls", list(BOTH))
def test_block_with_chains_and_key_slices(D, H, F, Ls):
    """Blocks whose O and cross-O products are chained, whose self-attention runs its last tiles in key slices, and that do both on scratch
    that stands side by side, on a workspace that starts anywhere: sampled rows against the oracle, gates near 1 and biases, so that
    each branch weighs in the result. Tolerances as for the full-size blocks."""
    chain, slices = BOTH[D, H, F, Ls]
    plan = B.chorus_gemm_bf16_chain_plan(Ls, D, D)
    assert (plan == chain if chain[3] else not plan[3]) and B.chorus_attention_slices_plan(Ls, H, D // H, 256, 2 * Ls * D - 1024, 6 * Ls * D) == slices
    print(f"[case] block chains and key slices D={D} Ls={Ls}", flush=True)
    bs = synth.BlockShape("chains", D, H, D // H, F, 40, 64, (1, 136, 128))
    w, inp = synth.block_weights(bs, 1), synth.block_inputs(bs, 1, L=Ls)
    w["mod_table"][[2, 5]] += 0.8
    for n in ("b_qkv", "b_o", "b_cq", "b_ckv", "b_co", "b_1", "b_2"):
        w[n] = synth.normal(2, n, w[n].shape, 0.1)
    shape = B.make_block_shape(D, H, D // H, F, 40, bs.grid)
    idx = np.sort(synth.stream(3, "idx").permutation(bs.L)[:Ls])
    x = dev_f32(inp["x"])
    ws = torch.full((B.chorus_dit_block_workspace_bytes(shape, Ls),), 255, dtype=torch.uint8, device="cuda")
    B.chorus_dit_block_step(shape, B.upload_block_weights(w), x, Ls, torch.from_numpy(idx.astype(np.int32)).cuda(), dev_bf16(inp["text_ctx"]),
                            dev_f32(inp["t_mod"]), None, 0.75, ws)
    got = x.cpu().numpy()
    assert np.isfinite(got).all()
    at = synth.stream(4, "rows").permutation(Ls)
    rows = np.unique(np.concatenate([at[:24], at[at >= Ls - 170][:12], [0, Ls - 1]]))
    ref, branch = O.dit_block(inp["x"], w, bs, inp["text_ctx"], inp["t_mod"], token_idx=idx, gamma_o=0.75, rows=rows, return_branches=True)
    change = ref - inp["x"][rows]
    for part in (branch["g1"] * branch["y_sa"], 0.75 * branch["y_ca"], branch["g2"] * branch["y_ffn"]):
        assert np.linalg.norm(part) > 0.05 * np.linalg.norm(change)
    check(got[rows], ref, "block chains and key slices x")
    a, r = errs(got[rows] - inp["x"][rows], change)
    print(f"[parity] block chains and key slices delta: max_abs={a:.3e} rel_l2={r:.3e}", flush=True)
    assert r <= 2e-2
