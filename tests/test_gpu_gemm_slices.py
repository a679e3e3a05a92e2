"""GPU parity of the GEMM tiles and slices that the automatic choice takes for problems that do not fill the chip:
64 x 64 tiles, 128 x 128 tiles with three stages, 128 x 256 tiles, and a product in slices of K on every tile, by name and as
the second FFN product of a block."""
import dataclasses

import numpy as np
import pytest
import torch

import synth
from oracle import chorus_oracle as O
import paper_2604_04451_amd as P
from paper_2604_04451_amd import binding as B
from gpu_util import DEV, check, dev_bf16, dev_f32, errs, host, host_bf16

pytestmark = pytest.mark.gpu


# (M, N, K): the kernels that the default choice takes, for bf16 output and for the gated residual (1: 64 x 64, 2: 128 x 256,
# 4 and 5: 128 x 128 with two and three stages)
DEFAULT_TILES = {
    (1, 8, 64): (4, 1), (63, 64, 128): (4, 1), (64, 72, 192): (4, 1), (65, 768, 256): (1, 1), (129, 256, 320): (1, 1),
    (480, 1536, 1536): (1, 1), (1000, 1536, 4096): (1, 1), (200, 3080, 1024): (1, 1), (1100, 2304, 64): (4, 4),
    (130, 13824, 512): (4, 5), (1990, 4088, 4096): (2, 2), (1025, 7000, 8960): (2, 2),
}


@pytest.mark.parametrize("M,N,K", list(DEFAULT_TILES))
def test_gemm_default_tiles(M, N, K):
    """Ragged rows and columns, fewer rows or columns than a tile, K of fewer steps than the kernels have stages, on the
    default choice."""
    plans = [B.chorus_gemm_bf16_plan(M, N, K, e) for e in (B.EPI_BF16, B.EPI_RESID)]
    assert tuple(p[1] for p in plans) == DEFAULT_TILES[M, N, K], plans
    print(f"[case] gemm default tile M={M} N={N} K={K}", flush=True)
    A = synth.round_bf16(synth.normal(K, "s.A", (M, K)))
    W = synth.round_bf16(synth.normal(K, "s.W", (N, K), 0.05))
    bias, gate, resid = synth.normal(K, "s.b", (N,), 0.5), synth.normal(K, "s.g", (N,), 0.5), synth.normal(K, "s.r", (M, N))
    ref = O.linear(A, W, bias)
    dA, dW, db = dev_bf16(A), dev_bf16(W), dev_f32(bias)
    out = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    B.chorus_gemm_bf16(dA, dW, B.EPI_BF16, out, db)
    check(host_bf16(out), ref, "bf16", max_abs=np.abs(ref).max() * 2 ** -8, rel_l2=3e-3)
    B.chorus_gemm_bf16(dA, dW, B.EPI_GELU_BF16, out, db)
    gref = O.gelu_tanh(ref)
    check(host_bf16(out), gref, "gelu", max_abs=max(np.abs(gref).max() * 2 ** -8, 1e-3), rel_l2=3e-3)
    o32 = torch.empty(M, N, dtype=torch.float32, device=DEV)
    B.chorus_gemm_bf16(dA, dW, B.EPI_F32, o32, db)
    check(host(o32), ref, "f32", max_abs=1e-3, rel_l2=1e-5)
    r = dev_f32(resid)
    B.chorus_gemm_bf16(dA, dW, B.EPI_RESID, r, db, dev_f32(gate), None, 1.5)
    check(host(r), resid + 1.5 * gate.astype(np.float64) * ref, "resid", max_abs=1e-3, rel_l2=1e-5)


@pytest.mark.parametrize("kernel", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("M,N,K,slices", [
    (1, 8, 128, 2), (65, 72, 192, 3), (257, 264, 256, 4),   # as many steps as slices: one each
    (130, 520, 448, 2), (300, 136, 448, 3), (127, 1000, 640, 4), (513, 520, 320, 3),  # steps that do not divide evenly
    (260, 1536, 8960, 2), (700, 768, 4096, 4), (64, 64, 640, 1),
])
def test_gemm_in_slices(M, N, K, slices, kernel):
    """The gated residual with K in slices on every tile: ragged rows and columns, slices of one step (fewer than the tiles
    have stages) and of unequal length, with gates and without; the sum has a fixed order."""
    print(f"[case] gemm slices M={M} N={N} K={K} slices={slices} kernel={kernel}", flush=True)
    A = synth.round_bf16(synth.normal(K + slices, "p.A", (M, K)))
    W = synth.round_bf16(synth.normal(K + slices, "p.W", (N, K), 0.05))
    bias, resid = synth.normal(K, "p.b", (N,), 0.5), synth.normal(K, "p.r", (M, N))
    g0, g1 = synth.normal(K, "p.g0", (N,), 0.5), synth.normal(K, "p.g1", (N,), 0.5)
    ref = O.linear(A, W, bias)
    dA, dW, db = dev_bf16(A), dev_bf16(W), dev_f32(bias)
    guard = torch.full((max(slices - 1, 1) * M * N + 64,), 7.0, device=DEV)
    for gates, scale, want in (((dev_f32(g0), dev_f32(g1)), 1.5, resid + 1.5 * (g0.astype(np.float64) + g1) * ref),
                               ((None, None), 0.5, resid + 0.5 * ref)):
        outs = []
        for _ in range(2):
            out = dev_f32(resid)
            B.chorus_gemm_bf16_slices(dA, dW, out, kernel, slices, db, *gates, scale, parts=guard[:max(slices - 1, 1) * M * N])
            outs.append(host(out))
        assert np.array_equal(*outs)
        check(outs[0], want, f"slices gates={gates[0] is not None}", max_abs=1e-3, rel_l2=1e-5)
    assert bool((guard[max(slices - 1, 1) * M * N:] == 7.0).all())
    if slices == 1:
        by_name = dev_f32(resid)
        B.chorus_gemm_bf16(dA, dW, B.EPI_RESID, by_name, db, None, None, 0.5, kernel=kernel)
        assert np.array_equal(host(by_name), outs[0])


def test_gemm_slices_refuses():
    A, W = torch.zeros(8, 128, dtype=torch.bfloat16, device=DEV), torch.zeros(64, 128, dtype=torch.bfloat16, device=DEV)
    out = torch.zeros(8, 64, device=DEV)
    for kernel, slices, values in ((0, 2, 512), (6, 2, 512), (1, 0, 512), (1, 5, 2048), (1, 3, 1024), (1, 2, 511)):
        with pytest.raises(P.ChorusError):
            B.chorus_gemm_bf16_slices(A, W, out, kernel, slices, parts=torch.zeros(values, device=DEV))


def ffn2_scratch(shape, Ls):
    """What a block's workspace leaves for the slices of its second FFN product: the two bf16 rows of width D in front, and
    everything behind the FFN's hidden rows (each piece is rounded up to 256 bytes)."""
    up = lambda n: -(-n // 256) * 256  # noqa: E731
    first, hidden = 2 * up(Ls * shape.D * 2), up(Ls * shape.F * 2)
    return first, B.chorus_dit_block_workspace_bytes(shape, Ls) - first - hidden


# (Ls, Lt, F) of a block of width 256: the slices of its second FFN product, all on 64 x 64 tiles
FFN_SLICES = {(200, 16, 8960): 2, (200, 128, 8960): 3, (200, 512, 8960): 4, (1, 16, 8960): 4, (131, 77, 4160): 3,
              (384, 300, 13824): 3, (2000, 16, 8960): 2}


@pytest.mark.parametrize("Ls,Lt,F", list(FFN_SLICES))
def test_block_ffn_in_slices(Ls, Lt, F):
    """The FFN of a narrow block with a long hidden row: its second product runs in two, three or four slices of K,
    by what the workspace holds behind the hidden rows (more with more text tokens); slices of unequal length."""
    print(f"[case] ffn slices Ls={Ls} Lt={Lt} F={F}", flush=True)
    bs = dataclasses.replace(synth.SHAPES["c1"], F=F, Lt=Lt, grid=(6, 8, 8) if Ls <= 384 else (8, 16, 16), latent_std=1.0, text_std=1.0)
    w = synth.stress_block_weights(bs, 3)
    for n in ("w_qkv", "w_cq"):  # the attention branches small: the FFN is what is compared
        w[n] = synth.round_bf16(w[n] * 0.25)
    inp = synth.block_inputs(bs, 3, L=Ls)
    idx = np.sort(synth.stream(3, "slices.idx").permutation(bs.L)[:Ls]).astype(np.int32)
    shape = P.make_block_shape(bs.D, bs.H, bs.dh, bs.F, bs.Lt, bs.grid)
    assert B.chorus_gemm_bf16_plan(Ls, bs.D, F, B.EPI_RESID, *ffn2_scratch(shape, Ls)) == (0, 1, FFN_SLICES[Ls, Lt, F])
    outs = []
    for _ in range(2):
        x = dev_f32(inp["x"])
        P.chorus_dit_block_step(shape, P.upload_block_weights(w), x, Ls, torch.from_numpy(idx).to(DEV), dev_bf16(inp["text_ctx"]),
                                dev_f32(inp["t_mod"]), None, 1.0)
        outs.append(host(x))
    assert np.array_equal(outs[0], outs[1]), "the sum over slices has a fixed order"
    ref = O.dit_block(inp["x"], w, bs, inp["text_ctx"], inp["t_mod"], token_idx=idx)
    # stress inputs: the bound scales with the output (bf16 operands at every product)
    check(outs[0], ref, "x", max_abs=np.abs(ref).max() * 2 ** -6, rel_l2=1e-2)
    _, rel = errs(outs[0] - inp["x"], ref - inp["x"])
    assert rel <= 2e-2


@pytest.mark.parametrize("D,H,Lt", [(256, 4, 1), (256, 4, 65), (512, 8, 63), (512, 4, 64), (1536, 12, 130), (320, 5, 17)])
def test_text_kv_equals_the_single_operations(D, H, Lt):
    """Keys and values prepared in one launch against the three calls that it stands for, bit for bit (rows and tiles at
    their edges, padding rows included)."""
    print(f"[case] text kv D={D} H={H} Lt={Lt}", flush=True)
    dh, g = D // H, torch.Generator(device=DEV).manual_seed(Lt)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    t = {n: torch.zeros(1, device=DEV) for n in B._W_FIELDS}
    t.update(w_ckv=(rnd(2 * D, D) * 0.05).bfloat16(), b_ckv=rnd(2 * D), g_ck=rnd(D))
    w = B.DeviceBlock(t, B.BlockWeights(**{n: t[n].data_ptr() for n in B._W_FIELDS}))
    ctx, pad = rnd(Lt, D).bfloat16(), -(-Lt // 64) * 64
    kv = B.chorus_text_kv_project(P.make_block_shape(D, H, dh, 64, Lt, (1, 1, 1)), w, ctx)
    proj = torch.empty(Lt, 2 * D, dtype=torch.bfloat16, device=DEV)
    B.chorus_gemm_bf16(ctx, t["w_ckv"], B.EPI_BF16, proj, t["b_ckv"])
    k = torch.empty(H, pad, dh, dtype=torch.bfloat16, device=DEV)
    vt = torch.empty(D, pad, dtype=torch.bfloat16, device=DEV)
    B.chorus_qk_norm_rope(proj, 0, t["g_ck"], k, Lt, H, dh, None, (1, 1, 1), False)
    B.chorus_v_transpose(proj, D, vt, Lt)
    half = kv.numel() // 2
    assert torch.equal(kv[:k.numel() * 2], k.view(torch.uint8).flatten())
    assert torch.equal(kv[half:half + vt.numel() * 2], vt.view(torch.uint8).flatten())


@pytest.mark.parametrize("D,H,Ls", [(256, 4, 1), (512, 4, 67), (1536, 12, 300), (320, 5, 250)])
def test_block_queries_and_keys_rotate_alike(D, H, Ls):
    """Self-attention alone (the other branches' output weights are zero) on a scattered selection: queries and keys are
    turned by the angles of their token's place on the grid, against the oracle."""
    print(f"[case] block rotation D={D} H={H} Ls={Ls}", flush=True)
    bs = dataclasses.replace(synth.SHAPES["c1"], D=D, H=H, dh=D // H, F=64, Lt=8, grid=(6, 8, 8), latent_std=1.0)
    w = synth.stress_block_weights(bs, 4)
    for n in ("w_co", "b_co", "w_2", "b_2"):
        w[n] = np.zeros_like(w[n])
    inp = synth.block_inputs(bs, 4, L=Ls)
    idx = np.sort(synth.stream(4, "rot.idx").permutation(bs.L)[:Ls]).astype(np.int32)
    x = dev_f32(inp["x"])
    P.chorus_dit_block_step(P.make_block_shape(bs.D, bs.H, bs.dh, bs.F, bs.Lt, bs.grid), P.upload_block_weights(w), x, Ls,
                            torch.from_numpy(idx).to(DEV), dev_bf16(inp["text_ctx"]), dev_f32(inp["t_mod"]), None, 1.0)
    ref = O.dit_block(inp["x"], w, bs, inp["text_ctx"], inp["t_mod"], token_idx=idx)
    _, rel = errs(host(x) - inp["x"], ref - inp["x"])
    assert rel <= 2e-2, rel
