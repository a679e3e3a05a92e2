"""GPU parity of the GEMM tiles and slices that the automatic choice takes for problems that do not fill the chip:
64 x 64 tiles, 128 x 128 tiles with three stages, and the second FFN product of a block in slices of K."""
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


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 64), (63, 64, 128), (64, 72, 192), (65, 768, 256), (129, 256, 320), (480, 1536, 1536),   # 64 x 64, 1 to 24 steps
    (1000, 1536, 4096), (200, 3080, 1024), (1100, 2304, 64), (130, 13824, 512),                      # two per unit, or 128 x 128 deep
])
def test_gemm_default_tiles(M, N, K):
    """Ragged rows and columns, fewer rows or columns than a tile, K of fewer steps than the kernels have stages."""
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


@pytest.mark.parametrize("Ls,Lt,F", [(200, 16, 8960), (200, 128, 8960), (200, 512, 8960), (1, 16, 8960), (131, 77, 4160),
                                     (384, 300, 13824)])
def test_block_ffn_in_slices(Ls, Lt, F):
    """The FFN of a narrow block with a long hidden row: its second product runs in two, three or four slices of K,
    by what the workspace holds behind the hidden rows (more with more text tokens); slices of unequal length."""
    print(f"[case] ffn slices Ls={Ls} Lt={Lt} F={F}", flush=True)
    bs = dataclasses.replace(synth.SHAPES["c1"], F=F, Lt=Lt, grid=(6, 8, 8), latent_std=1.0, text_std=1.0)
    w = synth.stress_block_weights(bs, 3)
    for n in ("w_qkv", "w_cq"):  # the attention branches small: the FFN is what is compared
        w[n] = synth.round_bf16(w[n] * 0.25)
    inp = synth.block_inputs(bs, 3, L=Ls)
    idx = np.sort(synth.stream(3, "slices.idx").permutation(bs.L)[:Ls]).astype(np.int32)
    shape = P.make_block_shape(bs.D, bs.H, bs.dh, bs.F, bs.Lt, bs.grid)
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
