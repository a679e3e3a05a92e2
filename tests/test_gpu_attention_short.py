"""GPU parity of attention launches that leave compute units idle (128-row tiles throughout) and of short key sequences on
128-key tiles: the default choice there and the form on pre-scaled queries, with and without key factors, the row sums, and
the cross-attention of a block against its single operations."""
import numpy as np
import pytest
import torch

import synth
from paper_2604_04451_amd import binding as B
from gpu_util import DEV, dev_f32, host_bf16
from test_gpu_ops import _attn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dh,Lq,Lk", [
    (2, 128, 1, 65), (3, 64, 127, 128), (1, 128, 128, 129), (2, 64, 129, 300), (2, 128, 257, 511), (12, 128, 500, 77),  # half tiles
    (10, 64, 3300, 130),   # full tiles, less than a round: by default 64-key tiles without factors, 128-key tiles with
    (40, 64, 2000, 200),   # more than a round
    (2, 64, 70, 1), (2, 64, 70, 64),
])
@pytest.mark.parametrize("variant", [0, 6])
@pytest.mark.parametrize("factor", [False, True])
def test_attention_short(H, dh, Lq, Lk, variant, factor):
    print(f"[case] attention short H={H} dh={dh} Lq={Lq} Lk={Lk} variant={variant} factor={factor}", flush=True)
    cs = synth.tdiff_scale(Lk, 1.5, n_diff=max(1, Lk // 3)) if factor else None
    _attn_case(H, dh, Lq, Lk, variant, col_scale=cs, q_std=2.0, seed=Lq + Lk, name="short")


@pytest.mark.parametrize("Lk", [128, 256, 640, 1000])
def test_key_factors_follow_their_tile(Lk):
    """Every key its own factor, so that a factor of another tile, group or key would show."""
    print(f"[case] attention key factors Lk={Lk}", flush=True)
    cs = (0.25 + 1.75 * synth.stream(Lk, "cs").random(Lk)).astype(np.float32)
    for Lq in (100, 3000):
        _attn_case(12, 64, Lq, Lk, 6, col_scale=cs, q_std=2.0, seed=Lk, name="factors")


@pytest.mark.parametrize("H,Lq,Lk", [(1, 1, 1), (2, 15, 31), (3, 16, 32), (2, 17, 33), (4, 63, 64), (1, 65, 65), (2, 64, 96), (4, 130, 97),
                                     (9, 200, 128)])
@pytest.mark.parametrize("factor", [False, True])
def test_attention_few_keys(H, Lq, Lk, factor):
    """The kernel without tiles at the edges of its 16 queries and 32 keys, against the oracle and, bit for bit, against the one that
    stages a tile of 128 keys."""
    print(f"[case] attention few keys H={H} Lq={Lq} Lk={Lk} factor={factor}", flush=True)
    cs = (0.25 + 1.75 * synth.stream(Lk, "cs").random(Lk)).astype(np.float32) if factor else None
    _attn_case(H, 64, Lq, Lk, 7, col_scale=cs, q_std=2.0, seed=Lq + Lk, name="few")
    g, pad = torch.Generator(device=DEV).manual_seed(Lk), -(-Lk // 128) * 128
    q, k, vt = (torch.randn(s, device=DEV, generator=g).bfloat16() for s in ((H, 256, 64), (H, pad, 64), (H * 64, pad)))
    k[:, Lk:], vt[:, Lk:] = 0, 0
    a, b = (torch.zeros(Lq, H * 64, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    dcs = dev_f32(cs) if factor else None
    B.chorus_attention(q, k, vt, a, dcs, Lq, Lk, 7)
    B.chorus_attention(q, k, vt, b, dcs, Lq, Lk, 5)
    assert torch.equal(a, b)


def _bf16(x):
    return synth.round_bf16(np.float32(x)).astype(np.float64)


@pytest.mark.parametrize("H,dh,Lq,Lk", [(4, 64, 128, 128), (2, 128, 300, 65), (12, 128, 480, 480), (12, 128, 6000, 226),
                                        (12, 128, 6000, 511), (2, 64, 40, 100), (1, 64, 200, 64)])
@pytest.mark.parametrize("variant", [0, 3, 5, 6])
@pytest.mark.parametrize("factor", [False, True])
def test_short_keys_row_sums_in_fp32(H, dh, Lq, Lk, variant, factor):
    """Fewer than 512 keys: the row sum is fp32 over the probabilities before their rounding to bf16, on either kernel.
    One key with probability 1 and the others a little above 1/2, which all round down to 1/2 (by 0.35 %): with every
    value 1 the output is (1 + (Lk - 1) / 2) / (1 + (Lk - 1) p), which rounds to 1 - 2^-8; a sum over the rounded
    probabilities gives 1."""
    print(f"[case] row sums H={H} dh={dh} Lq={Lq} Lk={Lk} variant={variant} factor={factor}", flush=True)
    c = 1.0 if variant == 6 else np.log2(np.e) / np.sqrt(dh)
    # bf16 numbers a, b with 2^(c a b) = (1 + u 2^-8) / 2, u about 0.9 (bf16 rounds down below u = 1)
    a = _bf16(1.0 + np.arange(128) / 128)
    b = _bf16(-1.0 / (c * a) * (1 - 0.9 * 2.0 ** -8 / np.log(2)))
    u = (2.0 ** (c * a * b + 1) - 1) * 2 ** 8
    i = int(np.argmin(np.abs(u - 0.9)))
    assert 0.85 < u[i] < 0.95, u[i]
    p = 2.0 ** (c * a[i] * b[i])
    want = (1 + (Lk - 1) * 0.5) / (1 + (Lk - 1) * p)
    assert 1 - 2.0 ** -8 - 2.0 ** -10 < want < 1 - 2.0 ** -9 - 2.0 ** -10, want  # half a step of bf16 away from either neighbour
    kpad = 64 if variant == 3 else 128
    LqPad, LkPad = -(-Lq // 256) * 256, -(-Lk // kpad) * kpad
    Q = torch.zeros(H, LqPad, dh, dtype=torch.bfloat16, device=DEV)
    K = torch.zeros(H, LkPad, dh, dtype=torch.bfloat16, device=DEV)
    Q[:, :Lq, 0] = a[i]
    K[:, :Lk, 0] = b[i]
    K[:, 0, 0] = 0.0
    Vt = torch.ones(H * dh, LkPad, dtype=torch.bfloat16, device=DEV)
    out = torch.zeros(Lq, H * dh, dtype=torch.bfloat16, device=DEV)
    B.chorus_attention(Q, K, Vt, out, dev_f32(np.ones(Lk, np.float32)) if factor else None, Lq, Lk, variant)
    got = host_bf16(out)
    assert (got == 1 - 2.0 ** -8).all(), (got.min(), got.max(), want)


@pytest.mark.parametrize("D,H,Ls,Lt", [(256, 4, 128, 77), (1536, 12, 480, 226), (1536, 12, 480, 77), (512, 8, 300, 16), (512, 4, 200, 512),
                                       (1536, 12, 3300, 77)])
@pytest.mark.parametrize("factor", [False, True])
def test_block_cross_attention_equals_the_single_operations(D, H, Ls, Lt, factor):
    """The cross-attention branch of a block (the other branches' output weights are zero) against the calls it stands for,
    bit for bit. Over fewer than 512 keys its queries are the plain ones, rounded once, whichever kernel runs the
    attention; from 512 on they carry log2(e) / sqrt(dh)."""
    print(f"[case] block cross-attention D={D} H={H} Ls={Ls} Lt={Lt} factor={factor}", flush=True)
    dh, g = D // H, torch.Generator(device=DEV).manual_seed(Ls + Lt)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    F, t = 64, {}
    for n, o, i in (("qkv", 3 * D, D), ("o", D, D), ("cq", D, D), ("ckv", 2 * D, D), ("co", D, D), ("1", F, D), ("2", D, F)):
        zero = n in ("o", "2")
        t["w_" + n] = torch.zeros(o, i, dtype=torch.bfloat16, device=DEV) if zero else (rnd(o, i) * 0.05).bfloat16()
        t["b_" + n] = torch.zeros(o, device=DEV) if zero else rnd(o) * 0.1
    t.update(mod_table=rnd(6, D), g_q=rnd(D), g_k=rnd(D), g_cq=rnd(D), g_ck=rnd(D), ln3_w=rnd(D), ln3_b=rnd(D))
    w = B.DeviceBlock(t, B.BlockWeights(**{n: t[n].data_ptr() for n in B._W_FIELDS}))
    shape = B.make_block_shape(D, H, dh, F, Lt, (7, 24, 24))
    x, ctx, t_mod = rnd(Ls, D), rnd(Lt, D).bfloat16(), rnd(6, D)
    scale = torch.rand(Lt, device=DEV, generator=g) + 0.5 if factor else None
    got = x.clone()
    B.chorus_dit_block_step(shape, w, got, Ls, None, ctx, t_mod, scale, 1.25)

    LtPad, Lpad, long_keys = -(-Lt // 64) * 64, -(-Ls // 256) * 256, Lt >= 512
    h = torch.empty(Ls, D, dtype=torch.bfloat16, device=DEV)
    B.chorus_ln_modulate(x, h, t["ln3_w"], None, t["ln3_b"], None, False)
    q = torch.empty_like(h)
    B.chorus_gemm_bf16(h, t["w_cq"], B.EPI_BF16, q, t["b_cq"])
    qh = torch.empty(H, Lpad, dh, dtype=torch.bfloat16, device=DEV)
    B.chorus_qk_norm_rope(q, 0, t["g_cq"], qh, Ls, H, dh, None, (7, 24, 24), False, float(np.float32(np.log2(np.e)) / np.sqrt(np.float32(dh))) if long_keys else 1.0)
    kv = B.chorus_text_kv_project(shape, w, ctx).view(torch.bfloat16)
    k, v = kv[:H * LtPad * dh].view(H, LtPad, dh), kv[kv.numel() // 2:][:D * LtPad].view(D, LtPad)
    ao = torch.empty(Ls, D, dtype=torch.bfloat16, device=DEV)
    B.chorus_attention(qh, k, v, ao, scale, Ls, Lt, 6 if long_keys else 0)
    want = x.clone()
    B.chorus_gemm_bf16(ao, t["w_co"], B.EPI_RESID, want, t["b_co"], None, None, 1.25)
    assert torch.equal(got, want)
