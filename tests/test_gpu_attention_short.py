"""GPU parity of attention launches that leave compute units idle (128-row tiles throughout) and of short key sequences on
128-key tiles, the default choice there and the pre-scaled form that the block uses, with and without key factors."""
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
    (10, 64, 3300, 130),   # full tiles, less than a round: 64-key tiles without factors, 128-key tiles with
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
