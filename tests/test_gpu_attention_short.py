"""GPU parity of attention launches that leave compute units idle (128-row tiles throughout) and of short key sequences on
128-key tiles, the default choice there and the pre-scaled form that the block uses, with and without key factors."""
import numpy as np
import pytest

import synth
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
