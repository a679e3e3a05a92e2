"""GPU parity of attention over more tiles than the GPU has compute units, where workgroups walk over tiles: one tile more than units, ranges
that do not divide over the XCDs, rows and keys that end inside a tile, heads that change from tile to tile, with and without factors."""
import numpy as np
import pytest

import synth
from test_gpu_ops import _attn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dh,Lq,Lk", [
    (257, 64, 200, 512), (260, 128, 256, 513),   # a tile a head, just over one round
    (40, 64, 1700, 640), (37, 128, 1800, 1000),  # 280 and 296 tiles, five and eight tiles of keys: half tiles behind the walk
    (40, 128, 1700, 512), (66, 64, 2050, 520),   # four and five tiles of keys, 280 and 594 tiles
])
@pytest.mark.parametrize("variant", [5, 6])
@pytest.mark.parametrize("factor", [False, True])
def test_attention_walk(H, dh, Lq, Lk, variant, factor):
    print(f"[case] attention walk H={H} dh={dh} Lq={Lq} Lk={Lk} variant={variant} factor={factor}", flush=True)
    cs = (0.25 + 1.75 * synth.stream(Lk, "cs").random(Lk)).astype(np.float32) if factor else None
    _attn_case(H, dh, Lq, Lk, variant, col_scale=cs, q_std=2.0, seed=Lq + Lk, name="walk")
