"""GPU parity of attention over more tiles than the GPU has compute units, where workgroups walk over tiles: one tile more than units, ranges
that do not divide over the XCDs, rows and keys that end inside a tile, heads that change from tile to tile, with and without factors."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import DEV, check
from paper_2604_04451_amd import binding as B
from test_gpu_ops import _attn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dh,Lq,Lk", [
    (257, 64, 200, 512), (260, 128, 256, 513),   # a tile a head, just over one round
    (40, 64, 1700, 640), (37, 128, 1800, 1000),  # 280 and 296 tiles, five and eight tiles of keys: half tiles behind the walk
    (40, 128, 1700, 512), (66, 64, 2050, 520),   # four and five tiles of keys, 280 and 594 tiles
    (40, 128, 3300, 512), (38, 128, 3000, 512),  # 520 and 456 tiles of four tiles of keys
    (47, 64, 7000, 512), (60, 64, 5900, 513),    # 1316 and 1440 tiles: two shares a unit
    (24, 64, 5600, 2048), (24, 64, 5600, 2049),  # the longest keys that are walked, two tiles a share, and one more
])
@pytest.mark.parametrize("variant", [5, 6])
@pytest.mark.parametrize("factor", [False, True])
def test_attention_walk(H, dh, Lq, Lk, variant, factor):
    print(f"[case] attention walk H={H} dh={dh} Lq={Lq} Lk={Lk} variant={variant} factor={factor}", flush=True)
    cs = (0.25 + 1.75 * synth.stream(Lk, "cs").random(Lk)).astype(np.float32) if factor else None
    _attn_case(H, dh, Lq, Lk, variant, col_scale=cs, q_std=2.0, seed=Lq + Lk, name="walk")


@pytest.mark.parametrize("variant", [0, 5, 6])
@pytest.mark.parametrize("H,dh,Lq,Lk", [(40, 128, 1700, 512), (40, 128, 3300, 512), (12, 128, 10000, 640),
                                         (66, 64, 2050, 520)])  # 280, 520, 480 and 594 tiles
def test_attention_walk_low_logits(H, dh, Lq, Lk, variant):
    """A shift of all logits of a row changes nothing, in whichever of a workgroup's tiles the row is: a third of the rows has logits about
    -150 (in natural units, far below what exp2 against a reference of 0 can hold), a third about -85 (at its edge), a third about 0."""
    print(f"[case] attention walk low logits H={H} dh={dh} Lq={Lq} Lk={Lk} variant={variant}", flush=True)
    g, LqPad, LkPad = torch.Generator(device=DEV).manual_seed(Lq), -(-Lq // 256) * 256, -(-Lk // 128) * 128
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    shift = torch.tensor([-150.0, -85.0, 0.0], device=DEV)[torch.arange(LqPad, device=DEV) % 3]
    q = rnd(H, LqPad, dh) + (shift / 40.0).view(1, -1, 1)  # every component of a key is 40 / sqrt(dh) off: a row's logits move by its shift
    c = 1.4426950408889634 / dh ** 0.5 if variant == 6 else 1.0
    q = (q * c).bfloat16()
    k = (0.5 * rnd(H, LkPad, dh) + 40.0 / dh ** 0.5).bfloat16()
    v = rnd(H * dh, LkPad).bfloat16()
    k[:, Lk:], v[:, Lk:] = 0, 0
    at = torch.arange(LkPad, device=DEV)
    vt = v[:, at // 16 * 16 + (at // 4 % 2) * 8 + at // 8 % 2 * 4 + at % 4].contiguous()  # chorus_v_transpose's order
    out = torch.full((Lq, H * dh), 9.0, dtype=torch.bfloat16, device=DEV)
    B.chorus_attention(q, k, vt, out, None, Lq, Lk, variant)
    ref = torch.empty(Lq, H * dh, dtype=torch.float64, device=DEV)
    for h in range(H):
        p = (q[h, :Lq].double() / c @ k[h, :Lk].double().T.contiguous() / dh ** 0.5).softmax(1)
        ref[:, h * dh:(h + 1) * dh] = p @ v[h * dh:(h + 1) * dh, :Lk].double().T.contiguous()
    ref = ref.cpu().numpy()
    check(out.float().cpu().numpy(), ref, "walk, low logits", max_abs=max(np.abs(ref).max() * 2 ** -7, 2e-3), rel_l2=5e-3)
