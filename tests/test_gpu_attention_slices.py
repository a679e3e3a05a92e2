"""GPU parity of self-attention whose last tiles run in slices of the keys, each slice a workgroup that leaves its part for the last one
to add: against the same attention without slices, which the oracle tests cover, and the block that takes this way by itself."""
import pytest
import torch

from paper_2604_04451_amd import binding as B
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _case(H, dh, L, seed):
    g, LPad = torch.Generator(device=DEV).manual_seed(seed), -(-L // 256) * 256
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    q, k, v = (rnd(H, LPad, dh) * 2.0 * 1.4426950408889634 / dh ** 0.5).bfloat16(), rnd(H, LPad, dh).bfloat16(), rnd(H * dh, LPad).bfloat16()
    k[:, L:] = 0
    v[:, L:] = 0
    return q, k, v


def _scratch(tiles, slices, dh, fill):
    slab = (dh // 16 * 2 + 1) * 2 * 512 * 8
    n = -(-(2 * tiles + tiles * (slices - 1)) * 4 // 256) * 256 + tiles * (slices - 1) * slab
    return torch.full((n,), fill, dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("H,L,whole,slices", [
    (1, 513, 0, 2),     # five key tiles, the last with one key, in 2 + 3
    (2, 640, 2, 5),     # a key tile a slice; whole tiles in front
    (3, 1000, 5, 3),    # rows and keys that end inside a tile
    (2, 2303, 17, 4),   # one tile alone
    (1, 4096, 0, 2),
])
def test_slices_against_whole(H, dh, L, whole, slices):
    """Each side rounds the probabilities to bf16 against references of its own: two results of the same precision. A rounding is
    off by 2^-9 at most, 2^-9 / sqrt(3) on average, independent from key to key, and rows of N(0, 1) logits weigh hundreds of
    keys: the sums differ by less than one rounding of the output to bf16 does, 2^-9 / sqrt(3) on either side."""
    print(f"[case] attention slices H={H} dh={dh} L={L} whole={whole} slices={slices}", flush=True)
    q, k, v = _case(H, dh, L, L + H)
    k[0, L // 2] *= 8.0  # a key that some rows follow: references of their own in the slices
    want = torch.empty(L, H * dh, dtype=torch.bfloat16, device=DEV)
    B.chorus_attention(q, k, v, want, None, L, L, 6)
    tiles = -(-L // 256) * H - whole
    out = []
    for fill in (0, 255, 255):  # nothing in the scratch has to start at any value
        o = torch.zeros(L, H * dh, dtype=torch.bfloat16, device=DEV)
        out.append(B.chorus_attention_slices(q, k, v, o, L, whole, slices, _scratch(tiles, slices, dh, fill)))
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    rel = float((out[0].float() - want.float()).norm() / want.float().norm())
    assert rel < 3 * 2.0 ** -9 / 3 ** 0.5, rel
    with pytest.raises(B.ChorusError):
        B.chorus_attention_slices(q, k, v, o, L, whole, slices, _scratch(tiles, slices, dh, 0)[:-1])


def test_block_with_slices():
    """A block of 17000 tokens and four heads of 64 (its own choice: the last 12 tiles in four slices), three replays of a captured graph
    with other work in between against the same call outside."""
    D, H, Ls, F, Lt = 256, 4, 17000, 512, 64
    assert B.chorus_attention_slices_plan(Ls, H, 64, 256, 2 * Ls * D, 6 * Ls * D) == (256, 4)
    g = torch.Generator(device=DEV).manual_seed(7)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    t = {}
    for n, o, i in (("qkv", 3 * D, D), ("o", D, D), ("cq", D, D), ("ckv", 2 * D, D), ("co", D, D), ("1", F, D), ("2", D, F)):
        t["w_" + n], t["b_" + n] = (rnd(o, i) * 0.05).bfloat16(), rnd(o) * 0.1
    t.update(mod_table=rnd(6, D) * 0.3, g_q=rnd(D), g_k=rnd(D), g_cq=rnd(D), g_ck=rnd(D), ln3_w=rnd(D), ln3_b=rnd(D))
    w = B.DeviceBlock(t, B.BlockWeights(**{n: t[n].data_ptr() for n in B._W_FIELDS}))
    shape = B.make_block_shape(D, H, 64, F, Lt, (4, 68, 64))
    x, ctx, t_mod = rnd(Ls, D), rnd(Lt, D).bfloat16(), rnd(6, D) * 0.3
    ws = torch.full((B.chorus_dit_block_workspace_bytes(shape, Ls),), 255, dtype=torch.uint8, device=DEV)
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
