"""A block that projects its text beside the tokens gives the bits of one on a cached projection, which runs the same products
and norms in launches of their own: few and many text tokens, sizes on both sides of the line behind which each product takes
a launch of its own."""
import pytest
import torch

from paper_2604_04451_amd import binding as B

pytestmark = pytest.mark.gpu


# D, H, F, tokens, text tokens, and the kernel of the launch that takes both products (0: a launch each)
CASES = [(256, 4, 1024, 1, 1, 1), (256, 4, 1024, 64, 16, 1), (256, 4, 1024, 129, 130, 1), (512, 8, 1024, 300, 77, 1),
         (1536, 12, 2048, 300, 512, 5), (1536, 12, 2048, 480, 65, 5), (1536, 12, 2048, 800, 16, 0), (1536, 12, 2048, 900, 512, 5),
         (1536, 12, 2048, 300, 2048, 0), (1536, 12, 2048, 1500, 512, 0)]


@pytest.mark.parametrize("D,H,F,Ls,Lt", [c[:5] for c in CASES])
def test_text_beside_the_tokens(D, H, F, Ls, Lt):
    print(f"[case] block with its text D={D} Ls={Ls} Lt={Lt}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Ls)
    n = lambda *s, std=1.0: torch.randn(*s, generator=g, device="cuda") * std  # noqa: E731
    w = {"mod_table": n(6, D, std=0.1)}
    for k, o, i in (("qkv", 3 * D, D), ("o", D, D), ("cq", D, D), ("ckv", 2 * D, D), ("co", D, D), ("1", F, D), ("2", D, F)):
        w["w_" + k], w["b_" + k] = n(o, i, std=0.02).bfloat16(), n(o, std=0.05)
    for k in ("g_q", "g_k", "g_cq", "g_ck", "ln3_w"):
        w[k] = 1 + n(D, std=0.1)
    w["ln3_b"] = n(D, std=0.1)
    weights = B.DeviceBlock(w, B.BlockWeights(**{k: w[k].data_ptr() for k in B._W_FIELDS}))
    shape = B.make_block_shape(D, H, D // H, F, Lt, (4, 20, 20))
    x, ctx, t_mod, scale = n(Ls, D), n(Lt, D).bfloat16(), n(6, D, std=0.1), 1 + n(Lt, std=0.2).abs()
    ws = torch.empty(B.chorus_dit_block_workspace_bytes(shape, Ls), dtype=torch.uint8, device="cuda").fill_(255)
    a, b = x.clone(), x.clone()
    B.chorus_dit_block_step(shape, weights, a, Ls, None, ctx, t_mod, scale, 1.25, ws)
    kv = B.chorus_text_kv_project(shape, weights, ctx)
    B.chorus_dit_block_step_kv(shape, weights, b, Ls, None, kv, t_mod, scale, 1.25, ws.fill_(255))
    assert torch.isfinite(a).all() and torch.equal(a, b)
