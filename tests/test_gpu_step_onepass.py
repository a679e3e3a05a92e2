"""GPU parity of the one-pass patch embedding and the one-pass head + sampler update against the oracle, at the edges of
their tiles (16 and 64 tokens), on widths that are no multiple of a wave's row and on patch shapes other than 2 x 2; the
widths and patches beside them run the separate passes and are held to the same numbers."""
import numpy as np
import pytest
import torch

import synth
from oracle import chorus_oracle as O
from paper_2604_04451_amd import binding as B
from gpu_util import DEV, check, dev_f32, host

pytestmark = pytest.mark.gpu


def _weights(D, P, seed):
    w = {"w_patch": synth.round_bf16(synth.normal(seed, "op.wp", (D, P), 0.1)), "b_patch": synth.normal(seed, "op.bp", (D,), 0.1),
         "w_head": synth.round_bf16(synth.normal(seed, "op.wh", (P, D), 0.05)), "b_head": synth.normal(seed, "op.bh", (P,), 0.1),
         "head_table": synth.normal(seed, "op.ht", (2, D), 0.2)}
    return w, B.upload_glue_weights(w)


@pytest.mark.parametrize("tokens,D,C,patch", [(1, 64, 16, (2, 2)), (15, 192, 16, (2, 2)), (16, 256, 32, (1, 2)), (17, 1280, 4, (4, 4)),
                                              (63, 1536, 16, (2, 2)), (64, 320, 64, (1, 1)), (33, 768, 4, (2, 4)), (209, 512, 16, (2, 2)),
                                              (65, 1536, 16, (2, 2)), (5000, 256, 16, (2, 2)), (200, 1600, 16, (2, 2)), (97, 256, 32, (2, 2))])
@pytest.mark.parametrize("mode", ["euler", "region", "solver", "guided"])
def test_embed_and_head(tokens, D, C, patch, mode):
    print(f"[case] one pass tokens={tokens} D={D} C={C} patch={patch} {mode}", flush=True)
    ph, pw = patch
    grid = (3, 7, 10) if tokens < 1000 else (5, 30, 40)  # the latter: several groups of 16 tokens per workgroup
    shape = (C, grid[0], grid[1] * ph, grid[2] * pw)
    P, L, seed = C * ph * pw, grid[0] * grid[1] * grid[2], tokens + D
    w, glue = _weights(D, P, seed)
    lat, prev, SL = (synth.normal(seed, n, shape) for n in ("op.lat", "op.prev", "op.SL"))
    idx = np.sort(synth.stream(seed, "op.idx").permutation(L)[:tokens])
    t_head = synth.normal(seed, "op.th", (2, D), 0.2)
    didx = torch.from_numpy(idx.astype(np.int32)).to(DEV)
    pp = (1, ph, pw)
    toks, ptoks, stoks = (O.patchify(a.astype(np.float64), pp) for a in (lat, prev, SL))
    # patch embedding: bf16 weights exactly, the fp32 patch as a bf16 pair (2^-16 of each element)
    if P % 64 == 0:  # the embedding takes no other patches
        x = torch.empty(tokens, D, device=DEV)
        B.chorus_patch_embed(dev_f32(lat), didx, tokens, glue, D, x, patch)
        xref = O.patch_embed(toks[idx], w)
        check(host(x), xref, "x", max_abs=np.abs(xref).max() * 2 ** -12, rel_l2=2e-5)
    # head on rows of its own, so that its error is not the embedding's
    hx, hu = synth.normal(seed, "op.x", (tokens, D)) + 0.5, synth.normal(seed, "op.xu", (tokens, D))
    v = O.head(hx, w, t_head)
    edit = (synth.stream(seed, "op.edit").random(L) < 0.6).astype(np.uint8)
    hist = (synth.stream(seed, "op.hist").random(L) < 0.5).astype(np.uint8)
    d_lat, d_prev, cur = dev_f32(lat), dev_f32(prev), toks[idx]
    out, pout = toks.copy(), ptoks.copy()
    if mode in ("euler", "region"):
        new = cur - 0.3 * v
        B.chorus_head_update_region(d_lat, dev_f32(hx), tokens, didx, glue, dev_f32(t_head), -0.3,
                                    dev_f32(SL) if mode == "region" else None,
                                    torch.from_numpy(edit).to(DEV) if mode == "region" else None, patch)
        out[idx] = np.where(edit[idx][:, None] != 0, new, stoks[idx]) if mode == "region" else new
    else:
        if mode == "guided":
            u = O.head(hu, w, t_head)
            v = u + 3.0 * (v - u)
        cf = B.chorus_sampler_coefficients([1.0, 0.8, 0.5, 0.2, 0.0], 2, 2)
        x0 = cur - cf.sigma_s * v
        d = np.where(hist[idx][:, None] != 0, cf.c0 * x0 + cf.c1 * ptoks[idx], x0)
        out[idx] = np.where(edit[idx][:, None] != 0, cf.rho * cur + cf.A * d, stoks[idx])
        pout[idx] = x0
        B.chorus_head_update_solver(d_lat, dev_f32(hx), tokens, didx, glue, dev_f32(t_head), cf, d_prev,
                                    torch.from_numpy(hist).to(DEV), dev_f32(hu) if mode == "guided" else None, 3.0, dev_f32(SL),
                                    torch.from_numpy(edit).to(DEV), patch)
    # v carries one bf16 rounding of its D operands (2^-9 each, random signs): 2^-9 |h| |w| per column, guidance three to
    # five times that; the latent takes a fraction of it
    vtol = 5.0 * 2 ** -9 * np.linalg.norm(w["w_head"], axis=1).max() * 2.0 * (5.0 if mode == "guided" else 1.0)
    check(host(d_lat), O.unpatchify(out, shape, pp), "latent", max_abs=vtol, rel_l2=5e-3)
    check(host(d_prev), O.unpatchify(pout, shape, pp), "x0_prev", max_abs=vtol, rel_l2=5e-3)
    untouched = np.ones(L, bool)
    untouched[idx] = False
    assert np.array_equal(O.patchify(host(d_lat), pp)[untouched], O.patchify(lat, pp)[untouched])
