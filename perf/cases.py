"""The work that a serving program has this library do, as cases that can be timed and compared.

`listed()` names the fixed cases, `draw(rng)` gives more of the same ranges, `prepare` makes on the GPU what a program
holds before the call (inputs, weights, workspaces), `run` is one pass through the public entry points, `work` the
bytes and operations that the pass cannot do without, `exact` the same results in 64 bits in plain torch, and
`tolerance` how far another correct implementation at the same precision may be from this one.

Kinds of case
  lookup     chorus_cache_lookup: top-1 cosine over the fp32 prompt-embedding cache, once per request
  batch      chorus_cache_lookup_batch: the k best entries for each of a queue of requests
  lowprec    chorus_cache_lookup_lowprec: the lookup over a bf16 or FP8 copy of a large cache
  masks      key-frame pixel masks -> token masks (M_base, M_edit, M_see) -> list of selected tokens, once per request
  step_io    what surrounds the block stack in every denoising step: patch embedding of the selected tokens, output
             head and multistep sampler update with Eq. 6, with and without classifier-free guidance
  block      one DiT block in place on the residual stream; a request runs it blocks x steps times
  request    text projection, timestep rows, and the whole three-stage run on a small model
"""
import math

import torch

from paper_2604_04451_amd import binding as B

DEV = "cuda"

# widths of a block: hidden, heads, FFN, raw text embedding
_WIDTHS = {"tiny": (256, 4, 1024, 256), "1p3b": (1536, 12, 8960, 4096), "14b": (5120, 40, 13824, 4096)}
_GRID = {"tiny": (4, 8, 8), "1p3b": (21, 30, 52), "14b": (21, 45, 80)}  # 4 x 8 x 8, 480p and 720p token grids


def _block(name, width, grid, tokens, text, tgaa, kv):
    return {"name": name, "kind": "block", "width": width, "T": grid[0], "Hg": grid[1], "Wg": grid[2], "tokens": tokens,
            "text": text, "tgaa": tgaa, "kv": kv}


def listed():
    g, h, t = _GRID["1p3b"], _GRID["14b"], _GRID["tiny"]
    return [
        # the smallest call: a thousand entries of a 768-d text encoder, the store size the method is described with
        {"name": "lookup_1000x768", "kind": "lookup", "N": 1000, "d": 768},
        # the benchmark's cache: one prompt of a 4096-d text encoder against 4096 entries
        {"name": "lookup_4096x4096", "kind": "lookup", "N": 4096, "d": 4096},
        # a full queue: 32 waiting prompts, 8 candidates each, against the same cache
        {"name": "batch_32x8_4096x4096", "kind": "batch", "N": 4096, "d": 4096, "Q": 32, "k": 8},
        # a cache large enough that its FP8 copy is what gets scanned; the prompt is close to an entry (a hit)
        {"name": "lowprec_fp8_16384x4096", "kind": "lowprec", "N": 16384, "d": 4096, "fp8": True, "near": True},
        # masks of an 81-frame 480 x 832 clip with 21 key frames
        {"name": "masks_480p", "kind": "masks", "Tp": 81, "Kf": 21, "Hp": 480, "Wp": 832, "r_edit": 1, "r_see": 2},
        # a full 480p step of the 1.3B model around its blocks, with guidance (the 50-step models run it)
        {"name": "step_io_480p", "kind": "step_io", "width": "1p3b", "T": g[0], "Hg": g[1], "Wg": g[2], "tokens": 32760,
         "cfg": True, "region": False},
        # the tiny block on half of its tokens with amplification: launches and latency
        _block("block_tiny_128", "tiny", t, 128, 16, True, False),
        # 1.3B stage-2 steps: a small region (an odd number of tokens) and the benchmark's 40 % region
        _block("block_1p3b_3271", "1p3b", g, 3271, 512, True, True),
        _block("block_1p3b_13104", "1p3b", g, 13104, 512, True, True),
        # 1.3B stage-3 step: every token of the 480p clip, text keys and values projected once per request
        _block("block_1p3b_32760", "1p3b", g, 32760, 512, False, True),
        # the largest: a 14B block on every token of a 720p clip
        _block("block_14b_75600", "14b", h, 75600, 512, False, True),
        # a whole four-step request on the 1.3B widths, small grid, two blocks: stages 1, 2, 3, 3
        {"name": "request_1p3b_1200", "kind": "request", "width": "1p3b", "T": 5, "Hg": 12, "Wg": 20, "blocks": 2,
         "text": 512, "N": 64, "d": 4096, "region": 0.4, "solver": 1, "cfg": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_grid(rng, least, most):
    """A token grid of `least` to `most` tokens, log-uniform: 1 to 21 latent frames of anything from square to 2 : 1."""
    tokens = _log(rng, least, most)
    T = rng.randint(1, 21)
    while T > 1 and tokens < 16 * T:
        T -= 1
    Hg = max(1, int(math.sqrt(tokens / T / rng.uniform(1.0, 2.0))))
    Wg = max(1, tokens // (T * Hg))
    return T, Hg, Wg


def draw(rng):
    kind = rng.choice(["lookup", "batch", "lowprec", "masks", "step_io", "block", "block", "block", "request"])
    if kind == "lookup":
        return {"kind": kind, "N": _log(rng, 200, 65536), "d": 4 * _log(rng, 64, 1024)}
    if kind == "batch":
        return {"kind": kind, "N": _log(rng, 500, 20000), "d": 4 * _log(rng, 64, 1024), "Q": rng.randint(2, 48),
                "k": rng.choice([1, 4, 8, 16, 50])}
    if kind == "lowprec":
        return {"kind": kind, "N": _log(rng, 2000, 65536), "d": 16 * _log(rng, 24, 256), "fp8": rng.random() < 0.5,
                "near": rng.random() < 0.7}
    if kind == "masks":
        Tp = 1 + 4 * rng.randint(0, 30)
        re = rng.randint(0, 2)
        return {"kind": kind, "Tp": Tp, "Kf": max(1, min(Tp, rng.randint(1, 31))), "Hp": _log(rng, 160, 1088),
                "Wp": rng.choice([16 * rng.randint(12, 120), rng.randint(200, 1920), 854]), "r_edit": re,
                "r_see": re + rng.randint(0, 4)}
    if kind == "step_io":
        width = rng.choice(["tiny", "1p3b", "1p3b", "14b"])
        T, Hg, Wg = _draw_grid(rng, 64, {"tiny": 4096, "1p3b": 32760, "14b": 75600}[width])
        L = T * Hg * Wg
        region = rng.random() < 0.5
        return {"kind": kind, "width": width, "T": T, "Hg": Hg, "Wg": Wg,
                "tokens": max(1, int(L * rng.uniform(0.1, 0.95))) if region else L, "cfg": rng.random() < 0.5,
                "region": region}
    if kind == "block":
        width = rng.choice(["tiny", "1p3b", "1p3b", "1p3b", "14b"])
        T, Hg, Wg = _draw_grid(rng, 96, {"tiny": 4096, "1p3b": 32760, "14b": 40000}[width])
        L = T * Hg * Wg
        c = _block(None, width, (T, Hg, Wg), L if rng.random() < 0.4 else max(1, int(L * rng.uniform(0.1, 0.95))),
                   rng.choice([512, 512, 512, 16, 77, 226]), rng.random() < 0.5, rng.random() < 0.7)
        c.pop("name")
        return c
    width = rng.choice(["tiny", "1p3b", "1p3b"])
    T, Hg, Wg = _draw_grid(rng, 96, 4096)
    return {"kind": kind, "width": width, "T": T, "Hg": Hg, "Wg": Wg, "blocks": rng.randint(1, 4),
            "text": rng.choice([512, 512, 77, 226]), "N": _log(rng, 16, 1024), "d": rng.choice([768, 1024, 4096]),
            "region": rng.uniform(0.1, 0.9), "solver": rng.choice([1, 2]), "cfg": rng.random() < 0.4}


# ------------------------------------------------------------------------------------------------ inputs

class _Gen:
    """Seeded draws on the GPU, in the order in which prepare() asks for them."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, shape, std=1.0, mean=0.0, dtype=torch.float32):
        t = torch.empty(shape, dtype=torch.float32, device=DEV)
        t.normal_(mean, std, generator=self.g)
        return t.to(dtype)

    def subset(self, L, n):
        """n of L token ids, ascending."""
        return torch.randperm(L, generator=self.g, device=DEV)[:n].sort().values.to(torch.int32)

    def below(self, n):
        return int(torch.randint(0, n, (1,), generator=self.g, device=DEV).item())


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _unit(t):
    return t / t.norm(dim=-1, keepdim=True)


def _cache(g, N, d):
    """Clustered unit rows (up to 256 centroids), as prompt embeddings are."""
    cen = _unit(g.normal((min(256, N), d)))
    which = torch.randint(0, cen.shape[0], (N,), generator=g.g, device=DEV)
    return _unit(cen[which] + g.normal((N, d), 0.5 / math.sqrt(d)))


def _near(g, cache, row):
    """A prompt like entry `row`: cosine about 0.9."""
    return _unit(cache[row] + g.normal((cache.shape[1],), 0.5 / math.sqrt(cache.shape[1])))


def _block_weights(g, D, F):
    """Matrices N(0, 0.02) in bf16, biases, norm gains and gates of the size a trained block has, so that no branch vanishes."""
    bf = torch.bfloat16
    w = {"mod_table": g.normal((6, D), 0.1)}
    w["mod_table"][2] += 0.5
    w["mod_table"][5] += 0.5
    for n, o, i in (("qkv", 3 * D, D), ("o", D, D), ("cq", D, D), ("ckv", 2 * D, D), ("co", D, D), ("1", F, D), ("2", D, F)):
        w["w_" + n] = g.normal((o, i), 0.02, dtype=bf)
        w["b_" + n] = g.normal((o,), 0.05)
    for n in ("g_q", "g_k", "g_cq", "g_ck"):
        w[n] = g.normal((D,), 0.1, 1.2)
    w["ln3_w"] = g.normal((D,), 0.1, 1.0)
    w["ln3_b"] = g.normal((D,), 0.1)
    return w


def _glue_weights(g, D, P, text_dim):
    bf = torch.bfloat16
    w = {"w_patch": g.normal((D, P), 0.1, dtype=bf), "b_patch": g.normal((D,), 0.05), "w_head": g.normal((P, D), 0.02, dtype=bf),
         "b_head": g.normal((P,), 0.05), "head_table": g.normal((2, D), 0.1)}
    if text_dim:
        w.update({"w_text1": g.normal((D, text_dim), 0.02, dtype=bf), "b_text1": g.normal((D,), 0.05),
                  "w_text2": g.normal((D, D), 0.02, dtype=bf), "b_text2": g.normal((D,), 0.05)})
    return w


def _device_block(w):
    return B.DeviceBlock(w, B.BlockWeights(**{n: w[n].data_ptr() for n in B._W_FIELDS}))


def _device_glue(w):
    return B.DeviceGlue(w, B.GlueWeights(**{n: w[n].data_ptr() for n in ("w_patch", "b_patch", "w_head", "b_head", "head_table")}))


def _device_time(w, D):
    tw = B.DeviceTime.__new__(B.DeviceTime)
    tw.tensors, tw.freq_dim, tw.D = w, w["w_t1"].shape[1], D
    tw.cstruct = B.TimeWeights(*[w[n].data_ptr() for n in ("w_t1", "b_t1", "w_t2", "b_t2", "w_tp", "b_tp")])
    return tw


def _result_views(out):
    """The result words of a lookup under their types: index, score, hit."""
    return {"index": out[0:1], "score": out[1:2].view(torch.float32), "hit": out[2:3]}


_TAU = 0.75
_GUIDANCE = 5.0
_SIGMAS = [1.0, 0.75, 0.5, 0.25, 0.0]


def prepare(case, seed):
    g = _Gen(seed)
    kind = case["kind"]
    s = {"case": case}
    if kind in ("lookup", "lowprec", "batch"):
        N, d = case["N"], case["d"]
        s["cache"] = _cache(g, N, d)
        if kind == "batch":
            rows = torch.randint(0, N, (case["Q"],), generator=g.g, device=DEV)
            s["queries"] = _unit(s["cache"][rows] + g.normal((case["Q"], d), 0.5 / math.sqrt(d)))
            s["ws"] = _bytes(B.load().chorus_cache_lookup_batch_workspace_bytes(N, d, case["Q"]))
            return s
        s["query"] = _near(g, s["cache"], g.below(N)) if case.get("near", True) else _unit(g.normal((d,)))
        s["out"] = torch.zeros(3, dtype=torch.int32, device=DEV)
        s["views"] = _result_views(s["out"])
        if kind == "lookup":
            s["ws"] = _bytes(B.load().chorus_cache_lookup_workspace_bytes(N))
        else:
            s["fmt"] = B.LP_FP8 if case["fp8"] else B.LP_BF16
            s["copy"] = B.chorus_cache_lowprec_store(s["cache"], s["fmt"])
            s["n"] = torch.zeros(1, dtype=torch.int32, device=DEV)
            s["ws"] = _bytes(B.load().chorus_cache_lookup_lowprec_workspace_bytes(N))
        return s
    if kind == "masks":
        Tp, Kf, Hp, Wp = case["Tp"], case["Kf"], case["Hp"], case["Wp"]
        yy = torch.arange(Hp, device=DEV).view(Hp, 1).float()
        xx = torch.arange(Wp, device=DEV).view(1, Wp).float()
        m = torch.zeros(Kf, Hp, Wp, dtype=torch.bool, device=DEV)
        u = torch.rand((2, 6), generator=g.g, device=DEV).tolist()
        for cy, cx, vy, vx, asp, ph in u:  # two objects that drift from key frame to key frame
            ry, rx = Hp * (0.12 + 0.1 * asp), Wp * (0.22 - 0.1 * asp)
            for k in range(Kf):
                a = (yy - Hp * (0.2 + 0.6 * cy + 0.02 * (vy - 0.5) * k)) / (ry * (1 + 0.1 * math.sin(0.7 * k + ph)))
                b = (xx - Wp * (0.2 + 0.6 * cx + 0.02 * (vx - 0.5) * k)) / rx
                m[k] |= a * a + b * b <= 1.0
        s["keys"] = m.to(torch.uint8)
        s["frame_key"] = (torch.arange(Tp, device=DEV) * Kf // Tp).clamp(max=Kf - 1).to(torch.int32)
        To, Ho, Wo = 1 + (Tp - 1 + 3) // 4, -(-Hp // 16), -(-Wp // 16)
        s["base"] = torch.empty(To, Ho, Wo, dtype=torch.uint8, device=DEV)
        s["idx"] = torch.zeros(To * Ho * Wo, dtype=torch.int32, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        s["ws"] = _bytes(B.load().chorus_region_compact_workspace_bytes(To * Ho * Wo))
        re, rs = case["r_edit"], case["r_see"]
        s["r_edit"], s["r_see"] = (min(re, 1), re, re), (min(rs, 1), rs, rs)
        return s
    D, H, F, text_dim = _WIDTHS[case["width"]]
    grid = (case["T"], case["Hg"], case["Wg"])
    L = grid[0] * grid[1] * grid[2]
    if kind == "block":
        Ls, Lt = case["tokens"], case["text"]
        s["w"] = _block_weights(g, D, F)
        s["weights"] = _device_block(s["w"])
        s["shape"] = B.make_block_shape(D, H, D // H, F, Lt, grid)
        s["x"] = g.normal((Ls, D))
        s["idx"] = g.subset(L, Ls) if Ls < L else None
        s["ctx"] = g.normal((Lt, D), dtype=torch.bfloat16)
        s["t_mod"] = g.normal((6, D), 0.1)
        s["scale"], s["gamma_o"] = None, 1.0
        if case["tgaa"]:  # amplification on a third of the text tokens
            s["scale"] = torch.where(torch.rand((Lt,), generator=g.g, device=DEV) < 0.33, 1.5, 1.0).float()
            s["gamma_o"] = 1.25
        s["ws"] = _bytes(B.chorus_dit_block_workspace_bytes(s["shape"], Ls))
        if case["kv"]:
            s["kv"] = B.chorus_text_kv_project(s["shape"], s["weights"], s["ctx"])
        return s
    latent_shape = (16, grid[0], 2 * grid[1], 2 * grid[2])
    if kind == "step_io":
        Ls = case["tokens"]
        s["w"] = _glue_weights(g, D, 64, 0)
        s["glue"] = _device_glue(s["w"])
        s["idx"] = g.subset(L, Ls) if Ls < L else None
        s["latent"] = g.normal(latent_shape)
        s["x0_prev"] = g.normal(latent_shape)
        s["SL"], s["edit"], s["hist"] = None, None, None
        if case["region"]:  # stage 2: the inner part of the selection is edited, the rest keeps the source latent
            s["SL"] = g.normal(latent_shape)
            keep = (torch.rand((L,), generator=g.g, device=DEV) < 0.6).to(torch.uint8)
            see = torch.zeros(L, dtype=torch.uint8, device=DEV)
            see[s["idx"].long() if s["idx"] is not None else slice(None)] = 1
            s["edit"], s["hist"] = keep * see, see
        s["t_head"] = g.normal((2, D), 0.1)
        s["coef"] = B.chorus_sampler_coefficients(_SIGMAS, 2, 2)
        s["x"] = torch.empty(Ls, D, device=DEV)
        s["x_uncond"] = g.normal((Ls, D)) if case["cfg"] else None
        lib = B.load()
        s["ws"] = _bytes(max(lib.chorus_glue_workspace_bytes(D, 64, Ls),
                             lib.chorus_head_solver_workspace_bytes(D, 64, Ls, int(case["cfg"]))))
        return s
    # request
    Lt, N, d, n = case["text"], case["N"], case["d"], case["blocks"]
    s["w"] = [_block_weights(g, D, F) for _ in range(n)]
    s["weights"] = [_device_block(w) for w in s["w"]]
    s["blocks"] = B.block_array(s["weights"])
    s["gw"] = _glue_weights(g, D, 64, text_dim)
    s["glue"] = _device_glue(s["gw"])
    s["tw"] = {"w_t1": g.normal((D, 256), 0.02, dtype=torch.bfloat16), "b_t1": g.normal((D,), 0.02),
               "w_t2": g.normal((D, D), 0.02, dtype=torch.bfloat16), "b_t2": g.normal((D,), 0.02),
               "w_tp": g.normal((6 * D, D), 0.02, dtype=torch.bfloat16), "b_tp": g.normal((6 * D,), 0.02)}
    s["time"] = _device_time(s["tw"], D)
    s["model"] = B.make_model_shape(B.make_block_shape(D, H, D // H, F, Lt, grid), latent_shape, (2, 2), n)
    s["text"] = g.normal((Lt, text_dim), dtype=torch.bfloat16)
    s["ctx"] = torch.empty(Lt, D, dtype=torch.bfloat16, device=DEV)
    s["text_u"] = g.normal((Lt, text_dim), dtype=torch.bfloat16) if case["cfg"] else None
    s["ctx_u"] = torch.empty(Lt, D, dtype=torch.bfloat16, device=DEV) if case["cfg"] else None
    s["t_mods"], s["t_heads"] = torch.empty(4, 6, D, device=DEV), torch.empty(4, 2, D, device=DEV)
    s["noise"] = g.normal(latent_shape)
    s["latent"] = torch.empty(latent_shape, device=DEV)
    s["cache"] = _cache(g, N, d)
    s["cache_latents"] = g.normal((N, 1) + latent_shape)
    s["near"] = g.below(N)
    s["query"] = _near(g, s["cache"], s["near"])
    see = torch.zeros(L, dtype=torch.uint8, device=DEV)
    see[g.subset(L, max(1, int(L * case["region"]))).long()] = 1
    s["see"] = see
    s["edit"] = see * (torch.rand((L,), generator=g.g, device=DEV) < 0.7).to(torch.uint8)
    s["tdiff"] = (torch.rand((Lt,), generator=g.g, device=DEV) < 0.33).to(torch.uint8)
    lib = B.load()
    s["ws"] = _bytes(B.chorus_denoise_run_workspace_bytes(s["model"], N))
    s["ws_text"] = _bytes(lib.chorus_text_project_workspace_bytes(Lt, D))
    s["ws_time"] = _bytes(lib.chorus_time_mod_workspace_bytes(D, 256))
    return s


# ------------------------------------------------------------------------------------------------ one pass

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "lookup":
        B.chorus_cache_lookup(s["cache"], s["query"], _TAU, s["out"], s["ws"])
        return s["views"]
    if kind == "batch":
        idx, score, hit = B.chorus_cache_lookup_batch(s["cache"], s["queries"], _TAU, case["k"], s["ws"])
        return {"index": idx, "score": score, "hit": hit}
    if kind == "lowprec":
        B.chorus_cache_lookup_lowprec(s["cache"], s["copy"], s["fmt"], s["query"], _TAU, s["out"], s["n"], s["ws"])
        return s["views"]
    if kind == "masks":
        B.chorus_mask_project(s["keys"], s["frame_key"], case["Tp"], (4, 16, 16), 1, s["base"])
        edit, see = B.chorus_mask_hierarchy(s["base"], s["r_edit"], s["r_see"])
        B.chorus_region_compact(see, s["idx"], s["count"], s["ws"])
        return {"base": s["base"], "edit": edit, "see": see, "idx": s["idx"], "count": s["count"]}
    if kind == "block":
        if case["kv"]:
            B.chorus_dit_block_step_kv(s["shape"], s["weights"], s["x"], case["tokens"], s["idx"], s["kv"], s["t_mod"],
                                       s["scale"], s["gamma_o"], s["ws"])
        else:
            B.chorus_dit_block_step(s["shape"], s["weights"], s["x"], case["tokens"], s["idx"], s["ctx"], s["t_mod"],
                                    s["scale"], s["gamma_o"], s["ws"])
        return s["x"]
    if kind == "step_io":
        B.chorus_patch_embed(s["latent"], s["idx"], case["tokens"], s["glue"], s["x"].shape[1], s["x"], ws=s["ws"])
        B.chorus_head_update_solver(s["latent"], s["x"], case["tokens"], s["idx"], s["glue"], s["t_head"], s["coef"],
                                    s["x0_prev"], s["hist"], s["x_uncond"], _GUIDANCE if case["cfg"] else 1.0, s["SL"],
                                    s["edit"], ws=s["ws"])
        return {"x": s["x"], "latent": s["latent"], "x0_prev": s["x0_prev"]}
    B.chorus_stage1_copy(s["latent"], s["noise"])
    B.chorus_text_project(s["text"], s["glue"], s["ctx"], s["ws_text"])
    if case["cfg"]:
        B.chorus_text_project(s["text_u"], s["glue"], s["ctx_u"], s["ws_text"])
    for i in range(4):
        B.chorus_time_mod(1000.0 * _SIGMAS[i], s["time"], s["t_mods"][i], s["t_heads"][i], s["ws_time"])
    r = B.chorus_denoise_run(s["model"], s["blocks"], s["glue"], s["latent"], s["cache"], s["cache_latents"], s["query"],
                             _TAU, _SIGMAS, s["t_mods"], s["t_heads"], s["ctx"], tdiff=s["tdiff"], mask_see=s["see"],
                             mask_edit=s["edit"], sched={"gamma_override": 1.5}, ws=s["ws"], solver_order=case["solver"],
                             text_ctx_uncond=s["ctx_u"], guidance=2.0 if case["cfg"] else 1.0, latent_steps=[1])
    return {"latent": s["latent"], "index": r["index"], "K1": r["K1"], "K2": r["K2"], "Ls": r["Ls"]}


# ------------------------------------------------------------------------------------------------ what a pass needs

def _block_work(case, tokens, kv=None):
    D, _, F, _ = _WIDTHS[case["width"]]
    Lt = case["text"]
    kv = case["kv"] if kv is None else kv
    weights = 2.0 * (3 * D * D + 3 * D * D + 2 * D * F + (0 if kv else 2 * D * D))
    flops = 4.0 * tokens * tokens * D + 2.0 * tokens * D * (6 * D + 2 * F) + 4.0 * tokens * Lt * D + (0 if kv else 4.0 * Lt * D * D)
    return weights + 8.0 * tokens * D + 2.0 * Lt * D * (2 if kv else 1), flops


def work(case):
    kind = case["kind"]
    if kind == "lookup":
        return {"bytes": 4.0 * case["d"] * (case["N"] + 1) + 12, "flops": 4.0 * case["N"] * case["d"]}
    if kind == "batch":
        N, d, Q, k = case["N"], case["d"], case["Q"], case["k"]
        return {"bytes": 4.0 * d * (N + Q) + Q * (8.0 * k + 4), "flops": 2.0 * N * d * (Q + 1)}
    if kind == "lowprec":
        return {"bytes": case["N"] * case["d"] * (1.0 if case["fp8"] else 2.0) + 8.0 * case["d"], "flops": 4.0 * case["N"] * case["d"]}
    if kind == "masks":
        L = (1 + (case["Tp"] - 1 + 3) // 4) * -(-case["Hp"] // 16) * -(-case["Wp"] // 16)
        return {"bytes": float(case["Kf"]) * case["Hp"] * case["Wp"] + 5.0 * L, "flops": 0.0}
    if kind == "block":
        b, f = _block_work(case, case["tokens"])
        return {"bytes": b, "flops": f}
    if kind == "step_io":
        D = _WIDTHS[case["width"]][0]
        L, n = case["T"] * case["Hg"] * case["Wg"], 2 if case["cfg"] else 1
        cells = case["tokens"] * 64 * 4.0
        return {"bytes": case["tokens"] * D * 4.0 * (n + 1) + cells * (6 if case["region"] else 5) + 256.0 * D + L,
                "flops": 2.0 * case["tokens"] * D * 64 * (n + 1)}
    L = case["T"] * case["Hg"] * case["Wg"]
    n, Ls = 2 if case["cfg"] else 1, max(1, int(L * case["region"]))
    D, _, _, text_dim = _WIDTHS[case["width"]]
    b = f = 0.0
    for tokens in (Ls, L, L):
        bb, bf = _block_work(case, tokens, kv=True)
        b, f = b + case["blocks"] * n * bb, f + case["blocks"] * n * bf
        f += 2.0 * tokens * D * 64 * (n + 1)
    f += n * (case["blocks"] * 4.0 * case["text"] * D * D + 2.0 * case["text"] * D * (text_dim + D)) + 4 * 2.0 * 7 * D * D
    b += n * (case["blocks"] * 4.0 * D * D + 2.0 * D * (text_dim + D)) + 4 * 14.0 * D * D + 4.0 * case["N"] * case["d"] + 16.0 * L * 64
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind == "masks":
        return "exact"
    if kind in ("lookup", "lowprec", "batch"):  # fp32 sums of up to 4096 products; a tie may swap two neighbours
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.005 if kind == "batch" else 0.0}
    # measured against the 64-bit results over listed and drawn cases: block 0.0003 to 0.004, step_io up to 0.0016,
    # request up to 0.002 (bf16 operands at every product, fp32 residual stream); about four times that
    if kind == "block":
        return {"rel": 1e-2, "max": 0.15}
    if kind == "step_io":
        return {"rel": 6e-3, "max": 0.15}
    return {"rel": 1e-2, "max": 0.2}


# ------------------------------------------------------------------------------------------------ 64-bit results

def _f(t):
    return t.double()


def _linear(x, w, b):
    return x @ _f(w).T + _f(b)


def _layernorm(x):
    m = x.mean(-1, keepdim=True)
    return (x - m) / ((x - m).square().mean(-1, keepdim=True) + 1e-6).sqrt()


def _rms(z, gain):
    return z / (z.square().mean(-1, keepdim=True) + 1e-6).sqrt() * _f(gain)


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x * x * x)))


def _rope(z, idx, grid, H):
    """Rotation of the pairs (2p, 2p + 1) by pos * 10000^(-2p / g) in three groups of a head's dimensions: t, h, w."""
    n, D = z.shape
    dh = D // H
    s6 = dh // 6
    ang, i = [], _f(idx)
    pos = (torch.floor(i / (grid[1] * grid[2])), torch.floor(i / grid[2]) % grid[1], i % grid[2])
    for size, p in zip((dh - 4 * s6, 2 * s6, 2 * s6), pos):
        e = torch.arange(0, size, 2, dtype=torch.float64, device=z.device) / size
        ang.append(p[:, None] * torch.pow(torch.tensor(10000.0, dtype=torch.float64, device=z.device), -e)[None, :])
    a = torch.cat(ang, 1)[:, None, :]
    c, sn = a.cos(), a.sin()
    zh = z.view(n, H, dh // 2, 2)
    return torch.stack((zh[..., 0] * c - zh[..., 1] * sn, zh[..., 0] * sn + zh[..., 1] * c), -1).reshape(n, D)


def _attend(q, k, v, H, scale=None):
    """Softmax attention per head; `scale` multiplies the logit of each key. Logits are small enough for exp as they are."""
    n, D = q.shape
    dh = D // H
    out = torch.empty_like(q)
    rows = max(1, (1 << 28) // k.shape[0])
    for h in range(H):
        c = slice(h * dh, (h + 1) * dh)
        kh, vh = k[:, c].t().contiguous(), v[:, c].contiguous()
        if scale is not None:
            kh = kh * _f(scale)
        for r in range(0, n, rows):
            p = (q[r:r + rows, c] / math.sqrt(dh)) @ kh
            p.exp_()
            out[r:r + rows, c] = (p @ vh) / p.sum(1, keepdim=True)
            del p
    return out


def _block64(x, w, H, grid, idx, ctx, t_mod, scale, gamma_o):
    """The block on x (float64), written out; large products in slices of rows."""
    D = x.shape[1]
    sh1, sc1, g1, sh2, sc2, g2 = _f(w["mod_table"]) + _f(t_mod)
    h = _layernorm(x) * (1 + sc1) + sh1
    wq, bq = w["w_qkv"], w["b_qkv"]
    q = _rope(_rms(_linear(h, wq[:D], bq[:D]), w["g_q"]), idx, grid, H)
    k = _rope(_rms(_linear(h, wq[D:2 * D], bq[D:2 * D]), w["g_k"]), idx, grid, H)
    v = _linear(h, wq[2 * D:], bq[2 * D:])
    del h
    x = x + g1 * _linear(_attend(q, k, v, H), w["w_o"], w["b_o"])
    del q, k, v
    qc = _rms(_linear(_layernorm(x) * _f(w["ln3_w"]) + _f(w["ln3_b"]), w["w_cq"], w["b_cq"]), w["g_cq"])
    kc = _rms(_linear(_f(ctx), w["w_ckv"][:D], w["b_ckv"][:D]), w["g_ck"])
    vc = _linear(_f(ctx), w["w_ckv"][D:], w["b_ckv"][D:])
    x = x + gamma_o * _linear(_attend(qc, kc, vc, H, scale), w["w_co"], w["b_co"])
    del qc
    for r in range(0, x.shape[0], 8192):
        y = x[r:r + 8192]
        y += g2 * _linear(_gelu(_linear(_layernorm(y) * (1 + sc2) + sh2, w["w_1"], w["b_1"])), w["w_2"], w["b_2"])
    return x


def _patches(latent):
    C, T, H, W = latent.shape
    return latent.view(C, T, H // 2, 2, W // 2, 2).permute(1, 2, 4, 0, 3, 5).reshape(-1, 4 * C)


def _unpatch(tok, shape):
    C, T, H, W = shape
    return tok.view(T, H // 2, W // 2, C, 2, 2).permute(3, 0, 1, 4, 2, 5).reshape(shape)


def _head64(x, w, t_head):
    sh, sc = _f(w["head_table"]) + _f(t_head)
    return _linear(_layernorm(x) * (1 + sc) + sh, w["w_head"], w["b_head"])


def _coef64(i, second):
    """DPM-Solver++ weights of the step from _SIGMAS[i]: sigma, rho, A, c0, c1."""
    s, t = _SIGMAS[i], _SIGMAS[i + 1]
    lam = lambda v: math.log((1 - v) / v)  # noqa: E731
    c0, c1 = 1.0, 0.0
    if second and i > 0 and t > 0 and _SIGMAS[i - 1] < 1:
        inv2r = (lam(t) - lam(s)) / (2 * (lam(s) - lam(_SIGMAS[i - 1])))
        c0, c1 = 1 + inv2r, -inv2r
    return s, t / s, (1 - t) - t * (1 - s) / s, c0, c1


def _update64(tok, prev, idx, v, coef, hist, SL, edit):
    """Sampler update of the token rows idx of `tok`, history and Eq. 6; returns (tok, prev)."""
    sigma, rho, A, c0, c1 = coef
    tok, prev = tok.clone(), prev.clone()
    x = tok[idx]
    x0 = x - sigma * v
    d = x0
    if c1:
        second = torch.ones(len(idx), dtype=torch.bool, device=tok.device) if hist is None else hist[idx] != 0
        d = torch.where(second[:, None], c0 * x0 + c1 * prev[idx], x0)
    new = rho * x + A * d
    if edit is not None:
        new = torch.where((edit[idx] != 0)[:, None], new, SL[idx])
    tok[idx], prev[idx] = new, x0
    return tok, prev


def _request64(s):
    case = s["case"]
    D, H, _, _ = _WIDTHS[case["width"]]
    grid, shape = (case["T"], case["Hg"], case["Wg"]), tuple(s["noise"].shape)
    project = lambda t: _linear(_gelu(_linear(_f(t), s["gw"]["w_text1"], s["gw"]["b_text1"])), s["gw"]["w_text2"], s["gw"]["b_text2"])  # noqa: E731
    ctx = project(s["text"])
    ctx_u = project(s["text_u"]) if case["cfg"] else None
    silu = torch.nn.functional.silu
    SL = _patches(_f(s["cache_latents"][s["near"], 0]))
    tok, prev, hist = SL, torch.zeros_like(SL), None
    w = torch.pow(torch.tensor(10000.0, dtype=torch.float64, device=SL.device), -torch.arange(128, dtype=torch.float64, device=SL.device) / 128)
    multi = case["solver"] == 2 or case["cfg"]
    for i in (1, 2, 3):  # step 0 is reused
        a = 1000.0 * _SIGMAS[i] * w
        e = _linear(silu(_linear(torch.cat((a.cos(), a.sin())), s["tw"]["w_t1"], s["tw"]["b_t1"])), s["tw"]["w_t2"], s["tw"]["b_t2"])
        t_mod = _linear(silu(e), s["tw"]["w_tp"], s["tw"]["b_tp"]).view(6, D)
        stage2 = i == 1
        idx = s["see"].nonzero()[:, 0] if stage2 else torch.arange(tok.shape[0], device=tok.device)
        scale = torch.where(s["tdiff"] != 0, 1.5, 1.0) if stage2 else None
        x = xu = _linear(tok[idx], s["gw"]["w_patch"], s["gw"]["b_patch"])
        for b in s["w"]:
            x = _block64(x, b, H, grid, idx, ctx, t_mod, scale, 1.5 if stage2 else 1.0)
            if case["cfg"]:
                xu = _block64(xu, b, H, grid, idx, ctx_u, t_mod, None, 1.0)
        v = _head64(x, s["gw"], torch.stack((e, e)))
        if case["cfg"]:
            u = _head64(xu, s["gw"], torch.stack((e, e)))
            v = u + 2.0 * (v - u)
        coef = _coef64(i, case["solver"] == 2 and i > 1) if multi else (_SIGMAS[i],) + _coef64(i, False)[1:]
        tok, prev = _update64(tok, prev, idx, v, coef, hist, SL if stage2 else None, s["edit"] if stage2 else None)
        hist = s["see"] if stage2 else None
    return {"latent": _unpatch(tok, shape), "index": None, "K1": None, "K2": None, "Ls": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "masks":
        return None
    s = prepare(case, seed)
    if kind in ("lookup", "lowprec"):
        c, q = _f(s["cache"]), _f(s["query"])
        return {"index": None, "score": ((c @ q) / c.norm(dim=1) / q.norm()).max().view(1), "hit": None}
    if kind == "batch":
        c, q = _f(s["cache"]), _f(s["queries"])
        best = ((q @ c.T) / c.norm(dim=1) / q.norm(dim=1, keepdim=True)).topk(case["k"], dim=1).values
        return {"index": None, "score": best, "hit": None}
    if kind == "request":
        return _request64(s)
    D, H, _, _ = _WIDTHS[case["width"]]
    grid = (case["T"], case["Hg"], case["Wg"])
    idx = s["idx"].long() if s["idx"] is not None else torch.arange(case["tokens"], device=DEV)
    if kind == "block":
        s["ws"] = s["kv"] = None
        return _block64(_f(s["x"]), s["w"], H, grid, idx, s["ctx"], s["t_mod"], s["scale"], s["gamma_o"])
    tok = _patches(_f(s["latent"]))
    x = _linear(tok[idx], s["w"]["w_patch"], s["w"]["b_patch"])
    v = _head64(x, s["w"], s["t_head"])
    if case["cfg"]:
        u = _head64(_f(s["x_uncond"]), s["w"], s["t_head"])
        v = u + _GUIDANCE * (v - u)
    tok, prev = _update64(tok, _patches(_f(s["x0_prev"])), idx, v, _coef64(2, True), s["hist"],
                          _patches(_f(s["SL"])) if s["SL"] is not None else None, s["edit"])
    shape = tuple(s["latent"].shape)
    return {"x": x, "latent": _unpatch(tok, shape), "x0_prev": _unpatch(prev, shape)}
